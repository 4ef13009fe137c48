// Attention of few rows over many keys (the same results as attn_fwd.hpp up to the rounding of the probabilities).
//
// The kernel of attn_fwd.hpp gives a wave 32 rows and all of its workgroup's keys.  Where a launch has few row tiles (one new
// token per sequence, a short prompt) that leaves the chip to a handful of waves, each with a long walk.  Here
// the eight waves of a workgroup are RG groups of 32 packed (token, head of the KV group) rows times KG = 8 / RG shares of the
// keys: share x takes the 32-key blocks x, x + KG, ... and the KG partial rows meet in LDS at the end.  With one
// row group a wave has LDS slots of its own and meets no barrier; with more, the waves of a share load its blocks together,
// four steps of KG blocks in rotation and one barrier a step, in the pipeline of attn_fwd_kernel.
// Whole, RG = 1: bound by the latency of one block's chain (request, scores, exponentials, PV), of which four (head_dim 64) or two
// waves share a SIMD: 1 token over 1 key 9.6 -> 6.4 us, 512 tokens x 1 head of 64 9.6 -> 6.3, 2000 x 8/8 of 128 31 -> 21.
// Divided, RG = 1 (one token per sequence): bound by HBM, every wave with requests of its own in flight: 8 sequences x 1 token,
// 97 MB of K and V, 27 to 31 (attn_fwd_kernel's tiles: one wave of four had rows) -> 21.6 us, 4.5 TB/s of a copy's 4.9.
// Divided, RG = 4 (chunks): bound by the matrix pipe and the exponentials of one workgroup per compute unit: 5 to 64 tokens x 4 behind
// 700 to 12345 keys, 32/8 heads 49 -> 35 us, from pieces that are as long as each other instead of 128 rows by a length for the
// longest sequence.  attn_join_kernel follows in 4 to 6 us.  As far from the result in 64 bits as the other forms (2.3e-3 of O).
#pragma once
#include "attn_fwd.hpp"
#include "wave_scan.hpp"

namespace pdd {

constexpr int kRowsWaves = 8;
template <int D, int RG>
struct RowsSmem {
    static constexpr int BLOCK = 32 * 2 * D;                        // a K or V block of 32 keys
    static constexpr int SLOTS = RG == 1 ? 1 : 4;                   // K and V blocks of a share
    static constexpr int BLOCKS = kRowsWaves / RG * SLOTS * 2 * BLOCK;
    // the rows of Q: behind the blocks, or (RG = 4) in the shares' last slots, two groups each
    static constexpr int q_at(int group) { return RG == 1 ? BLOCKS : (group >> 1) * SLOTS * 2 * BLOCK + (SLOTS - 1) * 2 * BLOCK + (group & 1) * BLOCK; }
    static constexpr int SUMS = BLOCKS + (RG == 1 ? BLOCK : 0);
    static constexpr int BYTES = SUMS + kRowsWaves * 32 * (int)sizeof(float2);
};

// a sequence's part: packed rows, tiles of ROWS of them, 64-key tiles
struct WorkSeq { int qs, ks, nq, nk, row_tiles, key_tiles; };
template <int ROWS>
__device__ __forceinline__ WorkSeq work_seq(const AttnParams &p, int b)
{
    WorkSeq s = {0, 0, 0, 0, 0, 0};
    if (b < p.B) {
        s.qs = min(p.cu_q[b], p.total_q);
        s.nq = min(p.cu_q[b + 1], p.total_q) - s.qs;
        s.ks = min(p.cu_k[b], p.total_k);
        s.nk = min(p.cu_k[b + 1], p.total_k) - s.ks;
        if (s.nq > 0) {
            s.row_tiles = (s.nq * p.G + ROWS - 1) / ROWS;
            s.key_tiles = max((s.nk + kBN - 1) / kBN, 1);
        }
    }
    return s;
}

// How the keys are divided: the key tiles of a (sequence, row tile) pair are cut into pieces of about `per` tiles, so that the
// pieces of all pairs are p.workers to a KV head at most, or p.min_tiles long.  Piece x of a sequence leaves its `nq` partial
// token rows from row `part + x nq` on.  Everything follows from the lengths, so every wave finds the same.
struct WorkPlace { uint32_t first, part; };                 // of a sequence: number of its first piece, its first partial row
__device__ __forceinline__ int pieces_of(int key_tiles, uint32_t per) { return (int)((key_tiles + per - 1) / per); }
template <int ROWS>
__device__ __forceinline__ uint32_t work_per(const AttnParams &p, const WorkSeq &mine, int lane)
{
    uint32_t tiles = 0, token_tiles = 0, pairs = 0;
    for (int b0 = 0; b0 < p.B; b0 += 64) {
        const WorkSeq s = b0 == 0 ? mine : work_seq<ROWS>(p, b0 + lane);
        uint32_t x[3] = {(uint32_t)s.row_tiles * s.key_tiles, (uint32_t)max(s.nq, 0) * s.key_tiles, (uint32_t)s.row_tiles};
        wave_incl_scan_n(x);
        tiles += (uint32_t)__builtin_amdgcn_readlane((int)x[0], 63);
        token_tiles += (uint32_t)__builtin_amdgcn_readlane((int)x[1], 63);
        pairs += (uint32_t)__builtin_amdgcn_readlane((int)x[2], 63);
    }
    // a pair has one piece more than per goes into its tiles, at most; p.workers > pairs, p.part_rows > p.total_q
    const uint32_t room = (uint32_t)(p.part_rows - p.total_q), spare = max((uint32_t)p.workers, pairs + 1) - pairs;
    return max(max((token_tiles + room - 1) / room, (tiles + spare - 1) / spare), (uint32_t)p.min_tiles);
}
// exclusive sums over the lanes' sequences, on top of what the sequences before them take
__device__ __forceinline__ WorkPlace work_place(const WorkSeq &s, uint32_t per, WorkPlace &before)
{
    const uint32_t pieces = (uint32_t)pieces_of(s.key_tiles, per), own[2] = {s.row_tiles * pieces, max(s.nq, 0) * pieces};
    uint32_t x[2] = {own[0], own[1]};
    wave_incl_scan_n(x);
    const WorkPlace at = {before.first + x[0] - own[0], before.part + x[1] - own[1]};
    before.first += (uint32_t)__builtin_amdgcn_readlane((int)x[0], 63);
    before.part += (uint32_t)__builtin_amdgcn_readlane((int)x[1], 63);
    return at;
}
__device__ __forceinline__ WorkSeq work_seq_of_lane(const WorkSeq &s, int l)
{
    return {__builtin_amdgcn_readlane(s.qs, l), __builtin_amdgcn_readlane(s.ks, l), __builtin_amdgcn_readlane(s.nq, l),
            __builtin_amdgcn_readlane(s.nk, l), __builtin_amdgcn_readlane(s.row_tiles, l), __builtin_amdgcn_readlane(s.key_tiles, l)};
}
// key tiles that the last row of a row tile sees (its packed row number given)
__device__ __forceinline__ int tiles_seen(const AttnParams &p, const WorkSeq &s, int last_row)
{
    return max(min(s.nk, div_group(max(last_row, 0), p.g_magic) + 1 + s.nk - s.nq) + kBN - 1, 0) / kBN;
}

template <int D, int RG, bool DIVIDED>
__global__ __launch_bounds__(kRowsWaves * 64) __attribute__((amdgpu_waves_per_eu(D == 64 && RG == 1 ? 4 : 2, D == 64 && RG == 1 ? 4 : 2)))
void attn_rows_kernel(const AttnParams p)
{
    static_assert(DIVIDED || RG == 1, "whole key ranges: one row group to a workgroup");
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int ROWB = 2 * D, CH = D / 8, RPI = 1024 / ROWB;
    constexpr int KG = kRowsWaves / RG, ROWS = 32 * RG, SLOTS = RowsSmem<D, RG>::SLOTS;
    constexpr int BLOCK = RowsSmem<D, RG>::BLOCK;
    constexpr int NKK = D / 16, NDB = D / 32;
    constexpr int NB = 32 / RPI, NL = NB / RG;                      // transfers of a block, of each wave of its share
    constexpr int FCH = D / 4;                                      // 16-byte chunks of a 32-bit row
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem_rows[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int share = wave / RG, group = wave % RG;
    const int n = lane & 31, hh = lane >> 5;
    uint8_t *const slots = smem_rows + share * SLOTS * 2 * BLOCK;   // of the share: K block, V block, K block, ...
    const uint32_t slots_lds = lds_addr_of(slots);
    float2 *const sums = (float2 *)(smem_rows + RowsSmem<D, RG>::SUMS);  // [wave][row]: reference exponent, sum

    int bid = blockIdx.x;
    const int g = bid % p.Hkv;  bid /= p.Hkv;
    const uint32_t k_row_bytes = (uint32_t)p.k_st * 2u, v_row_bytes = (uint32_t)p.v_st * 2u, q_row_bytes = (uint32_t)p.q_st * 2u;
    // transfer number x of a block brings its rows RPI x ..: lane -> row RPI x + lane / CH, chunk position lane % CH, which
    // holds chunk pos ^ swz(row)
    uint32_t kvoff[NL], vvoff[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        const int r = RPI * (group + RG * i) + lane / CH;
        const uint32_t c = (uint32_t)((lane % CH) ^ swz_row<D>(r)) * 16u;
        kvoff[i] = (uint32_t)r * k_row_bytes + c;
        vvoff[i] = (uint32_t)r * v_row_bytes + c;
    }
    uint32_t kaddr[NKK], vaddr[NDB][2];                             // fragment reads, see attn_fwd_kernel
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) kaddr[kk] = (uint32_t)(n * ROWB + ((2 * kk + hh) ^ swz_row<D>(n)) * 16);
#pragma unroll
    for (int eg = 0; eg < 2; ++eg) {
        const int s16 = lane & 15, row = 8 * eg + 4 * hh + (s16 >> 2);
#pragma unroll
        for (int db = 0; db < NDB; ++db) {
            const int chunk = 4 * db + 2 * ((lane >> 4) & 1) + ((s16 & 3) >> 1);
            vaddr[db][eg] = slots_lds + BLOCK + (uint32_t)(row * ROWB + (chunk ^ swz_row<D>(row)) * 16) + 8u * (s16 & 1);
            asm volatile("" : "+v"(vaddr[db][eg]));          // kept whole, see attn_fwd_kernel
        }
    }
    const float c2 = p.scale_log2;
    const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

    // Row tile rt of a sequence against its key tiles t0 .. t1 - 1.  whole: these are all that the rows see, and the
    // result is final; else it goes to the partial rows from token row part_row on.
    auto run = [&](const WorkSeq &s, int rt, int t0, int t1, bool whole, int64_t part_row) __attribute__((always_inline)) {
        const int n_rows = s.nq * p.G, m0 = n_rows - (s.row_tiles - rt) * ROWS;           // tiles are aligned to the end
        const int delta = s.nk - s.nq, k0 = t0 * kBN;
        const int last_tok = div_group(max(m0 + ROWS - 1, 0), p.g_magic);
        const int n_keys = min(min(s.nk, last_tok + 1 + delta), t1 * kBN) - k0;
        const int n_blocks = max(n_keys + 31, 0) / 32;
        const int w0 = m0 + 32 * group;                               // the wave's rows
        const int row = max(w0 + n, 0), tok = div_group(row, p.g_magic);
        const int lim = min(tok + delta - k0, n_keys - 1);            // last key of this lane's row
        const int lim_min = min(div_group(max(w0, 0), p.g_magic) + delta - k0, n_keys - 1);
        const int lim_max = min(div_group(max(w0 + 31, 0), p.g_magic) + delta - k0, n_keys - 1);
        const uint16_t *kbase = p.k + (int64_t)(s.ks + k0) * p.k_st + (int64_t)g * p.k_sh;
        const uint16_t *vbase = p.v + (int64_t)(s.ks + k0) * p.v_st + (int64_t)g * p.v_sh;
        const uint32_t k_span = n_keys > 0 ? (uint32_t)(n_keys - 1) * k_row_bytes + (uint32_t)ROWB : 0u;
        const uint32_t v_span = n_keys > 0 ? (uint32_t)(n_keys - 1) * v_row_bytes + (uint32_t)ROWB : 0u;
        auto issue = [&](const uint16_t *base, uint32_t span, uint32_t row_bytes, const uint32_t (&voff)[NL], int blk, uint32_t lds) {
            const uint32_t so = min((uint32_t)blk * 32u * row_bytes, span);      // past the last block: nothing, reads as zero
            const i32x4 rs = make_rsrc((const uint8_t *)base + so, span - so);
#pragma unroll
            for (int i = 0; i < NL; ++i) dma16_to_lds(rs, lds + 1024 * (group + RG * i), voff[i]);
        };
        auto issue_k = [&](int blk, int at) { issue(kbase, k_span, k_row_bytes, kvoff, blk, slots_lds + at * 2 * BLOCK); };
        auto issue_v = [&](int blk, int at) { issue(vbase, v_span, v_row_bytes, vvoff, blk, slots_lds + at * 2 * BLOCK + BLOCK); };
        // ---- the rows of Q, shared by the shares: a transfer or two each
        const int n_steps = (n_blocks + KG - 1) / KG;
        const bool works = share < n_blocks && w0 + 31 >= 0;
#pragma unroll
        for (int i = 0; i < (RG * NB + kRowsWaves - 1) / kRowsWaves; ++i) {
            const int x = wave + kRowsWaves * i;
            if (x < RG * NB) {
                const int q_first = div_group(max(m0, 0), p.g_magic);
                const uint16_t *qbase = p.q + (int64_t)(s.qs + q_first) * p.q_st + (int64_t)(g * p.G) * p.q_sh;
                const int q_last = div_group(m0 + ROWS - 1, p.g_magic);
                const uint32_t q_span = (uint32_t)(q_last - q_first) * q_row_bytes + (uint32_t)(p.G - 1) * (uint32_t)p.q_sh * 2u + (uint32_t)ROWB;
                const int r = RPI * x + lane / CH, rr = max(m0 + r, 0), ri = div_group(rr, p.g_magic);
                const uint32_t c = (uint32_t)((lane % CH) ^ swz_row<D>(r & 31)) * 16u;
                dma16_to_lds(make_rsrc(qbase, q_span), lds_addr_of(smem_rows) + (uint32_t)(RowsSmem<D, RG>::q_at(x / NB) + 1024 * (x % NB)),
                             (uint32_t)(ri - q_first) * q_row_bytes + (uint32_t)(rr - ri * p.G) * (uint32_t)p.q_sh * 2u + c);
            }
        }
        if constexpr (RG == 1) {
            if (works) {
                issue_k(share, 0);
                issue_v(share, 0);
                asm volatile("s_waitcnt vmcnt(%0)" : : "n"(2 * NL) : "memory");
            } else {
                __builtin_amdgcn_s_waitcnt(0);
            }
        } else {                                                      // a wave without rows still loads its part
            issue_k(share, 0);
            issue_k(share + KG, 1);
            issue_v(share, 0);
            issue_k(share + 2 * KG, 2);
            asm volatile("s_waitcnt vmcnt(%0)" : : "n"(2 * NL) : "memory");
        }
        __syncthreads();
        bf16x8 qf[NKK];
#pragma unroll
        for (int kk = 0; kk < NKK; ++kk) qf[kk] = *(const bf16x8 *)(smem_rows + RowsSmem<D, RG>::q_at(group) + kaddr[kk]);

        // Online softmax in the log2 domain with a lagging reference, as in attn_fwd_kernel.
        f32x16 oacc[NDB];
#pragma unroll
        for (int db = 0; db < NDB; ++db) oacc[db] = zero16;
        float l_part[4] = {0.f, 0.f, 0.f, 0.f}, ref = 0.f, thr = -INFINITY;
        auto to_log2 = [&](f32x16 &x) {
#pragma unroll
            for (int e = 0; e < 16; ++e) x[e] = fmaf(x[e], c2, ref);
        };
        auto mask = [&](f32x16 &x, int l) {                           // key 8 (e / 4) + e % 4 (+ 4 hh, in l) is hidden beyond l
#pragma unroll
            for (int e = 0; e < 16; ++e) x[e] = 8 * (e >> 2) + (e & 3) > l ? -INFINITY : x[e];
        };
        auto row_max = [&](const f32x16 &x) {
            const float t0 = max3(x[0], x[1], x[2]), t1 = max3(x[4], x[5], x[6]);
            const float t2 = max3(x[8], x[9], x[10]), t3 = max3(x[12], x[13], x[14]);
            const float u0 = max3(t0, t1, x[3]), u1 = max3(t2, t3, x[7]);
            const float t_max = max3(max3(u0, u1, x[11]), x[15], x[15]);
            return fmaxf(t_max, xchg_half(t_max));
        };
        auto renew = [&](float t_max, f32x16 &x) {                    // where a row exceeds its threshold (see attn_fwd_kernel)
            if (!__any(t_max > thr)) return;
            const bool up = t_max > thr;
            const float shift = up ? t_max : 0.f;
            const float alpha = fast_exp2(-fmaxf(shift, 0.f));        // (a first reference rescales nothing)
#pragma unroll
            for (int q = 0; q < 4; ++q) l_part[q] *= alpha;
#pragma unroll
            for (int db = 0; db < NDB; ++db)
#pragma unroll
                for (int e = 0; e < 16; ++e) oacc[db][e] *= alpha;
#pragma unroll
            for (int e = 0; e < 16; ++e) x[e] -= shift;
            ref -= shift;
            thr = up ? kLazyLog2 : thr;
        };
        bf16x8 kf[NKK], vf[2][NDB], pb[2];
        auto read_k = [&](int at) {
#pragma unroll
            for (int kk = 0; kk < NKK; ++kk) kf[kk] = *(const bf16x8 *)(slots + at * 2 * BLOCK + kaddr[kk]);
        };
        auto read_v = [&](int at) {
#pragma unroll
            for (int st = 0; st < 2; ++st)
#pragma unroll
                for (int db = 0; db < NDB; ++db)
                    vf[st][db] = lds_read_tr8(vaddr[db][0] + at * 2 * BLOCK + 16 * ROWB * st, vaddr[db][1] + at * 2 * BLOCK + 16 * ROWB * st);
        };
        auto qk = [&](f32x16 &x) {
#pragma unroll
            for (int kk = 0; kk < NKK; ++kk) x = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kk], qf[kk], kk == 0 ? zero16 : x, 0, 0, 0);
        };
        auto pack = [&](f32x16 &x) {                                  // probabilities
#pragma unroll
            for (int e = 0; e < 16; ++e) x[e] = fast_exp2(x[e]);
#pragma unroll
            for (int st = 0; st < 2; ++st) {
                f32x8 pf;
#pragma unroll
                for (int e = 0; e < 8; ++e) pf[e] = x[8 * st + e];
                pb[st] = __builtin_convertvector(pf, bf16x8);
            }
        };
        auto add_sums = [&](const f32x16 &x) {
#pragma unroll
            for (int e = 0; e < 16; ++e) l_part[e & 3] += x[e];
        };
        auto add_pv = [&](int first, int last) {
#pragma unroll
            for (int i = first; i < last; ++i)
                oacc[i % NDB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[i / NDB][i % NDB], pb[i / NDB], oacc[i % NDB], 0, 0, 0);
        };
        const int lim4 = lim - 4 * hh;
        if constexpr (RG == 1) {
            for (int i = wave; i < n_blocks; i += KG) {
                const bool more = i + KG < n_blocks;
                asm volatile("s_waitcnt vmcnt(%0)" : : "n"(NL) : "memory");       // K has landed, V may be on its way
                read_k(0);
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                if (more) issue_k(i + KG, 0);
                f32x16 x = zero16;
                qk(x);
                to_log2(x);
                if (32 * i + 31 > lim_min) mask(x, lim4 - 32 * i);
                renew(row_max(x), x);
                pack(x);
                add_sums(x);
                if (more) asm volatile("s_waitcnt vmcnt(%0)" : : "n"(NL) : "memory");
                else __builtin_amdgcn_s_waitcnt(0);
                read_v(0);
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                if (more) issue_v(i + KG, 0);
                add_pv(0, 2 * NDB);
            }
        } else {
            // Block `share` of step 0 enters the log2 domain here; a step then takes the exponentials and PV products of its
            // block while the scores of the next one are formed, K fragments read another step ahead.
            f32x16 sA = zero16, sB = zero16;
            read_k(0);
            qk(sA);
            read_k(1);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __syncthreads();                                         // Q and K blocks 0 and 1 are read
            issue_v(share + KG, 1);
            issue_k(share + 3 * KG, 3);
            issue_v(share + 2 * KG, 2);
            issue_k(share + 4 * KG, 0);
            to_log2(sA);
            if (32 * share + 31 > lim_min) mask(sA, lim4 - 32 * share);
            renew(row_max(sA), sA);
            const bool has_rows = w0 + 31 >= 0;
            auto step = [&](auto at_c, int j) __attribute__((always_inline)) {
                constexpr int AT = decltype(at_c)::value;
                const int i = j * KG + share;
                // all but the two youngest steps' blocks have landed: V of this step, K of the one after the next
                asm volatile("s_waitcnt vmcnt(%0)" : : "n"(4 * NL) : "memory");
                __syncthreads();                                     // and the last step's are read
                issue_v(i + 3 * KG, (AT + 3) % 4);
                issue_k(i + 5 * KG, (AT + 1) % 4);
                if (has_rows && 32 * i <= lim_max) {
                    f32x16 &cur = AT & 1 ? sB : sA, &nxt = AT & 1 ? sA : sB;
                    const int k_next = 32 * (i + KG);
                    __builtin_amdgcn_s_setprio(1);
                    read_v(AT);
                    qk(nxt);
                    pack(cur);
#pragma unroll
                    for (int x = 0; x < NKK; ++x) {                  // issue order as in attn_fwd_kernel
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);          // 1 MFMA
                        __builtin_amdgcn_sched_group_barrier(0x400, 16 / NKK, 0);   // transcendental
                        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);          // 2 DS reads
                        __builtin_amdgcn_sched_group_barrier(0x002, 8 / NKK, 0);    // VALU (bf16 packs)
                    }
                    __builtin_amdgcn_s_setprio(0);
                    read_k((AT + 2) % 4);
                    constexpr int NA = 2 * NDB - 2;                  // PV MFMAs before the mask's branch
                    add_pv(0, NA);
                    add_sums(cur);
                    to_log2(nxt);
#pragma unroll
                    for (int x = 0; x < NA; ++x) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                    // 1 MFMA
                        __builtin_amdgcn_sched_group_barrier(0x100, (NKK + NA - 1) / NA, 0);  // DS reads
                        __builtin_amdgcn_sched_group_barrier(0x002, (32 + NA - 1) / NA, 0);   // VALU
                    }
                    asm volatile("" : "+v"(l_part[0]), "+v"(l_part[1]), "+v"(l_part[2]), "+v"(l_part[3]));
                    if (k_next + 31 > lim_min) {
                        asm volatile("" ::: "memory");               // stays a branch
                        mask(nxt, lim4 - k_next);
                    }
                    add_pv(NA, 2 * NDB);
                    const float t_max = row_max(nxt);
#pragma unroll
                    for (int x = NA; x < 2 * NDB; ++x) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);          // 1 MFMA
                        __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);          // VALU
                    }
                    renew(t_max, nxt);
                }
            };
            for (int j = 0; j < n_steps; j += 4) {
                step(std::integral_constant<int, 0>{}, j);
                if (j + 1 < n_steps) step(std::integral_constant<int, 1>{}, j + 1);
                if (j + 2 < n_steps) step(std::integral_constant<int, 2>{}, j + 2);
                if (j + 3 < n_steps) step(std::integral_constant<int, 3>{}, j + 3);
            }
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();                                         // the rows below overwrite the slots
        }

        // ---- the shares' partial rows meet: references and sums first, then the rows, scaled to the common one
        const float l_run = (l_part[0] + l_part[1]) + (l_part[2] + l_part[3]), l_tot = l_run + xchg_half(l_run);
        const bool empty = __float_as_uint(l_tot) == 0u;             // (as bits: a NaN sum is none)
        if (works && hh == 0) sums[wave * 32 + n] = make_float2(empty ? -INFINITY : -ref, l_tot);
        __syncthreads();
        const int active = min(n_blocks, KG);                        // shares with a block
        float top = -INFINITY;
        for (int x = 0; x < active; ++x) top = fmaxf(top, sums[(group + RG * x) * 32 + n].x);
        top = top > -INFINITY ? top : 0.f;                            // a row that sees no key
        float total = 0.f;
        for (int x = 0; x < active; ++x) {
            const float2 t = sums[(group + RG * x) * 32 + n];
            total += fast_exp2(t.x - top) * t.y;
        }
        if (works) {
            const float scale = fast_exp2((empty ? -INFINITY : -ref) - top) * (total > 0.f ? 1.f / total : 0.f);
            uint8_t *const dst = smem_rows + wave * 2 * BLOCK;
#pragma unroll
            for (int db = 0; db < NDB; ++db)
#pragma unroll
                for (int bq = 0; bq < 4; ++bq) {
                    f32x4 x;
#pragma unroll
                    for (int r = 0; r < 4; ++r) x[r] = oacc[db][4 * bq + r] * scale;
                    *(f32x4 *)(dst + n * 2 * ROWB + (((8 * db + 2 * bq + hh) ^ (n & (FCH - 1))) * 16)) = x;
                }
        }
        if (share == 0 && hh == 0 && w0 + n >= 0) {
            const int h = g * p.G + row - tok * p.G;
            const float lse2 = __builtin_amdgcn_logf(total) + top;
            if (whole) p.lse[(int64_t)h * p.total_q + s.qs + tok] = total > 0.f ? lse2 * 0.6931471805599453f : -INFINITY;
            else p.part_l[(part_row + tok) * p.Hq + h] = __float_as_uint(total) == 0u ? -INFINITY : lse2;
        }
        __syncthreads();
        constexpr int ITEMS = ROWS * FCH / (kRowsWaves * 64);         // 16-byte chunks of the rows, per thread
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const int x = tid + i * kRowsWaves * 64, r = x / FCH, c = x % FCH, rr = m0 + r;
            const uint8_t *src = smem_rows + (r >> 5) * 2 * BLOCK + (r & 31) * 2 * ROWB + ((c ^ (r & 31 & (FCH - 1))) * 16);
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
            if (rr >= 0) {
                if constexpr (RG == 1) {
                    for (int y = 0; y < active; ++y) acc += *(const f32x4 *)(src + y * 2 * BLOCK);
                } else {
                    if (active > 0) acc = *(const f32x4 *)src;
                    if (active > 1) acc += *(const f32x4 *)(src + RG * 2 * BLOCK);
                }
                const int ri = div_group(rr, p.g_magic), h = g * p.G + rr - ri * p.G;
                if (whole) *(bf16x4 *)(p.o + (int64_t)(s.qs + ri) * p.o_st + (int64_t)h * p.o_sh + 4 * c) = __builtin_convertvector(acc, bf16x4);
                else *(f32x4 *)(p.part_o + ((part_row + ri) * p.Hq + h) * D + 4 * c) = acc;
            }
        }
    };

    if constexpr (!DIVIDED) {
        // a workgroup per (KV head, sequence, row tile), the longest walks first
        int rt_back;
        const int b = sequence_of(bid, p.B, p.n_qtiles, p.turn, rt_back);
        WorkSeq s = work_seq<ROWS>(p, b);
        s.qs = __builtin_amdgcn_readfirstlane(s.qs);  s.ks = __builtin_amdgcn_readfirstlane(s.ks);
        s.nq = __builtin_amdgcn_readfirstlane(s.nq);  s.nk = __builtin_amdgcn_readfirstlane(s.nk);
        const int rt = s.row_tiles - 1 - rt_back;
        if (rt < 0) return;
        run(s, rt, 0, s.key_tiles, true, 0);
    } else {
        WorkSeq seqs = work_seq<ROWS>(p, lane);
        if (bid == 0) {
            // Tokens before the first sequence or behind the last one, if there are any, are left alone: final for attn_join_kernel,
            // which would take what the scratch held for their entry.  (Asked there, by every row, a decoding step takes 0.4 us more.)
            const int begin = min(max(p.cu_q[0], 0), p.total_q), end = min(max(p.cu_q[p.B], begin), p.total_q);
            for (int x = tid; x < (p.total_q - end + begin) * p.G; x += kRowsWaves * 64) {
                const int t = x / p.G, tok = t < begin ? t : t - begin + end;
                p.part_of[(int64_t)tok * p.Hq + g * p.G + x - t * p.G] = make_uint4(0u, 0u, 1u, 0u);
            }
        }
        const uint32_t per = work_per<ROWS>(p, seqs, lane);
        WorkPlace before = {0, 0};
        for (int b0 = 0; b0 < p.B; b0 += 64) {
            if (b0 > 0) seqs = work_seq<ROWS>(p, b0 + lane);
            const WorkPlace places = work_place(seqs, per, before);
            if ((uint32_t)bid >= before.first) continue;
            const int l = 63 - __builtin_clzll(__ballot(places.first <= (uint32_t)bid && seqs.key_tiles > 0));
            const WorkSeq s = work_seq_of_lane(seqs, l);
            // the row tiles of a piece, which read the same keys, then those of the next one; a piece takes its share of the key tiles
            const int x = bid - __builtin_amdgcn_readlane((int)places.first, l), pieces = pieces_of(s.key_tiles, per);
            const int piece = x / s.row_tiles, rt = x - piece * s.row_tiles;
            const int t0 = s.key_tiles * piece / pieces, t1 = s.key_tiles * (piece + 1) / pieces;
            const int seen = tiles_seen(p, s, s.nq * p.G - 1 - (s.row_tiles - 1 - rt) * ROWS);
            const uint32_t part = (uint32_t)__builtin_amdgcn_readlane((int)places.part, l);
            if ((uint64_t)part + (uint64_t)pieces * s.nq > (uint64_t)p.part_rows) return;    // (lengths that are none)
            if (piece == 0) {                            // what attn_join_kernel finds the rows' pieces by
                int n = seen > 0 ? pieces : 0;           // that see a key
                while (n > 1 && s.key_tiles * (n - 1) / pieces >= seen) --n;
                const int row = s.nq * p.G - (s.row_tiles - rt) * ROWS + tid;
                if (tid < ROWS && row >= 0) {
                    const int tok = div_group(row, p.g_magic), h = g * p.G + row - tok * p.G;
                    p.part_of[(int64_t)(s.qs + tok) * p.Hq + h] = make_uint4((part + tok) * p.Hq + h, (uint32_t)s.nq * p.Hq, (uint32_t)n, 0u);
                }
            }
            if (t0 < seen) run(s, rt, t0, t1, t0 == 0 && t1 >= seen, part + (uint32_t)piece * s.nq);
            return;
        }
    }
#else
    (void)p;
#endif
}

// Second kernel of a launch that divides the keys: output and log-sum-exp of every (token, query head) that has more
// than one piece, from its partial rows,
//   lse2 = log2 sum_x 2^lse2_x,   o = sum_x 2^(lse2_x - lse2) o_x.
// One wave per row: a lane fetches the log2-sum-exp2 of one piece (all of them are in flight at
// once, 64 at a time) and the wave reads 256 / D partial rows at a time, 16 bytes per lane, the first four
// steps before the weights are known.  Bound by latency with few rows, by HBM with many.
template <int D>
__global__ __launch_bounds__(256) void attn_join_kernel(const AttnParams p)
{
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int LPR = D / 4, SPS = 64 / LPR, AHEAD = 4;        // lanes per partial row, pieces per step, steps in flight
    const int lane = threadIdx.x & 63;
    const int64_t x = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // token * Hq + head
    if (x >= (int64_t)p.total_q * p.Hq) return;
    const uint4 of = p.part_of[x];
    const uint32_t first = __builtin_amdgcn_readfirstlane(of.x), stride = __builtin_amdgcn_readfirstlane(of.y);
    const int pieces = __builtin_amdgcn_readfirstlane(of.z);
    if (pieces == 1) return;                          // the first kernel's result is final
    // (lengths that are none have no entries)
    if (pieces < 0 || pieces > p.workers || first + (uint64_t)max(pieces - 1, 0) * stride >= (uint64_t)p.part_rows * p.Hq) return;
    const int sub = lane / LPR, c = lane % LPR;
    const float *pl = p.part_l + first, *po = p.part_o + (uint64_t)first * D + 4 * c;
    auto rows = [&](int y0, f32x4 (&o)[AHEAD]) {
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) {
            const int y = y0 + i * SPS + sub;
            o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (y < pieces) o[i] = *(const f32x4 *)(po + (uint64_t)y * stride * D);
        }
    };
    f32x4 o[AHEAD];
    rows(0, o);
    float lse = lane < pieces ? pl[(uint64_t)lane * stride] : -INFINITY, top = lse;
    for (int y = lane + 64; y < pieces; y += 64) top = fmaxf(top, pl[(uint64_t)y * stride]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) top = fmaxf(top, __shfl_xor(top, off, 64));
    const float base = top > -INFINITY ? top : 0.f;   // a row that sees no key: every weight is 0
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    float sum = 0.f;
    for (int y0 = 0; y0 < pieces; y0 += 64) {
        if (y0 > 0) lse = y0 + lane < pieces ? pl[(uint64_t)(y0 + lane) * stride] : -INFINITY;
        const float w = fast_exp2(lse - base);
        sum += w;
#pragma unroll 1
        for (int y = 0; y < 64 && y0 + y < pieces; y += AHEAD * SPS) {
            if (y0 + y > 0) rows(y0 + y, o);
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) acc += __shfl(w, y + i * SPS + sub, 64) * o[i];      // weight 0 past the last piece
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
#pragma unroll
    for (int off = 32; off >= LPR; off >>= 1)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] += __shfl_xor(acc[e], off, 64);
    if (sum > 0.f) acc *= 1.f / sum;
    const int tok = (int)(x / p.Hq), h = (int)(x - (int64_t)tok * p.Hq);
    if (lane < LPR)
        *(bf16x4 *)(p.o + (int64_t)tok * p.o_st + (int64_t)h * p.o_sh + 4 * c) = __builtin_convertvector(acc, bf16x4);
    if (lane == 0)
        p.lse[(int64_t)h * p.total_q + tok] =
            sum > 0.f ? (top + __builtin_amdgcn_logf(sum)) * 0.6931471805599453f : -INFINITY;
#else
    (void)p;
#endif
}

}  // namespace pdd
