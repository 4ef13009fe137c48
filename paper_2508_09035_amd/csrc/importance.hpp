// Token importance from the observation window (paper Section 3.2, "Prompt
// Refiner": the normalised attention weight of the last segment of queries
// against the entire K, summed along the query dimension).
//
//   imp[g, j] = sum_{h in group g} sum_{i in window, i + delta >= j}
//               exp(s <q_i, k_j> - lse[h, i])
//
// The final log-sum-exp of every window row is an input, so each probability
// is recomputed from one QK^T tile and added into a per-key column sum; the
// attention matrix is never stored.  Work is split over KEYS: a workgroup of 4
// waves owns 256 keys, each wave 64 of them (two 32-key groups whose K
// fragments stay in registers as B operands for the whole kernel); with KG = 1
// it owns 128 keys, one 32-key group per wave, which small launches prefer.  The window
// rows of the G query heads are streamed through LDS in blocks of 32 (token, head) rows
// (buffer_load ... lds, double buffered, swizzled like the attention K tile)
// together with their log-sum-exp values (four buffers, three blocks in flight:
// with little arithmetic per block the kernel lives on hiding the load latency),
// so every Q fragment read from LDS feeds KG MFMAs and every Q row is fetched
// from L2 once per workgroup.
// S = Q K^T puts key (l % 32) in lane l and 16 query rows in its accumulator
// registers, so the sum over queries is in-lane; no atomics, fixed summation
// order, deterministic.
#pragma once
#include "attn_fwd.hpp"
#include "wave_scan.hpp"
#include <type_traits>

namespace pdd {

struct ImpParams {
    const uint16_t *q, *k;
    const float *lse;
    float *imp;
    const int32_t *cu_q, *cu_k;
    int64_t q_st, q_sh, k_st, k_sh;
    int32_t B, Hq, Hkv, G, total_q, total_k, n_ktiles;
    int32_t turn;      // rows_per_turn of the KV heads
    int32_t window;    // < 0: every query is a window query
    float scale_log2;  // softmax scale * log2(e)
    // Row split: the window rows of a workgroup's keys are divided over n_split workgroups; with
    // n_split > 1 workgroup r writes its partial column sums to part[r][Hkv][total_k] (every
    // element of a sequence, zeros included) and importance_reduce_kernel adds them in the
    // fixed order r = 0, 1, ...
    int32_t n_split;
    float *part;
    int32_t scan;      // whether a workgroup finds its piece of the keys among the sequences' lengths
    uint32_t g_magic;  // ceil(2^32 / G), 0 where G = 1
    // Only read by importance_rows_kernel: 32-key groups per wave, and workgroups per KV head that are on the chip at
    // once where the groups follow from the sequences' rows too (0: they do not).
    int32_t groups, places;
};

constexpr int kImpWaves = 4;
constexpr int kImpBK = 64 * kImpWaves;  // keys per workgroup
constexpr int kImpBufs = 4;             // LDS ring of query-row blocks
constexpr int kImpAhead = 3;            // blocks in flight

// 4 bytes per lane from the buffer into LDS at lds_addr + 4 * lane (see dma16_to_lds)
__device__ __forceinline__ void dma4_to_lds(i32x4 rsrc, uint32_t lds_addr, uint32_t voff)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds"
                 :
                 : "s"(lds_addr), "v"(voff), "s"(rsrc)
                 : "memory", "m0");
}

template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}

template <int D, int KG = 2>
__global__ __launch_bounds__(kImpWaves * 64) __attribute__((amdgpu_waves_per_eu(3, 4)))
void importance_kernel(const ImpParams p)
{
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int NKK = D / 16;
    constexpr int ROW_BYTES = D * 2;             // one Q row in LDS
    constexpr int CH = D / 8;                    // 16-byte chunks per row
    constexpr int QBLK_BYTES = 32 * ROW_BYTES;   // one block of 32 query rows
    constexpr int NLD = QBLK_BYTES / (kImpWaves * 1024);   // DMA instructions per block per wave (2 or 1)
    constexpr int PER_ITEM = NLD + 1;            // DMA instructions per block per wave (Q rows + LSE)
    __shared__ __attribute__((aligned(1024))) uint8_t qs_lds[kImpBufs][QBLK_BYTES];
    __shared__ __attribute__((aligned(256))) float lse_lds[kImpBufs][kImpWaves][64];   // a private copy per wave

    int bid = blockIdx.x;
    const int g = bid % p.Hkv;  bid /= p.Hkv;
    constexpr int WKEYS = 32 * KG;               // keys per wave
    const int tid = threadIdx.x, lane = tid & 63;
    int b, row, tiles = p.n_ktiles;
    if (!p.scan) {
        b = sequence_of(bid, p.B, p.n_ktiles * p.n_split, p.turn, row);
    } else {
        // Sequences of different lengths: only slices that exist, those of the sequence with the most window rows, whose walks
        // are the longest, first.  (With a grid of the longest sequence's slices for each, the empty ones held places that the
        // others waited for, and a long walk could start last: 4 to 279 new tokens x 4 behind 1468 to 15431 keys, 32/8 heads, whole call
        // 109.5 -> 88.2 us, 3 to 363 x 8 behind 141 to 12509, 16/2 heads 95.1 -> 83.5.  A launch of few slices pays 0.5 us for it.)
        const int nq = lane < p.B ? min(p.cu_q[lane + 1], p.total_q) - min(p.cu_q[lane], p.total_q) : 0;
        const int nk = lane < p.B ? max(min(p.cu_k[lane + 1], p.total_k) - min(p.cu_k[lane], p.total_k), 0) : 0;
        const int walk = nq > 0 && nk >= nq ? min(nq, p.window < 0 ? nq : p.window) : 0;
        const int slices = (nk + WKEYS * kImpWaves - 1) / (WKEYS * kImpWaves), own = slices * p.n_split;
        int before = 0;
        for (int x = 0; x < p.B; ++x) {
            const int other = __builtin_amdgcn_readlane(walk, x);
            before += other > walk || (other == walk && x < lane) ? __builtin_amdgcn_readlane(own, x) : 0;
        }
        const uint64_t at = __ballot(bid >= before && bid < before + own);
        if (at == 0) return;
        b = (int)__builtin_ctzll(at);
        row = bid - __builtin_amdgcn_readlane(before, b);
        tiles = __builtin_amdgcn_readlane(slices, b);
    }
    const int kt = row % tiles;
    const int split = row / tiles;

    const int qs = min(p.cu_q[b], p.total_q), qe = min(p.cu_q[b + 1], p.total_q);
    const int ks = min(p.cu_k[b], p.total_k), ke = min(p.cu_k[b + 1], p.total_k);
    const int nq = qe - qs, nk = ke - ks;
    const int j_wg0 = kt * (WKEYS * kImpWaves);
    if (j_wg0 >= nk) return;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, hh = lane >> 5;
    const int delta = nk - nq;
    const int W = (p.window < 0 || p.window > nq) ? nq : p.window;
    const int iw0 = nq - W;                       // first window row
    const int jw0 = j_wg0 + WKEYS * wave;         // first key of this wave

    // K fragments (B operand) of the wave's KG 32-key groups: key j, dims 16 kk + 8 hh .. +7
    bf16x8 kf[KG][NKK];
    int jkey[KG];
#pragma unroll
    for (int kg = 0; kg < KG; ++kg) {
        jkey[kg] = jw0 + 32 * kg + n;
        const uint16_t *kp = p.k + (int64_t)(ks + min(jkey[kg], nk - 1)) * p.k_st + (int64_t)g * p.k_sh + 8 * hh;
#pragma unroll
        for (int kk = 0; kk < NKK; ++kk) kf[kg][kk] = *(const bf16x8 *)(kp + 16 * kk);
    }
    const float c2 = p.scale_log2;
    constexpr float kLog2e = 1.4426950408889634f;
    float colsum[KG] = {};

    if (nq > 0 && delta >= 0 && W > 0) {
        // rows: (token, head of the group) pairs of the window, token major, so that few tokens fill their blocks of 32
        // (blocks of one head's tokens cost G blocks for a chunk of 1 to 32 tokens: whole calls of 3 to 238 tokens x 3 to 8,
        // 64/8 heads, 81 -> 74, 96 -> 89, 67 -> 62 us; one chunk of 263 tokens 26.0 -> 26.6); blocks whose rows see none of this
        // workgroup's keys are skipped
        const int n_rows = W * p.G, n_rb = (n_rows + 31) / 32;
        auto row_of = [&](int j) { return min(max(0, j - delta - iw0), W) * p.G; };       // first row that sees key j
        const int rb_first = row_of(j_wg0) / 32;
        const int n_items_all = n_rb - rb_first;
        // this workgroup's share of the row blocks: items [item0, item0 + n_items)
        const int per_split = (n_items_all + p.n_split - 1) / p.n_split;
        const int item0 = min(split * per_split, n_items_all);
        const int n_items = min(per_split, n_items_all - item0);

        // Q rows of this sequence, all heads: buffer descriptor spanning the whole sequence
        const uint16_t *qbase = p.q + (int64_t)qs * p.q_st;
        const uint32_t q_row_bytes = (uint32_t)p.q_st * 2u;
        const uint32_t q_span = (uint32_t)(nq - 1) * q_row_bytes + (uint32_t)p.Hq * (uint32_t)p.q_sh * 2u;
        const i32x4 rsQ = make_rsrc(qbase, q_span);
        const i32x4 rsL = make_rsrc(p.lse, (uint32_t)p.Hq * (uint32_t)p.total_q * 4u);
        const uint32_t q_lds = lds_addr_of(&qs_lds[0][0]);
        const uint32_t l_lds = lds_addr_of(&lse_lds[0][wave][0]);
        // lane -> (row in block, chunk position); LDS chunk position holds chunk pos ^ swizzle(row)
        uint32_t qvoff[NLD];
        int qrow_l[NLD];
#pragma unroll
        for (int ci = 0; ci < NLD; ++ci) {
            const int flat = (wave + kImpWaves * ci) * 64 + lane;          // 16-byte slot in the block
            const int r = flat / CH, pos = flat % CH;
            const int c = D == 128 ? (pos ^ swz_row<128>(r)) : (pos ^ ((r >> 1) & 7));
            qrow_l[ci] = r;
            qvoff[ci] = (uint32_t)c * 16u;
        }
        // Blocks are requested and worked on in order, so a lane's rows are stepped along by 32: one division for the first
        // of them here, none per block.  Rows past the last one are the last one again.  (There are up to 2^30 rows, and
        // div_group is exact below 2^32 / G only: it takes the rows from the first token's on, 62 at most where G <= 31.)
        const int row0 = 32 * (rb_first + item0), tok0 = row0 / p.G, head0 = row0 - tok0 * p.G;
        auto token_of = [&](int r) { return tok0 + (p.G > 31 ? (head0 + r >= p.G ? 1 : 0) : div_group(head0 + r, p.g_magic)); };
        const int step_tok = div_group(32, p.g_magic), step_head = 32 - step_tok * p.G;
        const uint32_t q_head_bytes = (uint32_t)p.q_sh * 2u;
        const uint32_t q_step = (uint32_t)step_tok * q_row_bytes + (uint32_t)step_head * q_head_bytes, q_carry = q_row_bytes - (uint32_t)p.G * q_head_bytes;
        const uint32_t q_last = (uint32_t)(nq - 1) * q_row_bytes + (uint32_t)(g * p.G + p.G - 1) * q_head_bytes;
        const uint32_t l_head_bytes = (uint32_t)p.total_q * 4u;
        const uint32_t l_step = (uint32_t)step_tok * 4u + (uint32_t)step_head * l_head_bytes, l_carry = 4u - (uint32_t)p.G * l_head_bytes;
        const uint32_t l_last = (uint32_t)(g * p.G + p.G - 1) * l_head_bytes + (uint32_t)(qs + nq - 1) * 4u;
        uint32_t q_at[NLD], l_at;
        int q_head[NLD], l_head;
#pragma unroll
        for (int ci = 0; ci < NLD; ++ci) {
            const int tok = token_of(qrow_l[ci]);
            q_head[ci] = row0 + qrow_l[ci] - tok * p.G;
            q_at[ci] = (uint32_t)(iw0 + tok) * q_row_bytes + (uint32_t)(g * p.G + q_head[ci]) * q_head_bytes;
        }
        {
            const int tok = token_of(n);
            l_head = row0 + n - tok * p.G;
            l_at = (uint32_t)(g * p.G + l_head) * l_head_bytes + (uint32_t)(qs + iw0 + tok) * 4u;
        }
        int iss_left = n_rows - row0;                 // rows from the next request's first one on
        auto issue_item = [&](int buf) {              // the next block in order
#pragma unroll
            for (int ci = 0; ci < NLD; ++ci) {
                dma16_to_lds(rsQ, q_lds + buf * QBLK_BYTES + 1024 * (wave + kImpWaves * ci), (qrow_l[ci] < iss_left ? q_at[ci] : q_last) + qvoff[ci]);
                q_head[ci] += step_head;
                q_at[ci] += q_step;
                if (q_head[ci] >= p.G) { q_head[ci] -= p.G; q_at[ci] += q_carry; }
            }
            dma4_to_lds(rsL, l_lds + buf * (kImpWaves * 256), n < iss_left ? l_at : l_last);
            l_head += step_head;
            l_at += l_step;
            if (l_head >= p.G) { l_head -= p.G; l_at += l_carry; }
            iss_left -= 32;
        };
        int key_row[KG];
#pragma unroll
        for (int kg = 0; kg < KG; ++kg) key_row[kg] = row_of(jkey[kg]);
        const int first_row = row_of(jw0), whole_row = row_of(min(jw0 + WKEYS, nk) - 1);      // that sees the wave's first key, its last
        // A-operand read address of row n, chunk 2 kk + hh
        uint32_t qaddr[NKK];
#pragma unroll
        for (int kk = 0; kk < NKK; ++kk) {
            const int c = 2 * kk + hh;
            const int cs = D == 128 ? (c ^ swz_row<128>(n)) : (c ^ ((n >> 1) & 7));
            qaddr[kk] = (uint32_t)n * ROW_BYTES + (uint32_t)cs * 16u;
        }

        // The first row blocks are requested while the K fragment loads are still in flight; one
        // wait then ends both (the blocks were requested together and land together).  With the K
        // loads done here the compiler places no load waits inside the loop, where they would also
        // wait for the asynchronous row-block transfers in flight.
        for (int i = 0; i < kImpAhead && i < n_items; ++i) issue_item(i);
        __builtin_amdgcn_s_waitcnt(0);
        for (int item = 0; item < n_items; ++item) {
            const int buf = item & (kImpBufs - 1);
            // this block's loads are done once at most the blocks issued after it are outstanding
            const int newer = min(kImpAhead - 1, n_items - 1 - item);
            if (newer == 2) wait_vmcnt<2 * PER_ITEM>();
            else if (newer == 1) wait_vmcnt<PER_ITEM>();
            else wait_vmcnt<0>();
            __syncthreads();     // every wave's part of the block has landed; the buffer refilled below is free
            if (item + kImpAhead < n_items) issue_item((item + kImpAhead) & (kImpBufs - 1));
            const int r0 = row0 + 32 * item;
            if (r0 + 31 >= first_row && first_row < n_rows && jw0 < nk) {       // some row of the block sees some key of the wave
                const uint8_t *qb = &qs_lds[buf][0];
                f32x16 sc[KG];
                const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kk = 0; kk < NKK; ++kk) {
                    const bf16x8 a = *(const bf16x8 *)(qb + qaddr[kk]);
#pragma unroll
                    for (int kg = 0; kg < KG; ++kg)
                        sc[kg] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, kf[kg][kk], kk == 0 ? zero16 : sc[kg], 0, 0, 0);
                }
                // log2-domain LSE of rows 8 (e/4) + 4 hh + (e%4)
                f32x4 l2[4];
#pragma unroll
                for (int bq = 0; bq < 4; ++bq) l2[bq] = *(const f32x4 *)&lse_lds[buf][wave][8 * bq + 4 * hh] * kLog2e;
                // rows past the last one and keys beyond a row's reach contribute nothing
                const bool partial = r0 + 32 > n_rows || whole_row > r0;
                if (!partial) {
#pragma unroll
                    for (int e = 0; e < 16; ++e)
#pragma unroll
                        for (int kg = 0; kg < KG; ++kg)
                            colsum[kg] += fast_exp2(fmaf(sc[kg][e], c2, -l2[e >> 2][e & 3]));
                } else {
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        const int r = r0 + 8 * (e >> 2) + 4 * hh + (e & 3);
#pragma unroll
                        for (int kg = 0; kg < KG; ++kg) {
                            const float pe = fast_exp2(fmaf(sc[kg][e], c2, -l2[e >> 2][e & 3]));
                            colsum[kg] += r < n_rows && r >= key_row[kg] ? pe : 0.f;
                        }
                    }
                }
            }
        }
    }
#pragma unroll
    for (int kg = 0; kg < KG; ++kg) {
        const float tot = colsum[kg] + xchg_half(colsum[kg]);
        float *dst = p.n_split > 1 ? p.part + (int64_t)split * p.Hkv * p.total_k : p.imp;
        if (hh == 0 && jkey[kg] < nk) dst[(int64_t)g * p.total_k + ks + jkey[kg]] = tot;
    }
#else
    (void)p;
#endif
}

// The same sums with all window rows of the workgroup's (sequence, KV head) resident in LDS, for windows
// of few rows.  Rows are (token, head of the group) pairs, token major, so that a short window
// fills its 32-row blocks.  The rows and their log-sum-exp are loaded once, behind the one barrier of
// the kernel; then each wave walks `groups` groups of 32 keys by itself, K fragments of the next
// group requested while one is summed.  (The kernel above waits at a barrier for every block of 32 rows
// with some 0.3 us of work between barriers.)  Bound by the exponentials on long launches (32768
// tokens x 32/8 heads, 128 rows: 50 us streamed, 41), by the first loads on short ones (4096 tokens, 64 rows: 9.1 streamed,
// 7.2) and by K from memory between them (64 tokens x 4 behind 8192 keys: 17 us with one block of rows, 26 with
// eight).  What a wave does besides its 16 exponentials per block and lane was as much again and is kept short: LDS addresses from one
// register, rows of Q stepped along instead of divided out, two register sets for K instead of copies, blocks that need no
// mask in a loop of their own; and the barrier waits for the rows, not for K.  Together 46 -> 42 us at the first of these
// sizes, 29.7 -> 26.0 at the last, 8 prompts of 512 to 7900 tokens, 64 rows 28.4 -> 24.6 (traced, other inputs each call).
constexpr int kImpScanMax = 64;         // sequences whose lengths one wave scans
constexpr uint32_t kImpLoadSteps = 8;   // blocks of rows that a wave works on while 32 keys come from memory
constexpr int kImpLse = 3;              // rows per thread at most: 608 (19 blocks of head_dim 64 in 80 KB) for four waves, 1216 (38 in 160 KB) for 16
template <int D>
constexpr int importance_rows_block_bytes() { return 32 * 2 * D + 32 * (int)sizeof(float); }

template <int D>
__global__ __launch_bounds__(1024) void importance_rows_kernel(const ImpParams p)
{
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int NKK = D / 16, ROW_BYTES = D * 2, CH = D / 8, QBLK_BYTES = 32 * ROW_BYTES;
    constexpr int RPI = 1024 / ROW_BYTES;        // rows per DMA instruction
    extern __shared__ __attribute__((aligned(1024))) uint8_t imp_smem[];     // blocks of rows, then their log-sum-exp

    int bid = blockIdx.x;
    const int g = bid % p.Hkv;  bid /= p.Hkv;
    const int tid = threadIdx.x, lane = tid & 63, waves = blockDim.x >> 6;
    int b, kt, groups = p.groups;
    if (!p.scan) {                                // the last pieces, which may be short, come last
        b = bid % p.B;
        kt = bid / p.B;
    } else if (p.places > 0) {
        // Chunks of different lengths: a group of keys costs a wave kImpLoadSteps steps and one per block of the sequence's
        // rows, so a sequence's waves get groups for about `steps` steps, the same for all sequences and few enough groups
        // that all pieces are on the chip at once.  `steps` grows until they are, at the latest where each sequence is one
        // piece (p.B <= p.places).  Whole calls against one or two
        // groups for every sequence: 3 to 300 tokens x 6 behind 106 to 10913, 8/8 heads of head_dim 64 49.9 -> 44.8 us, 6 to 87 x 7
        // behind 214 to 15157, 32/8 heads 87.3 -> 80.8; 31 uneven launches 1.4 % faster in the mean, one of them 2 % slower.
        uint32_t keys32 = 0, cost = kImpLoadSteps + 1;
        if (lane < p.B) {
            const int nq = min(p.cu_q[lane + 1], p.total_q) - min(p.cu_q[lane], p.total_q);
            const int nk = max(min(p.cu_k[lane + 1], p.total_k) - min(p.cu_k[lane], p.total_k), 0);
            keys32 = (uint32_t)(nk + 31) / 32;
            if (nq > 0 && nk >= nq) cost = kImpLoadSteps + (uint32_t)(min(nq, p.window < 0 ? nq : p.window) * p.G + 31) / 32;
        }
        const uint32_t all = (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan(keys32 * cost), 63);
        uint32_t steps = max(all / (uint32_t)(p.places * waves), 1u), own, upto;
        for (;;) {
            const uint32_t keys = (uint32_t)waves * max((steps + cost / 2) / cost, 1u);
            own = (keys32 + keys - 1) / keys;
            upto = wave_incl_scan(own);
            if ((uint32_t)__builtin_amdgcn_readlane((int)upto, 63) <= (uint32_t)p.places || steps >= 1u << 27) break;
            steps += steps / 8 + 1;
        }
        const uint64_t after = __ballot(upto > (uint32_t)bid);
        if (after == 0) return;
        b = (int)__builtin_ctzll(after);
        kt = bid - __builtin_amdgcn_readlane((int)(upto - own), b);
        // the sequence's groups evenly over its pieces' waves
        const int pieces = __builtin_amdgcn_readlane((int)own, b) * waves;
        groups = (__builtin_amdgcn_readlane((int)keys32, b) + pieces - 1) / pieces;
    } else {
        // Sequences of different lengths: workgroup number `bid` takes the bid-th piece that has keys.  (With a
        // grid of the longest sequence's pieces for each, the ones without keys settle which shader engine the others
        // go to, because workgroups are dealt out round robin: 8 prompts of 512 to 7900 tokens, 128 rows, kept one in
        // four of the compute units for half of the work, 66 us; 37 like this.)
        const int n = lane < p.B ? max(min(p.cu_k[lane + 1], p.total_k) - min(p.cu_k[lane], p.total_k), 0) : 0;
        const int keys_log2 = 36 - __builtin_clz(waves * p.groups);          // 32 * waves * groups, a power of two
        const uint32_t own = (uint32_t)(n + (1 << keys_log2) - 1) >> keys_log2, upto = wave_incl_scan(own);
        const uint64_t after = __ballot(upto > (uint32_t)bid);
        if (after == 0) return;
        b = (int)__builtin_ctzll(after);
        kt = bid - __builtin_amdgcn_readlane((int)(upto - own), b);
    }
    const int qs = min(p.cu_q[b], p.total_q), qe = min(p.cu_q[b + 1], p.total_q);
    const int ks = min(p.cu_k[b], p.total_k), ke = min(p.cu_k[b + 1], p.total_k);
    const int nq = qe - qs, nk = ke - ks, delta = nk - nq;
    const int j_wg0 = kt * waves * groups * 32;
    if (j_wg0 >= nk) return;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, hh = lane >> 5;
    const int W = (nq > 0 && delta >= 0) ? ((p.window < 0 || p.window > nq) ? nq : p.window) : 0;
    const int iw0 = nq - W;                       // first window token
    const int n_rows = W * p.G, n_blocks = (n_rows + 31) / 32;
    // first row that sees key j
    auto row_of = [&](int j) { return min(max(0, j - delta - iw0), W) * p.G; };

    const uint16_t *const kbase = p.k + (int64_t)ks * p.k_st + (int64_t)g * p.k_sh + 8 * hh;
    auto load_k = [&](bf16x8 (&kf)[NKK], int j0) {
        const uint16_t *kp = kbase + (int64_t)min(j0 + n, nk - 1) * p.k_st;
#pragma unroll
        for (int kk = 0; kk < NKK; ++kk) kf[kk] = *(const bf16x8 *)(kp + 16 * kk);
    };
    const int j_first = j_wg0 + 32 * wave;
    const int block0 = row_of(j_wg0) / 32;        // blocks before it see none of the workgroup's keys
    float *const lse_sh = (float *)(imp_smem + n_blocks * QBLK_BYTES);
    // The rows of Q, their log-sum-exp and the first keys are requested in this order and return in it, so that the
    // barrier waits for the first two only.
    bf16x8 kf[2][NKK];
    if (n_rows > 0) {
        const uint16_t *qbase = p.q + (int64_t)(qs + iw0) * p.q_st + (int64_t)(g * p.G) * p.q_sh;
        const uint32_t q_row_bytes = (uint32_t)p.q_st * 2u, q_head_bytes = (uint32_t)p.q_sh * 2u;
        const uint32_t last = (uint32_t)(W - 1) * q_row_bytes + (uint32_t)(p.G - 1) * q_head_bytes;
        const i32x4 rs = make_rsrc(qbase, last + (uint32_t)ROW_BYTES);
        const uint32_t lds = lds_addr_of(imp_smem);
        // a transfer brings RPI rows, the wave's next one those `step` rows on (a multiple of 16, so the chunk of a lane,
        // which follows from its row modulo 16, stays)
        const int i0 = block0 * (32 / RPI) + wave, step = RPI * waves, step_tok = div_group(step, p.g_magic), step_head = step - step_tok * p.G;
        int r = RPI * i0 + lane / CH, head;
        const uint32_t chunk = (uint32_t)((lane % CH) ^ (D == 128 ? swz_row<128>(r & 31) : ((r >> 1) & 7))) * 16u;
        uint32_t at;
        {
            const int tok = div_group(r, p.g_magic);
            head = r - tok * p.G;
            at = (uint32_t)tok * q_row_bytes + (uint32_t)head * q_head_bytes + chunk;
        }
        const uint32_t step_bytes = (uint32_t)step_tok * q_row_bytes + (uint32_t)step_head * q_head_bytes, carry = q_row_bytes - (uint32_t)p.G * q_head_bytes;
        for (int i = i0; i < n_blocks * (32 / RPI); i += waves) {
            dma16_to_lds(rs, lds + 1024 * i, r < n_rows ? at : last + chunk);
            r += step;
            head += step_head;
            at += step_bytes;
            if (head >= p.G) {
                head -= p.G;
                at += carry;
            }
        }
        auto request = [&](auto loads_c) __attribute__((always_inline)) {
            constexpr int LOADS = decltype(loads_c)::value;          // rows per thread
            float l2[LOADS];
#pragma unroll
            for (int i = 0; i < LOADS; ++i) {
                const int row = min(32 * block0 + tid + i * (int)blockDim.x, n_rows - 1), tok = div_group(row, p.g_magic);
                l2[i] = p.lse[(int64_t)(g * p.G + row - tok * p.G) * p.total_q + qs + iw0 + tok];
            }
            asm volatile("" ::: "memory");            // the compiler keeps the order
            load_k(kf[0], j_first);
#pragma unroll
            for (int i = 0; i < LOADS; ++i) {
                const int x = 32 * block0 + tid + i * (int)blockDim.x;
                if (x < 32 * n_blocks) lse_sh[x] = x < n_rows ? l2[i] * -1.4426950408889634f : -INFINITY;      // rows past the last one add nothing
            }
        };
        if (n_rows - 32 * block0 <= (int)blockDim.x) request(std::integral_constant<int, 1>{});
        else request(std::integral_constant<int, kImpLse>{});
        wait_vmcnt<NKK>();
    }
    __syncthreads();

    // LDS addresses: row n, chunk hh of block 0 (chunk 2 kk + hh: with 32 kk exclusive-or'ed in), and the log-sum-exp of its rows 4 hh ..
    typedef const __attribute__((address_space(3))) bf16x8 *LdsRow;
    typedef const __attribute__((address_space(3))) f32x4 *LdsLse;
    const uint32_t qaddr = lds_addr_of(imp_smem) + (uint32_t)n * ROW_BYTES + (uint32_t)(hh ^ (D == 128 ? swz_row<128>(n) : (n >> 1) & 7)) * 16u;
    const uint32_t laddr = lds_addr_of(lse_sh) + 16u * hh;
    const float c2 = p.scale_log2;
    // (waited for in one place, or the compiler, which cannot tell whether kn was requested, waits for it at the first use of kc)
    auto wait_keys = [] { __builtin_amdgcn_s_waitcnt(0x0f70); };                // vmcnt(0)
    // keys j0 .. j0 + 31, whose K fragments are in kc, against their blocks; the next group's fragments go to kn
    auto group = [&](const bf16x8 (&kc)[NKK], bf16x8 (&kn)[NKK], int t) __attribute__((always_inline)) {
        const int j0 = j_first + 32 * waves * t;
        if (t + 1 < groups) load_k(kn, j0 + 32 * waves);
        const int key_row = row_of(j0 + n);
        int rb = row_of(j0) / 32;
        const int masked = min((row_of(j0 + 31) + 31) / 32, n_blocks);          // from this block on every row sees every key
        float colsum = 0.f;
        uint32_t qa = qaddr + (uint32_t)rb * QBLK_BYTES, la = laddr + 128u * rb;
        auto block = [&](auto at_c, auto masked_c) __attribute__((always_inline)) {
            constexpr uint32_t AT = decltype(at_c)::value;
            f32x16 sc;
            const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kk = 0; kk < NKK; ++kk)
                sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(LdsRow)((qa ^ 32u * kk) + AT * QBLK_BYTES), kc[kk], kk == 0 ? zero16 : sc, 0, 0, 0);
            f32x4 nl[4];                          // rows 8 (e / 4) + 4 hh + e % 4
#pragma unroll
            for (int bq = 0; bq < 4; ++bq) nl[bq] = *(LdsLse)(la + AT * 128 + 32 * bq);
            __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);           // three reads ahead of the products: registers allow no more
#pragma unroll
            for (int kk = 0; kk < NKK; ++kk) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const float pe = fast_exp2(fmaf(sc[e], c2, nl[e >> 2][e & 3]));
                if constexpr (decltype(masked_c)::value) colsum += 32 * rb + 8 * (e >> 2) + 4 * hh + (e & 3) >= key_row ? pe : 0.f;
                else colsum += pe;
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        auto advance = [&](int by) {
            rb += by;
            la += 128u * by;
            qa += (uint32_t)by * QBLK_BYTES;
        };
        constexpr std::integral_constant<uint32_t, 0> first{};
        constexpr std::integral_constant<uint32_t, 1> second{};
        for (; rb < masked; advance(1)) block(first, std::true_type{});
        for (; rb + 2 <= n_blocks; advance(2)) {
            block(first, std::false_type{});
            block(second, std::false_type{});
        }
        if (rb < n_blocks) block(first, std::false_type{});
        const float tot = colsum + xchg_half(colsum);
        wait_keys();
        if (hh == 0 && j0 + n < nk) p.imp[(int64_t)g * p.total_k + ks + j0 + n] = tot;
    };
    wait_keys();
    const int todo = min(groups, (max(nk - j_first, 0) + 32 * waves - 1) / (32 * waves));      // groups with keys
    for (int t = 0; t < todo; t += 2) {
        group(kf[0], kf[1], t);
        if (t + 1 < todo) group(kf[1], kf[0], t + 1);
    }
#else
    (void)p;
#endif
}

// imp[x] = part[0][x] + part[1][x] + ... in that order, x over Hkv * total_k elements
__global__ __launch_bounds__(256) void importance_reduce_kernel(const float *part, float *imp, int64_t n, int n_split)
{
    const int64_t x = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (x >= n) return;
    float acc = part[x];
    for (int r = 1; r < n_split; ++r) acc += part[(int64_t)r * n + x];
    imp[x] = acc;
}

}  // namespace pdd
