// Top-k selection with the candidates of a row divided over workgroups (paper Section 3.2, "Prompt
// Refiner"; the same outputs as select_topk.hpp, byte for byte), for rows that one workgroup is
// too little for.
//
// One workgroup of 1024 threads per (row, chunk of 4096 candidates); four launches with a caller
// workspace between them, and no workgroup that waits for another one.  A radix search over the
// 32-bit keys, 11 + 11 + 10 bits from the top:
//   select_level_kernel<0>     histogram of the chunk's keys over their first digit, and its sums
//                              over groups of 32 bins;
//   select_level_kernel<1, 2>  every workgroup sums the chunks' group sums and then the one group
//                              that holds the kk-th largest key (96 of 2048 bins are read), which
//                              gives the digit of the threshold and how many keys of the chunks before
//                              lie above it; histogram of the next digit over the chunk's keys
//                              that share the digits found so far;
//   select_finish_kernel       the last digit, and with it the threshold and the number of kept keys in
//                              the chunks before; the chunk's indices and mask.
// The counts are integers, so every workgroup of a row finds the same digits, and the work does not depend
// on the scores (a list of the keys that share the first 13 bits, searched directly, took one
// launch and 1 us less where they are few, and up to 2 ms where most scores agree to 1 %).
// Bound by the latency of its steps (loads, scans, barriers, launches) up to some 10 rows, by
// instruction issue beyond.  8 rows of 131072 candidates, k = 10 %: 225 -> 21 us, 24 rows 226 -> 39.
#pragma once
#include "select_topk.hpp"

namespace pdd {

constexpr int kSplitSelChunk = 4 * kSelThreads;       // candidates per workgroup, four per thread
constexpr int kSplitSelBins = 2 * kSelThreads;        // 11 bits
constexpr int kSplitSelGroups = 64, kSplitSelFine = kSplitSelBins / kSplitSelGroups;

// What a workgroup knows of its row before a digit is looked for: the digits found so far, the rank
// of the threshold among the keys that share them, the keys above them in the chunks before its own.
struct SplitSelState { uint32_t prefix, rank, before, unused; };

// Workspace: histograms of two levels, because a level is still read while the next one is written
// (16 bits a bin: a chunk has 4096 keys), their group sums, the workgroups' states.
struct SplitSelParams {
    SelParams s;
    int32_t n_chunks;          // of the longest sequence
    uint32_t *hist[2];         // [rows][n_chunks][1024] two bins per word
    uint32_t *group[2];        // [rows][n_chunks][64]
    SplitSelState *state;      // [rows][n_chunks]
};
constexpr size_t kSplitSelChunkBytes = 2 * (kSplitSelBins / 2 + kSplitSelGroups) * sizeof(uint32_t) + sizeof(SplitSelState);

typedef float sel_f32x4 __attribute__((ext_vector_type(4), aligned(4)));        // four scores at any score's address
typedef uint32_t sel_u32_any __attribute__((aligned(1)));                       // four mask bytes at any address

struct SelRow {
    const float *cand;         // the row's candidates
    int nk, c0, n, chunks, kk, slots, keep0;
    int64_t row, at;           // row = head * B + sequence; first mask element of the sequence
};

__device__ __forceinline__ SelRow split_sel_row(const SelParams &p)
{
    SelRow r;
    const int b = blockIdx.y, g = blockIdx.z;
    const int ks = min(max(p.cu_k[b], 0), p.total_k);
    const int ke = min(max(p.cu_k[b + 1], ks), p.total_k);
    r.nk = ke - ks;
    const int c0 = min(max(p.cand_b ? p.cand_b[b] : 0, 0), r.nk);
    const int c1 = min(max(p.cand_e ? p.cand_e[b] : r.nk, c0), r.nk);
    r.c0 = c0;
    r.n = min(c1 - c0, (int)gridDim.x * kSplitSelChunk);         // what the workspace has room for
    r.chunks = (r.n + kSplitSelChunk - 1) / kSplitSelChunk;
    r.keep0 = min(max(p.cu_keep[b], 0), p.total_keep);
    const int keep1 = min(max(p.cu_keep[b + 1], r.keep0), p.total_keep);
    r.slots = keep1 - r.keep0;
    r.kk = min(min(max(p.k_per[b], 0), r.n), r.slots);
    r.row = (int64_t)g * p.B + b;
    r.at = (int64_t)g * p.total_k + ks;
    r.cand = p.scores + r.at + c0;
    return r;
}

// keys of the thread's four candidates, 0 (below every key) past the row's end
__device__ __forceinline__ void split_sel_keys(const SelRow &r, int x0, uint32_t (&key)[4])
{
    if (x0 + 4 <= r.n) {
        const sel_f32x4 t = *(const sel_f32x4 *)(r.cand + x0);
#pragma unroll
        for (int j = 0; j < 4; ++j) key[j] = order_key(t[j]);
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) key[j] = x0 + j < r.n ? order_key(r.cand[x0 + j]) : 0u;
    }
}

// The next digit of the threshold, from the histograms of the row's chunks: `st` moves on by one
// digit; the return value is the number of keys in the digit's bin in the chunks before this one.
// Two barriers; the same in every thread.
__device__ __forceinline__ uint32_t split_sel_digit(const uint32_t *hist, const uint32_t *group, int chunks, int chunk,
                                                    int bits, int lane, int wave, SplitSelState &st)
{
    __shared__ uint32_t grp_all[kSelWaves][kSplitSelGroups], grp_pre[kSelWaves][kSplitSelGroups];
    __shared__ uint32_t bin_all[kSelWaves][64], bin_pre[kSelWaves][64];
    // ---- the group (lane = group): sums over all chunks, and over those before this one
    uint32_t all = 0, pre = 0;
#pragma unroll 4
    for (int c = wave; c < chunks; c += kSelWaves) {
        const uint32_t x = group[c * kSplitSelGroups + lane];
        all += x;
        pre += c < chunk ? x : 0u;
    }
    grp_all[wave][lane] = all;
    grp_pre[wave][lane] = pre;
    __syncthreads();
    all = pre = 0;
#pragma unroll
    for (int w = 0; w < kSelWaves; ++w) { all += grp_all[w][lane]; pre += grp_pre[w][lane]; }
    uint32_t sc[2] = {all, pre};
    wave_incl_scan_n(sc);
    // a group holds the key of this rank iff above < rank <= above + its own
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)sc[0], 63);
    const uint32_t total_pre = (uint32_t)__builtin_amdgcn_readlane((int)sc[1], 63);
    uint32_t above = total - sc[0];
    const int g = __builtin_amdgcn_readfirstlane(__ffsll((unsigned long long)__ballot(above < st.rank && st.rank <= above + all)) - 1);
    above = (uint32_t)__builtin_amdgcn_readlane((int)above, g);
    uint32_t before = total_pre - (uint32_t)__builtin_amdgcn_readlane((int)sc[1], g);

    // ---- the bin inside the group (lane & 31 = bin, a half wave per chunk)
    const uint16_t *h16 = (const uint16_t *)hist + g * kSplitSelFine + (lane & 31);
    all = pre = 0;
#pragma unroll 2
    for (int c = 2 * wave + (lane >> 5); c < chunks; c += 2 * kSelWaves) {
        const uint32_t x = h16[c * kSplitSelBins];
        all += x;
        pre += c < chunk ? x : 0u;
    }
    bin_all[wave][lane] = all;
    bin_pre[wave][lane] = pre;
    __syncthreads();
    all = pre = 0;
#pragma unroll
    for (int w = 0; w < kSelWaves; ++w) {
        all += bin_all[w][lane & 31] + bin_all[w][32 + (lane & 31)];
        pre += bin_pre[w][lane & 31] + bin_pre[w][32 + (lane & 31)];
    }
    if (lane >= 32) all = pre = 0;
    sc[0] = all;
    sc[1] = pre;
    wave_incl_scan_n(sc);
    const uint32_t above_bin = above + (uint32_t)__builtin_amdgcn_readlane((int)sc[0], 63) - sc[0];
    const int f = __builtin_amdgcn_readfirstlane(__ffsll((unsigned long long)__ballot(above_bin < st.rank && st.rank <= above_bin + all)) - 1);
    before += (uint32_t)__builtin_amdgcn_readlane((int)sc[1], 63) - (uint32_t)__builtin_amdgcn_readlane((int)sc[1], f);
    st.prefix = st.prefix << bits | (uint32_t)(g * kSplitSelFine + f);
    st.rank -= (uint32_t)__builtin_amdgcn_readlane((int)above_bin, f);
    st.before += before;
    return (uint32_t)__builtin_amdgcn_readlane((int)pre, f);
}

template <int LEVEL>
__global__ __launch_bounds__(kSelThreads) void select_level_kernel(const SplitSelParams p)
{
    __shared__ __attribute__((aligned(16))) uint32_t hist[kSplitSelBins];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int chunk = blockIdx.x;
    const SelRow r = split_sel_row(p.s);
    if (chunk >= r.chunks || r.kk == 0) return;
    const int x0 = chunk * kSplitSelChunk + 4 * tid;
    uint32_t key[4];
    split_sel_keys(r, x0, key);
    ((uint2 *)hist)[tid] = make_uint2(0u, 0u);
    const int64_t row0 = r.row * p.n_chunks;
    SplitSelState st = {0u, (uint32_t)r.kk, 0u, 0u};
    if constexpr (LEVEL == 0) {
        __syncthreads();
    } else {
        if constexpr (LEVEL > 1) st = p.state[row0 + chunk];
        split_sel_digit(p.hist[(LEVEL - 1) & 1] + row0 * (kSplitSelBins / 2), p.group[(LEVEL - 1) & 1] + row0 * kSplitSelGroups,
                        r.chunks, chunk, 11, lane, wave, st);
    }
    uint32_t bin[4];
    bool part[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        bin[j] = LEVEL == 0 ? key[j] >> 21 : LEVEL == 1 ? key[j] >> 10 & 2047u : key[j] & 1023u;
        part[j] = x0 + j < r.n && (LEVEL == 0 || key[j] >> (LEVEL == 1 ? 21 : 10) == st.prefix);
    }
    // Atomics on one address go one after another.  Where the wave's first keys all share a bin, the lanes that have
    // the common bin add as one (equal scores: 320 rows of 33000 207 -> 115 us, 8 of 131072 32 -> 24).
    const uint32_t common = (uint32_t)__builtin_amdgcn_readfirstlane((int)bin[0]);
    if (__ballot(part[0] && bin[0] == common) == ~0ull) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool same = part[j] && bin[j] == common;
            const uint32_t n = (uint32_t)__popcll(__ballot(same));
            if (lane == 0) atomicAdd(&hist[common], n);
            if (part[j] && !same) atomicAdd(&hist[bin[j]], 1u);
        }
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (part[j]) atomicAdd(&hist[bin[j]], 1u);
    }
    __syncthreads();
    const uint2 h = ((const uint2 *)hist)[tid];
    p.hist[LEVEL & 1][(row0 + chunk) * (kSplitSelBins / 2) + tid] = h.x | h.y << 16;
    // the 16 lanes of a DPP row hold a group's 32 bins
    uint32_t s = h.x + h.y;
    s += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)s, 0x111, 0xf, 0xf, true);
    s += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)s, 0x112, 0xf, 0xf, true);
    s += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)s, 0x114, 0xf, 0xf, true);
    s += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)s, 0x118, 0xf, 0xf, true);
    if ((lane & 15) == 15) p.group[LEVEL & 1][(row0 + chunk) * kSplitSelGroups + (tid >> 4)] = s;
    if (LEVEL > 0 && tid == 0) p.state[row0 + chunk] = st;
}

__global__ __launch_bounds__(kSelThreads) void select_finish_kernel(const SplitSelParams p)
{
    __shared__ uint32_t wave_own[kSelWaves];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int chunk = blockIdx.x;
    const SelRow r = split_sel_row(p.s);
    int32_t *out = p.s.out_idx + (int64_t)blockIdx.z * p.s.total_keep + r.keep0;
    uint8_t *mrow = p.s.out_mask ? p.s.out_mask + r.at : nullptr;

    // what lies outside the candidates, shared by the row's workgroups
    const int t0 = chunk * kSelThreads + tid, t_step = p.n_chunks * kSelThreads;
    if (p.s.pooled_out)
        for (int x = t0; x < r.nk; x += t_step) p.s.pooled_out[r.at + x] = p.s.scores[r.at + x];
    const bool none = r.kk == 0;                                 // the same in every thread
    if (mrow) {
        const int z = none ? r.nk : r.c0;
        for (int x = t0; x < z; x += t_step) mrow[x] = 0;
        for (int x = max(r.c0 + r.n, z) + t0; x < r.nk; x += t_step) mrow[x] = 0;
    }
    for (int x = r.kk + t0; x < r.slots; x += t_step) out[x] = -1;
    if (none || chunk >= r.chunks) return;

    const int x0 = chunk * kSplitSelChunk + 4 * tid;
    uint32_t key[4];
    split_sel_keys(r, x0, key);
    const int64_t row0 = r.row * p.n_chunks;
    SplitSelState st = p.state[row0 + chunk];
    int eq_before = (int)split_sel_digit(p.hist[0] + row0 * (kSplitSelBins / 2), p.group[0] + row0 * kSplitSelGroups, r.chunks,
                                         chunk, 10, lane, wave, st);
    const uint32_t T = st.prefix;
    const int krem = (int)st.rank;                               // ties at T to keep (>= 1), lowest index first
    int gt_before = (int)st.before;

    // ---- the chunk's own keys > T | == T << 16, in index order
    uint32_t own = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {                                // empty slots hold key 0, below every finite score
        own += key[j] > T ? 1u : 0u;
        own += key[j] == T ? 0x10000u : 0u;
    }
    const uint32_t incl = wave_incl_scan(own);
    if (lane == 63) wave_own[wave] = incl;
    __syncthreads();
    uint32_t before = incl - own;
#pragma unroll
    for (int w = 0; w < kSelWaves; ++w) before += w < wave ? wave_own[w] : 0u;
    gt_before += (int)(before & 0xffffu);
    eq_before += (int)(before >> 16);

    // ---- stable compaction
    uint32_t mbytes = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const bool is_gt = key[j] > T, is_eq = key[j] == T;
        const bool sel = is_gt || (is_eq && eq_before < krem);
        if (sel) out[gt_before + min(eq_before, krem)] = r.c0 + x0 + j;
        gt_before += is_gt ? 1 : 0;
        eq_before += is_eq ? 1 : 0;
        mbytes |= sel ? (1u << (8 * j)) : 0u;
    }
    if (mrow && x0 < r.n) {
        uint8_t *mp = mrow + r.c0 + x0;
        if (x0 + 4 <= r.n) *(sel_u32_any *)mp = mbytes;
        else
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (x0 + j < r.n) mp[j] = (uint8_t)(mbytes >> (8 * j));
    }
}

}  // namespace pdd
