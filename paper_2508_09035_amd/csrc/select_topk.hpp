// Top-k token selection and stable index compaction (paper Section 3.2,
// "Prompt Refiner": the indices with the top summed scores are kept at ratio
// r and the positions are filtered; the mask tensor has 1 at position i when
// token i is selected).
//
// One workgroup of 1024 threads per (sequence, head) row; scores become
// order-preserving uint32 keys.  Two kernels:
//
//  * select_topk_reg_kernel<QPT> (rows of up to 4096 * QPT <= 32768 candidates):
//    every thread keeps its 4 QPT keys in registers for the whole kernel.  A histogram (of a
//    sample, where the row is long) places a bracket around the k-th largest key; one pass over the
//    keys counts those inside and above it and one moves those inside to LDS, where a few rounds of two probes
//    on the key value find it (one round = two compares per key, one LDS counter).  Passes are
//    few because each costs by its instructions, 16 cycles each with four waves per SIMD.  The row is
//    not read again.  The kept indices are written in ascending order from
//    prefix counts, with a 16 * QPT-entry scan across waves.
//    By single interpolated or bisecting probes from the row's range on (8 to 11, 27 with many
//    ties) 8 rows took, scores spread over octaves / log-normal: 4096 9.5 / 10.5 us, 16384 13.6 / 16.2,
//    32768 20.0 / 21.3, 512 rows of 32768 42.1 / 47.4; with all keys' range, two probes a round over all keys and loads behind
//    branches 6.5 / 6.3, 11.6 / 11.6, 17.0 / 17.2, 36.7 / 37.0.  With the sample's own range, requested ahead of the row and
//    placed while that is on its way (uniform scores to the sixth power, kept 1/10 to 1/2, before -> now): 8 rows of 4096 6.5 -> 5.8 us, 16384
//    12.3 -> 11.2, 32768 16.7 -> 14.1, 512 rows of 32768 34.3 -> 29.8, 512 of 4000 9.6 -> 8.6.  Rows of few
//    different scores, which the sample misjudges, take 0.8 to 1.3 times as long (8 of 32768, k = 1/10 / half: one value 9.4 / 11.2 -> 10.2 / 12.0,
//    two 12.6 / 13.8 -> 11.9 / 15.5, seven 12.7 / 19.1 -> 12.7 / 14.9, nine zeros in ten 18.3 / 14.9 -> 20.2 / 14.3).
//    Bound by the latency of some ten steps where the rows are few; 512 rows read 67 MB and write 23 (18.5 us) before and after the
//    passes, with all rows at the same point at once.
//    Histograms of all keys of long rows were slower: 50 cycles per LDS atomic of a wave.  So
//    were fewer threads with more keys each (256 x 16: 9.7 us at 4096).
//  * select_topk_kernel (longer rows without a workspace, pooled, or beyond the limits of
//    select_split.hpp, which has the others): most-significant-first radix select,
//    8 bits per pass, digits taken from (key - min key) scaled to the row's
//    range, LDS histograms; the row is re-read from L2 in every pass.
//
// Ties at the threshold are resolved towards the lower index in both.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "wave_scan.hpp"

namespace pdd {

enum { kPoolNone = 0, kPoolMax = 1, kPoolAvg = 2 };

struct SelParams {
    const float *scores;
    const int32_t *cu_k, *cand_b, *cand_e, *k_per, *cu_keep;
    int32_t *out_idx;
    uint8_t *out_mask;
    int32_t n_heads, B, total_k, total_keep;
    int32_t pool_r, pool_mode;   // 1-D pooling radius (kernel = 2r+1) and kPool* mode; r = 0: none
    float pool_inv;              // 1 / kernel for the average
    float *pooled_out;           // optional [n_heads, total_k]: the pooled scores that were ranked
};

constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / 64;
constexpr int kSelFinish = 128;   // keys left in the bracket that are ranked directly
constexpr uint32_t kSelRun = 64;  // keys of the sample in one bin that may be a run of equal scores
constexpr int kSelList = 4 * kSelThreads;     // keys left in the bracket that move to four per thread
constexpr int kSelBins = 1024;    // of the histograms that place the bracket, one bin per thread
constexpr int kSelRegCap = 32 * 1024;  // rows up to this many candidates stay in registers

// Score of key j after 1-D pooling along the sequence (paper Section 3.2: a pooling step
// between the sum over queries and the sort, so that neighbours are kept together).  Window = keys
// [j-r, j+r] inside the sequence; max over the valid part, or sum of the valid part divided by
// the kernel size (zero padding).  seq = first score of the sequence row, nk = its length.
__device__ __forceinline__ float pooled_score(const float *seq, int nk, int j, int r, int mode, float inv)
{
    if (r == 0) return seq[j];
    const int lo = max(j - r, 0), hi = min(j + r, nk - 1);
    float acc = seq[lo];
    if (mode == kPoolMax) {
        for (int t = lo + 1; t <= hi; ++t) acc = fmaxf(acc, seq[t]);
        return acc;
    }
    for (int t = lo + 1; t <= hi; ++t) acc += seq[t];
    return acc * inv;
}

__device__ __forceinline__ uint32_t order_key(float x)
{
    // monotone map fp32 -> uint32 (larger float <=> larger key); -0.0 == +0.0.  Never 0, which stands
    // for a slot without a candidate: the NaN of all ones would be, and would miss in every count
    const uint32_t u = __float_as_uint(x + 0.0f);
    return max(u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u), 1u);    // negative: all bits flipped; else the sign bit set
}


// ---------------------------------------------------------------------------
// Register-resident selection for rows of at most 4096 * QPT candidates, four consecutive
// candidates per lane and step.  Thread `tid` owns the quads q = i * 1024 + tid, i < QPT, of the
// row's part that starts at a 16-byte boundary of the score tensor (the up to three candidates
// before it sit one each in the first lanes of wave 0): 16-byte loads, the mask written four
// bytes at a time where the mask tensor's alignment allows it.
// POOL = true ranks the 1-D pooled scores (see PoolStage);
// the instantiation for unpooled scores carries none of the pooling code.
// ---------------------------------------------------------------------------
constexpr int kSelMaxProbes = 72;       // a 32-bit bracket needs at most 2 x 21 rounds by thirds, 8 that cut the keys to a quarter

// Next value to probe in the threshold search over the bracket [lo, hi] (lo < hi) that holds
// `inside` keys, of which the `need` largest (1 <= need <= inside) lie at or above the threshold.
// With interpolate set, the keys are taken as evenly spread over the bracket, which is nearly true
// once the bracket is a narrow slice of the score distribution, and the probe lands a few keys
// away from the threshold instead of halving the bracket; otherwise the bracket is bisected.  The
// callers interpolate as long as the previous probe cut the number of keys in the bracket to a
// quarter or less and bisect after one that did not, which bounds the worst case at twice the
// probes of plain bisection.  The result is in [lo + 1, hi]: either outcome shrinks the bracket.
__device__ __forceinline__ uint32_t next_probe(uint32_t lo, uint32_t hi, uint32_t inside, uint32_t need, bool interpolate)
{
    const uint32_t span = hi - lo;
    if (!interpolate) return lo + ((span + 1u) >> 1);
    const float f = ((float)need - 0.5f) / (float)inside;          // share of the bracket above the threshold
    const uint32_t down = (uint32_t)min(f * (float)span, 4294967040.f);
    return hi - min(down, span - 1u);
}

// minimum / maximum over the 64 lanes of a wave, valid in lane 63 (same DPP pattern as the scan)
__device__ __forceinline__ void wave_min_max(uint32_t &mn, uint32_t &mx)
{
    // lanes without a source keep their own value (old = the value itself)
#define PDD_MINMAX_STEP(CTRL, ROWS)                                                                         \
    {                                                                                                       \
        const uint32_t a = (uint32_t)__builtin_amdgcn_update_dpp((int)mn, (int)mn, CTRL, ROWS, 0xf, false); \
        const uint32_t b = (uint32_t)__builtin_amdgcn_update_dpp((int)mx, (int)mx, CTRL, ROWS, 0xf, false); \
        mn = min(mn, a);                                                                                    \
        mx = max(mx, b);                                                                                    \
    }
    PDD_MINMAX_STEP(0x111, 0xf)
    PDD_MINMAX_STEP(0x112, 0xf)
    PDD_MINMAX_STEP(0x114, 0xf)
    PDD_MINMAX_STEP(0x118, 0xf)
    PDD_MINMAX_STEP(0x142, 0xa)
    PDD_MINMAX_STEP(0x143, 0xc)
#undef PDD_MINMAX_STEP
}

// The bracket [lo, hi] of a threshold search, which holds a key at least, cut to the keys that it holds.  A bisecting
// probe that cuts nothing has met a run of equal scores, and bisection would close in on it bit by bit, a round for each.
// First range_of_key for every key of the thread (from mn = 2^32 - 1, mx = 0): keys outside the bracket wrap past
// those inside, empty slots too.  Then narrow_bracket, with a word pair of this round's own, {2^32 - 1, 0} before.
__device__ __forceinline__ void range_of_key(uint32_t key, uint32_t lo, uint32_t hi, uint32_t &mn, uint32_t &mx)
{
    mn = min(mn, key - lo);
    mx = max(mx, key - (hi + 1u));
}
__device__ __forceinline__ void narrow_bracket(uint2 *range, uint32_t mn, uint32_t mx, int lane, uint32_t &lo, uint32_t &hi)
{
    wave_min_max(mn, mx);
    if (lane == 63) { atomicMin(&range->x, mn); atomicMax(&range->y, mx); }
    __syncthreads();
    lo += range->x;
    hi += 1u + range->y;
}

// Pooled scores of kSelPoolStep consecutive keys at a time, four per thread.  The scores of a step
// and the pool_r on either side of it pass through LDS once, 16 bytes per lane (the scores outside
// the sequence as zero, or as the nearest one inside it where the maximum is taken), those of the
// next step requested meanwhile; a window is added up (or its maximum taken) in key order from its first
// score on, as in pooled_score (a window of NaN stays NaN), the four windows of a thread from shared reads.
// (Read from memory by every window on its own, 2 r + 1 loads per key, the four prompts of 2360 to 12001
// keys x 8 heads took 34 us with r = 3 and 2480 us with r = 512; 20 and 87 us like this.)
constexpr int kSelPoolStep = 4 * kSelThreads;
constexpr int kSelPoolMax = 512;        // largest radius
typedef float pool_f32x4 __attribute__((ext_vector_type(4), aligned(4)));       // four scores at any score's address

struct PoolStage {
    const int r;
    const bool is_max;
    const float scale;                  // what the sum is multiplied with
    pool_f32x4 next[2];
    __device__ explicit PoolStage(const SelParams &p)
        : r(p.pool_r), is_max(p.pool_mode == kPoolMax), scale(is_max ? 1.f : p.pool_inv) {}

    // scores first - r + 4 tid .. + 3 and, where they belong to the step, the same kSelPoolStep further
    __device__ __forceinline__ void request(const float *seq, int nk, int first, int tid)
    {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int at = q * kSelPoolStep + 4 * tid, x = first - r + at;
            if (at < kSelPoolStep + 2 * r) {
                if (x >= 0 && x + 4 <= nk) next[q] = *(const pool_f32x4 *)(seq + x);
                else
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int in = min(max(x + j, 0), nk - 1);
                        next[q][j] = is_max || in == x + j ? seq[in] : 0.f;
                    }
            }
        }
    }

    // the thread's four pooled scores of keys first + 4 tid .. + 3
    __device__ __forceinline__ void step(const float *seq, int nk, int first, int number, bool more, int tid, float (&out)[4])
    {
        __shared__ __attribute__((aligned(16))) float stages[2][kSelPoolStep + 2 * kSelPoolMax];     // in turn: one barrier a step
        float *const stage = stages[number & 1];
        if (number == 0) request(seq, nk, first, tid);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int at = q * kSelPoolStep + 4 * tid;
            if (at < kSelPoolStep + 2 * r) *(float4 *)(stage + at) = make_float4(next[q][0], next[q][1], next[q][2], next[q][3]);
        }
        __syncthreads();
        if (more) request(seq, nk, first + kSelPoolStep, tid);
        const float4 *quads = (const float4 *)stage + tid;
        if (is_max) windows(quads, out, [](float a, float x) { return fmaxf(a, x); });
        else windows(quads, out, [](float a, float x) { return a + x; });
#pragma unroll
        for (int j = 0; j < 4; ++j) out[j] *= scale;
    }

    // window j = elements j .. j + 2 r from the first quad on
    template <typename Op>
    __device__ __forceinline__ void windows(const float4 *quads, float (&out)[4], Op op)
    {
        auto edge = [&](int q) {
            const float4 t = quads[q];
            const float v[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (4 * q + e == j) out[j] = v[e];
                    else if (4 * q + e > j && 4 * q + e <= j + 2 * r) out[j] = op(out[j], v[e]);
        };
        edge(0);
        int q = 1;
        for (; 4 * q + 3 <= 2 * r; ++q) {                        // in all four windows
            const float4 t = quads[q];
            const float v[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int j = 0; j < 4; ++j) out[j] = op(out[j], v[e]);
        }
        for (; 4 * q <= 2 * r + 3; ++q) edge(q);
    }
};

// Next pair a <= b of values to probe in the threshold search of select_topk_reg_kernel over the
// bracket [lo, hi] (lo < hi) that holds `inside` keys, of which the `need` largest (1 <= need <=
// inside) lie at or above the threshold; both in [lo + 1, hi].  With interpolate set, the keys are taken as
// evenly spread over the bracket, and the pair encloses the threshold's place by two standard
// deviations of the number of keys above it and a sixteenth of the keys (scores are evenly spread
// over no more than an octave); otherwise the bracket is cut into thirds.  (The approximate
// reciprocal and root only place the probes.)
__device__ __forceinline__ void next_pair(uint32_t lo, uint32_t hi, uint32_t inside, uint32_t need, bool interpolate,
                                          uint32_t &a, uint32_t &b)
{
    const uint32_t span = hi - lo;
    if (!interpolate) {
        a = lo + 1u + span / 3u;
        b = hi - span / 3u;
        return;
    }
    const float keys = (float)inside, each = __builtin_amdgcn_rcpf(keys), per_key = (float)span * each;
    const float down = (float)need - 0.5f;                        // keys between hi and the threshold
    const float dev = 2.f * __builtin_amdgcn_sqrtf(down * fmaxf(1.f - down * each, 0.f)) + 0.0625f * keys + 2.f;
    a = hi - min((uint32_t)fminf((down + dev) * per_key, 4294967040.f), span - 1u);
    b = hi - min((uint32_t)fminf(fmaxf(down - dev, 0.f) * per_key, 4294967040.f), hi - a);
}

// Wave 0's part of a histogram step over kSelBins bins, of which lane l looks after the 16 from 16 l on: the keys in
// the lane's bins, in those above them and in its fullest, and the bin with the key of a given rank from the top, the keys above that bin and in it.
struct SelBin { int bin; uint32_t above, own; };              // bin < 0: there is no such rank
__device__ __forceinline__ uint32_t hist_total(const uint32_t *hist, int lane, uint32_t &sum, uint32_t &above, uint32_t &most)
{
    sum = most = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint4 t = ((const uint4 *)hist)[4 * lane + ((q + lane) & 3)];     // turned, so that no two lanes meet in a bank
        sum += (t.x + t.y) + (t.z + t.w);
        most = max(max(most, max(t.x, t.y)), max(t.z, t.w));
    }
    const uint32_t incl = wave_incl_scan(sum), total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    above = total - incl;
    return total;
}
__device__ __forceinline__ SelBin hist_find(const uint32_t *hist, int lane, uint32_t sum, uint32_t above, int rank)
{
    const uint64_t at = __ballot((int)above < rank && rank <= (int)(above + sum));
    const int l = at ? (int)__builtin_ctzll(at) : 0;
    const uint32_t own = hist[16 * l + 15 - (lane & 15)];     // each row of 16 lanes: the lane's bins from the top
    uint32_t before = own;
    before += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)before, 0x111, 0xf, 0xf, true);
    before += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)before, 0x112, 0xf, 0xf, true);
    before += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)before, 0x114, 0xf, 0xf, true);
    before += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)before, 0x118, 0xf, 0xf, true);
    before += (uint32_t)__builtin_amdgcn_readlane((int)above, l) - own;
    const uint64_t in = __ballot((int)before < rank && rank <= (int)(before + own));
    const int e = in ? (int)__builtin_ctzll(in) : 0;
    return {at ? 16 * l + 15 - e : -1, (uint32_t)__builtin_amdgcn_readlane((int)before, e), (uint32_t)__builtin_amdgcn_readlane((int)own, e)};
}

// At most 64 vector registers, so that two workgroups (8 waves per SIMD) share a compute unit: the
// kernel lives on overlapping one row's barriers and latencies with another row's work
// (512 rows of 32768: 2.29 TB/s with two workgroups per compute unit, 1.85 with one).
template <int QPT, bool POOL>
__global__ __launch_bounds__(kSelThreads) __attribute__((amdgpu_waves_per_eu(8, 8)))
void select_topk_reg_kernel(const SelParams p)
{
    __shared__ uint32_t cnt[kSelWaves * QPT];          // per (i, wave): gt count | eq count << 16
    __shared__ uint32_t probe_tot[kSelMaxProbes];      // counts of pair number p, summed over the waves
    __shared__ __attribute__((aligned(16))) uint32_t hist[kSelBins], fin_keys[kSelFinish + 4];
    __shared__ uint32_t list[QPT > 1 ? kSelList : 1];
    __shared__ unsigned long long list_tot[2];         // keys inside a bracket | keys above it << 32
    __shared__ uint32_t sh_min, sh_max, fin_count, head_tot;
    __shared__ uint4 place;                            // lower and upper end of a bracket, keys above it and in it
    __shared__ struct { uint32_t T, above, upto; } fin;
    __shared__ uint2 range[kSelMaxProbes + 3];         // of round number p (and of two other steps), see narrow_bracket

    const int b = blockIdx.x, g = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int ks = min(max(p.cu_k[b], 0), p.total_k);
    const int ke = min(max(p.cu_k[b + 1], ks), p.total_k);
    const int nk = ke - ks;
    int c0 = p.cand_b ? p.cand_b[b] : 0;
    int c1 = p.cand_e ? p.cand_e[b] : nk;
    c0 = min(max(c0, 0), nk);
    c1 = min(max(c1, c0), nk);
    const int n = min(c1 - c0, 4 * kSelThreads * QPT);
    // Candidates 0 .. nhead-1 (at most three) precede the first 16-byte boundary of the row; lanes
    // 0 .. nhead-1 of wave 0 hold one each.  Candidate nhead + 4q + j is element j of quad q.
    const float *seq = p.scores + (int64_t)g * p.total_k + ks;
    const int nhead = POOL ? 0 : min((int)(((16u - ((uint32_t)(uintptr_t)(seq + c0) & 15u)) & 15u) >> 2), n);
    const int nq_el = n - nhead;                                 // candidates inside quads
    const int keep0 = min(max(p.cu_keep[b], 0), p.total_keep);
    const int keep1 = min(max(p.cu_keep[b + 1], keep0), p.total_keep);
    const int slots = keep1 - keep0;
    const int kk = min(min(max(p.k_per[b], 0), n), slots);

    int32_t *out = p.out_idx + (int64_t)g * p.total_keep + keep0;
    uint8_t *mrow = p.out_mask ? p.out_mask + (int64_t)g * p.total_k + ks : nullptr;

    // ---- everything that is read is requested here: a sample of a long row first, then the row.  Buffer loads, which
    // return zero outside the range: a branch around a load would wait for it.
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    const bool has_head = tid < nhead;
    const float *qbase = seq + c0 + nhead;                       // 16-byte aligned (unpooled)
    const int n_quads = nq_el / 4;                               // whole ones
    auto first_of = [&](int i) { return 4 * (i * kSelThreads + 64 * wave_u); };    // the wave's first index of a step
    uint32_t sample = 0, head = 0;
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    u32x4 quad[QPT];
    // QPT = 8: two steps at a time, else a wave waits to issue its loads while the chip's are queued (512 rows of 32768)
    constexpr int kEarly = QPT > 4 ? 3 : QPT > 2 ? 2 : QPT;
    const auto quads = __builtin_amdgcn_make_buffer_rsrc((void *)qbase, 0, 16 * n_quads, 0x00020000);
    auto request = [&](int from, int to) {
#pragma unroll
        for (int i = from; i < to; ++i) quad[i] = __builtin_amdgcn_raw_buffer_load_b128(quads, 16 * (i * kSelThreads + tid), 0, 0);
    };
    if constexpr (!POOL) {
        const auto row = __builtin_amdgcn_make_buffer_rsrc((void *)(seq + c0), 0, 4 * n, 0x00020000);
        // two lanes to each of 512 places spread over the row, so that a part of its lines holds it and it is there early
        if constexpr (QPT > 1)
            sample = __builtin_amdgcn_raw_buffer_load_b32(row, n > kSelList ? 4 * (((tid >> 1) * n >> 9) + 4 * (tid & 1)) : -4, 0, 0);
        head = __builtin_amdgcn_raw_buffer_load_b32(row, has_head ? 4 * tid : -4, 0, 0);
        request(0, kEarly);
    }

    hist[tid] = 0;
    if (tid < kSelMaxProbes + 3) range[tid] = make_uint2(0xffffffffu, 0u);
    if (tid < kSelMaxProbes) probe_tot[tid] = 0;
    if (tid < kSelFinish + 4) fin_keys[tid] = 0;
    if (tid == 0) {
        list_tot[0] = list_tot[1] = 0;
        fin_count = 0;
        sh_min = 0xffffffffu;
        sh_max = 0;
    }
    __syncthreads();
    if (p.pooled_out) {
        float *po = p.pooled_out + (int64_t)g * p.total_k + ks;
        if constexpr (POOL) {
            for (int x = tid; x < nk; x += kSelThreads) po[x] = pooled_score(seq, nk, x, p.pool_r, p.pool_mode, p.pool_inv);
        } else {
            for (int x = tid; x < nk; x += kSelThreads) po[x] = seq[x];
        }
    }
    if (mrow) {
        for (int x = tid; x < c0; x += kSelThreads) mrow[x] = 0;
        for (int x = c0 + n + tid; x < nk; x += kSelThreads) mrow[x] = 0;
    }
    for (int x = kk + tid; x < slots; x += kSelThreads) out[x] = -1;
    if (kk == 0) {
        if (mrow)
            for (int x = c0 + tid; x < c0 + n; x += kSelThreads) mrow[x] = 0;
        return;
    }

    uint32_t lo = 1u, hi = 0xffffffffu, c_lo = (uint32_t)n, c_above = 0;       // see the threshold search
    constexpr bool kLong = QPT > 1;                              // the instantiation takes rows beyond kSelList
    const bool is_long = kLong && n > kSelList;
    // ---- long rows: a histogram of some 1024 keys places the first bracket.  It encloses the threshold but for some three
    // standard deviations of its rank in the sample, and is made while the row is on its way.
    auto place_sample = [&](uint32_t k) {                        // k = 0: the thread has none
        uint32_t mn = k - 1u, mx = k;
        wave_min_max(mn, mx);
        if (lane == 63) { atomicMin(&sh_min, mn); atomicMax(&sh_max, mx); }
        if constexpr (!POOL && kEarly < QPT) request(kEarly, 2 * kEarly);
        __syncthreads();
        const uint32_t first = sh_min + 1u;
        const int shift = max(32 - __builtin_clz((sh_max - first) | 1u) - 10, 0);      // kSelBins = 2^10
        if (k != 0 && first < sh_max) atomicAdd(&hist[(k - first) >> shift], 1u);
        if constexpr (!POOL && kEarly < QPT) request(2 * kEarly, QPT);
        if (first == sh_max) {                                   // one value (1024 atomics on one bin take 2.5 us)
            lo = hi = first;
            return;
        }
        __syncthreads();
        if (wave == 0) {
            uint32_t sum, above, most;
            const uint32_t m = hist_total(hist, lane, sum, above, most);
            const float share = (float)kk * __builtin_amdgcn_rcpf((float)n), rank = share * (float)m;
            const float dev = 3.f * __builtin_amdgcn_sqrtf(rank * fmaxf(1.f - share, 0.f)) + 1.f;
            const SelBin up = hist_find(hist, lane, sum, above, (int)(rank - dev));
            const SelBin down = hist_find(hist, lane, sum, above, (int)(rank + dev) + 1);
            // no such rank: the bracket is open there
            const uint32_t end = ((uint32_t)max(up.bin, 0) << shift) + ((1u << shift) - 1u);
            if (lane == 0) place = make_uint4(down.bin < 0 ? 1u : first + ((uint32_t)down.bin << shift),
                                              up.bin < 0 || end > 0xffffffffu - first ? 0xffffffffu : first + end,
                                              up.bin == down.bin ? up.own : 0u, 0u);
        }
        __syncthreads();
        lo = place.x;
        hi = place.y;
        if (place.z > kSelRun) {                                 // scores that are equal?  Then the bracket is the one value
            uint32_t mn = 0xffffffffu, mx = 0, from = lo, to = hi;
            range_of_key(k, lo, hi, mn, mx);
            narrow_bracket(&range[kSelMaxProbes], mn, mx, lane, from, to);
            if (from == to) lo = hi = from;
        }
    };
    if constexpr (kLong && !POOL) {
        if (is_long && kk > 1 && kk < n) place_sample(order_key(__uint_as_float(sample)));
        else if constexpr (kEarly < QPT) request(kEarly, QPT);
    }

    // ---- keys into registers.  Slots outside the row hold key 0, which is below the key of
    // every score.
    const uint32_t khead = has_head ? order_key(__uint_as_float(head)) : 0u;      // (POOL: none)
    uint32_t key[QPT][4];
    PoolStage pool(p);
#pragma unroll
    for (int i = 0; i < QPT; ++i) {
        const int xw = first_of(i);
        if constexpr (POOL) {
            if (i * kSelPoolStep < n) {                          // the same in every thread
                float pooled[4];
                pool.step(seq, nk, c0 + i * kSelPoolStep, i, (i + 1) * kSelPoolStep < n, tid, pooled);
#pragma unroll
                for (int j = 0; j < 4; ++j) key[i][j] = (xw + 4 * lane + j < n) ? order_key(pooled[j]) : 0u;
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) key[i][j] = 0u;
            }
        } else if (xw + 255 < nq_el) {                           // all of the wave's 64 quads lie inside the row
#pragma unroll
            for (int j = 0; j < 4; ++j) key[i][j] = order_key(__uint_as_float(quad[i][j]));
        } else {
            const int left = nq_el - (xw + 4 * lane);
            float v[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = __uint_as_float(quad[i][j]);
            if (left > 0 && left < 4)                            // the row's last quad, one at most
                for (int j = 0; j < left; ++j) v[j] = qbase[xw + 4 * lane + j];
#pragma unroll
            for (int j = 0; j < 4; ++j) key[i][j] = j < left ? order_key(v[j]) : 0u;
        }
    }
    if constexpr (kLong && POOL) {
        if (is_long && kk > 1 && kk < n) {
            uint32_t k = key[0][0];
#pragma unroll
            for (int o = 1; o < QPT; ++o) k = (tid & (QPT - 1)) == o ? key[o][0] : k;
            place_sample(k);
        }
    }

    // ---- threshold search: the largest T with count(key >= T) >= kk, over the bracket [lo, hi] with
    // c_lo = count(key >= lo) >= kk > c_above = count(key > hi).
    // A step over all keys costs the workgroup by its instructions, four wavefronts to a SIMD, so
    //   * rows of up to 4096 candidates count all of them into bins over the row's range and go on in
    //     the bin that holds the threshold;
    //   * longer rows count the keys inside the sample's bracket and above it, and where the threshold is inside and
    //     at most 4096 keys are, these move to LDS and four to a thread; else rounds of two probes (see next_pair)
    //     over all keys come between;
    //   * two probes a round go on over those, and once at most kSelFinish are left they are ranked directly.
    // Every probed value is > lo > 0, so empty slots never count.
    uint32_t pa = 0, pb = 0;
    bool interp = true;
    int round = 0;
    // One round: `count` adds this wave's keys >= pa to its first argument and those >= pb to the second.
    // The waves' sums meet in an LDS counter of their own (one fresh counter per round, so none is ever
    // cleared), two to a word: a count is at most 32768.  `each` calls its argument with the thread's keys: a round
    // that cut nothing, by thirds, goes on from the range of the keys inside (five values in 20606 keys 47 -> 17 us, 27 with
    // one probe a round).  A round for which `at_ends` holds asks for the keys at the bracket's two ends alone.
    auto probe = [&](auto &&count, auto &&each, auto &&at_ends) {
        const uint32_t inside = c_lo - c_above;
        if (at_ends()) {
            pa = lo + 1u;
            pb = hi;
        } else next_pair(lo, hi, inside, (uint32_t)kk - c_above, interp, pa, pb);
        uint32_t ca = 0, cb = 0, la = 0, lb = 0;                 // of the wave; of the lane
        count(ca, cb, la, lb);
        const uint32_t both = (ca | cb << 16) + (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan(la | lb << 16), 63);
        if (lane == 0) atomicAdd(&probe_tot[round], both);
        __syncthreads();
        const uint32_t tot = probe_tot[round], tot_a = tot & 0xffffu, tot_b = tot >> 16;
        ++round;
        if (tot_b >= (uint32_t)kk) { lo = pb; c_lo = tot_b; }
        else {
            c_above = tot_b;
            hi = pb - 1u;
            if (tot_a >= (uint32_t)kk) { lo = pa; c_lo = tot_a; }
            else { hi = pa - 1u; c_above = tot_a; }
        }
        const bool thirds = !interp;                             // after interpolation these are tried first
        interp = thirds || 4u * (c_lo - c_above) <= inside;
        if (__builtin_expect(thirds && c_lo - c_above == inside && lo < hi, 0)) {
            uint32_t mn = 0xffffffffu, mx = 0;
            each([&](uint32_t k) { range_of_key(k, lo, hi, mn, mx); });
            narrow_bracket(&range[round - 1], mn, mx, lane, lo, hi);
        }
    };
    auto all_keys = [&](auto &&f) {
        f(khead);
#pragma unroll
        for (int i = 0; i < QPT; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) f(key[i][j]);
    };
    constexpr int NL = kSelList / kSelThreads + 1;
    uint32_t lk[NL];                                             // the thread's keys of the second part of the search
    uint32_t list_above = 0;                                     // keys above all of those
    if (kk == n || (is_long && kk == 1)) {
        if (kk == n) hi = lo;                                    // everything is kept: below or at the minimum, and no tie is cut
        else {                                                   // T is the maximum
            uint32_t mn = 0xffffffffu, mx = 0;
            all_keys([&](uint32_t k) { mx = max(mx, k); });
            wave_min_max(mn, mx);
            if (lane == 63) atomicMax(&sh_max, mx);
            __syncthreads();
            lo = hi = sh_max;
        }
    } else if (is_long) {
        // the keys inside [lo, hi], a bit for each, and the number above
        uint32_t in = 0, at = 0;
        bool head_in = false;
        auto divide = [&](unsigned long long *tot) {
            uint32_t from = 0, over = 0;                         // key[i][j] >= lo and > hi: bit 4 i + j
#pragma unroll
            for (int i = QPT - 1; i >= 0; --i)
#pragma unroll
                for (int j = 3; j >= 0; --j) {                   // empty slots hold key 0 < lo
                    from = 2u * from + (key[i][j] >= lo ? 1u : 0u);
                    over = 2u * over + (key[i][j] > hi ? 1u : 0u);
                }
            in = from & ~over;
            head_in = khead >= lo && khead <= hi;
            const uint32_t la = (uint32_t)__popc(over) + (khead > hi ? 1u : 0u);
            const uint32_t c = (uint32_t)__popc(in) + (head_in ? 1u : 0u);
            const uint32_t incl = wave_incl_scan(c | la << 16), all = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
            uint32_t before = 0;
            if (lane == 0) before = (uint32_t)atomicAdd(tot, (unsigned long long)(all & 0xffffu) | (unsigned long long)(all >> 16) << 32);
            at = (uint32_t)__builtin_amdgcn_readfirstlane((int)before) + (incl & 0xffffu) - c;
            __syncthreads();
            c_above = (uint32_t)(*tot >> 32);
            c_lo = c_above + (uint32_t)*tot;
        };
        divide(&list_tot[0]);
        const bool inside = c_above < (uint32_t)kk && (uint32_t)kk <= c_lo;
        bool fits = inside && lo < hi && c_lo - c_above <= (uint32_t)kSelList;
        if (__builtin_expect(!fits && !(inside && lo == hi), 0)) {
            if (c_above >= (uint32_t)kk) {                       // the threshold is above the bracket
                lo = hi + 1u;
                hi = 0xffffffffu;
                c_lo = c_above;
                c_above = 0;
            } else if ((uint32_t)kk > c_lo) {                    // below it
                hi = lo - 1u;
                lo = 1u;
                c_above = c_lo;
                c_lo = (uint32_t)n;
            }
            uint32_t mn = 0xffffffffu, mx = 0;
            all_keys([&](uint32_t k) { range_of_key(k, lo, hi, mn, mx); });
            narrow_bracket(&range[kSelMaxProbes + 2], mn, mx, lane, lo, hi);
            // Half of the comparisons are counted with a ballot and a scalar population count, half per lane on the vector unit
            // with one wave sum at the end: all on the scalar unit, which the waves share, the probes queue there.
            while (lo < hi && c_lo - c_above > (uint32_t)kSelList)
                probe([&](uint32_t &ca, uint32_t &cb, uint32_t &la, uint32_t &lb) {
                    ca = (uint32_t)__popcll(__ballot(khead >= pa));
                    cb = (uint32_t)__popcll(__ballot(khead >= pb));
#pragma unroll
                    for (int i = 0; i < QPT; ++i) {
#pragma unroll
                        for (int j = 0; j < 2; ++j) {
                            ca += (uint32_t)__popcll(__ballot(key[i][j] >= pa));
                            cb += (uint32_t)__popcll(__ballot(key[i][j] >= pb));
                            la += key[i][j + 2] >= pa ? 1u : 0u;
                            lb += key[i][j + 2] >= pb ? 1u : 0u;
                        }
                    }
                }, all_keys, [&] {                               // twice what a sample of many values leaves inside: a few share them
                    // (8 rows of 32768, k = half, of two values 18.9 -> 15.5 us, of seven 18.3 -> 14.9; 512 rows 40.4 -> 34.6, 35.2 -> 31.0)
                    return round == 0 && 4u * (c_lo - c_above) > (uint32_t)n;
                });
            fits = lo < hi;
            if (fits) divide(&list_tot[1]);
        }
        if (fits) {
            uint32_t *dst = list + at;
            if (head_in) *dst++ = khead;
#pragma unroll
            for (int i = 0; i < QPT; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (in >> (4 * i + j) & 1u) *dst++ = key[i][j];
            list_above = c_above;
            __syncthreads();
#pragma unroll
            for (int q = 0; q < NL; ++q) lk[q] = q * kSelThreads + tid < (int)(c_lo - c_above) ? list[q * kSelThreads + tid] : 0u;
            if (lo == 1u || hi == 0xffffffffu) {                 // an open end: probes are placed by the bracket's width
                uint32_t mn = 0xffffffffu, mx = 0;
#pragma unroll
                for (int q = 0; q < NL; ++q) range_of_key(lk[q], lo, hi, mn, mx);
                narrow_bracket(&range[kSelMaxProbes + 1], mn, mx, lane, lo, hi);
            }
        }
    } else {
        // the row's keys are all in lk (key 0 wraps to the largest value under key - 1 and so never is the minimum)
        uint32_t mn = khead - 1u, mx = khead;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            lk[j] = key[0][j];
            mn = min(mn, lk[j] - 1u);
            mx = max(mx, lk[j]);
        }
        lk[4] = khead;
        wave_min_max(mn, mx);
        if (lane == 63) { atomicMin(&sh_min, mn); atomicMax(&sh_max, mx); }
        __syncthreads();
        lo = sh_min + 1u;                                        // back from key - 1 (the row has a real key)
        hi = sh_max;
        if (kk == 1) {
            c_lo = 0;                                            // (not known)
            lo = hi;                                             // T is the maximum (8 x 681 6.0 -> 3.7 us)
        } else if (lo < hi && n > kSelFinish) {
            const int shift = max(32 - __builtin_clz(hi - lo) - 10, 0);     // kSelBins = 2^10
#pragma unroll
            for (int q = 0; q < NL; ++q)
                if (lk[q] != 0) atomicAdd(&hist[(lk[q] - lo) >> shift], 1u);
            __syncthreads();
            if (wave == 0) {
                uint32_t sum, above, most;
                hist_total(hist, lane, sum, above, most);
                const SelBin at = hist_find(hist, lane, sum, above, kk);
                const uint32_t first = (uint32_t)at.bin << shift;
                if (lane == 0) place = make_uint4(lo + first, lo + min(first + ((1u << shift) - 1u), hi - lo), at.above, at.own);
            }
            __syncthreads();
            lo = place.x;
            hi = place.y;
            c_above = place.z;
            c_lo = place.z + place.w;
        }
    }
    while (lo < hi && c_lo - c_above > (uint32_t)kSelFinish)
        probe([&](uint32_t &ca, uint32_t &, uint32_t &la, uint32_t &lb) {
            // the list has none of the keys above it
            if (wave == 0) ca = list_above | list_above << 16;
#pragma unroll
            for (int q = 0; q < NL; ++q) {
                la += lk[q] >= pa ? 1u : 0u;
                lb += lk[q] >= pb ? 1u : 0u;
            }
        }, [&](auto &&f) {
#pragma unroll
            for (int q = 0; q < NL; ++q) f(lk[q]);
        }, [] { return false; });
    if (lo < hi) {
        // at most kSelFinish keys lie in [lo, hi]: the (kk - c_above)-th largest of them is T
        const uint32_t width = hi - lo;
#pragma unroll
        for (int q = 0; q < NL; ++q)
            if (lk[q] - lo <= width) fin_keys[atomicAdd(&fin_count, 1u)] = lk[q];
        __syncthreads();
        // eight lanes to a key
        constexpr int PER = kSelThreads / kSelFinish;
        const int m = (int)(c_lo - c_above);
        const uint32_t mine = fin_keys[tid / PER];
        uint32_t above = 0, upto = 0;
#pragma unroll
        for (int q = 0; q < kSelFinish / (4 * PER); ++q) {       // slots past m hold 0: below every key
            const uint4 o4 = *(const uint4 *)(fin_keys + 4 * (q * PER + (tid & (PER - 1))));
            const uint32_t o[4] = {o4.x, o4.y, o4.z, o4.w};
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                above += o[x] > mine ? 1u : 0u;
                upto += o[x] >= mine ? 1u : 0u;
            }
        }
        uint32_t both = above | upto << 16;
#pragma unroll
        for (int off = 1; off < PER; off <<= 1) both += (uint32_t)__shfl_xor((int)both, off, 64);
        above = both & 0xffffu;
        upto = both >> 16;
        const uint32_t r = (uint32_t)kk - c_above;               // 1 <= r <= m
        if (tid / PER < m && above < r && r <= upto) { fin.T = mine; fin.above = c_above + above; fin.upto = c_above + upto; }    // equal keys only
        __syncthreads();
        lo = fin.T;
        c_above = fin.above;
        c_lo = fin.upto;
    }
    const uint32_t T = lo;
    const int krem = kk - (int)c_above;     // ties at T to keep (>= 1), lowest index first

    // ---- counts in index order: the head, then (i major, lane, j).  Common case: count(key >= T) = kk, every key equal to T is
    // kept (no tie is cut, e.g. T is unique), and a key is selected iff it is >= T.  Else the keys > T and == T are
    // counted apart, and of the latter the first krem kept.
    const bool all_ties = kk == n || c_lo == (uint32_t)kk;
    const uint32_t c_head = (has_head && khead > T ? 1u : 0u) | (has_head && khead == T ? 0x10000u : 0u);
    uint32_t pre_head = 0;                  // wave 0: exclusive prefix over the head lanes
    if (wave == 0) {
        const uint32_t incl = wave_incl_scan(c_head);
        pre_head = incl - c_head;
        if (lane == 63) head_tot = incl;
    }
    uint32_t pre[QPT];                      // prefix inside the wave: >= T, or packed gt | eq << 16
    uint32_t kept = 0;                      // all_ties: key[i][j] >= T at bit 4 i + j
    if (all_ties) {
#pragma unroll
        for (int i = QPT - 1; i >= 0; --i)
#pragma unroll
            for (int j = 3; j >= 0; --j) kept = 2u * kept + (key[i][j] >= T ? 1u : 0u);       // empty slots hold key 0 < T
        constexpr int NW = (QPT + 1) / 2;                        // two steps to a word: a wave's step has 256 keys
        uint32_t own[NW], incl[NW];
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            own[w] = (uint32_t)__popc(kept >> (8 * w) & 15u) | (2 * w + 1 < QPT ? (uint32_t)__popc(kept >> (8 * w + 4) & 15u) << 16 : 0u);
            incl[w] = own[w];
        }
        wave_incl_scan_n(incl);
#pragma unroll
        for (int i = 0; i < QPT; ++i) {
            const uint32_t upto = i & 1 ? incl[i >> 1] >> 16 : incl[i >> 1] & 0xffffu;
            pre[i] = upto - (i & 1 ? own[i >> 1] >> 16 : own[i >> 1] & 0xffffu);
            if (lane == 63) cnt[i * kSelWaves + wave] = upto;
        }
    } else {
        uint32_t incl[QPT];
#pragma unroll
        for (int i = 0; i < QPT; ++i) {
            uint32_t c = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                c += key[i][j] > T ? 1u : 0u;
                c += key[i][j] == T ? 0x10000u : 0u;
            }
            pre[i] = incl[i] = c;
        }
        wave_incl_scan_n(incl);
#pragma unroll
        for (int i = 0; i < QPT; ++i) {
            pre[i] = incl[i] - pre[i];                 // exclusive
            if (lane == 63) cnt[i * kSelWaves + wave] = incl[i];
        }
    }
    __syncthreads();
    // every wave scans the (step, wave) totals itself (at most 128 of them, two per lane) and picks
    // the offsets of its own QPT steps: no further barrier
    constexpr int NC = kSelWaves * QPT;
    uint32_t step_off[QPT];                 // the same before this wave's part of step i
    {
        const uint32_t ahead = all_ties ? (head_tot & 0xffffu) + (head_tot >> 16) : head_tot;
        uint32_t v[2] = {lane < NC ? cnt[lane] : 0u, 64 + lane < NC ? cnt[64 + lane] : 0u};
        uint32_t sc[2] = {v[0], v[1]};
        wave_incl_scan_n(sc);
        const uint32_t tot0 = (uint32_t)__builtin_amdgcn_readlane((int)sc[0], 63);
        const uint32_t ex0 = sc[0] - v[0] + ahead, ex1 = sc[1] - v[1] + tot0 + ahead;
#pragma unroll
        for (int i = 0; i < QPT; ++i) {
            const int e = i * kSelWaves + wave_u;
            step_off[i] = e < 64 ? (uint32_t)__builtin_amdgcn_readlane((int)ex0, e)
                                 : (uint32_t)__builtin_amdgcn_readlane((int)ex1, e - 64);
        }
    }

    // ---- stable compaction
    if (has_head) {
        const int gt_before = (int)(pre_head & 0xffffu), eq_before = (int)(pre_head >> 16);
        const bool sel = khead > T || (khead == T && eq_before < krem);
        if (sel) out[gt_before + min(eq_before, krem)] = c0 + tid;
        if (mrow) mrow[c0 + tid] = sel ? 1 : 0;
    }
    // the quads' mask bytes go out as one 4-byte store where the mask tensor is aligned like that
    const bool mask_dwords = mrow && (((uint32_t)(uintptr_t)(mrow + c0 + nhead)) & 3u) == 0;
    // The comparisons of the counting pass are made again here, against a copy of T the compiler
    // cannot relate to the first: kept alive across the scans, their 64 lane masks per wave do not
    // fit the scalar registers and are spilled lane by lane.
    uint32_t Tc = T;
    asm volatile("" : "+v"(Tc));
#pragma unroll
    for (int i = 0; i < QPT; ++i) {
        const int x0 = 4 * (i * kSelThreads + tid);
        const uint32_t before = step_off[i] + pre[i];
        uint32_t mbytes = 0;
        if (all_ties) {
            uint32_t pos = 4u * before;                          // in bytes
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool sel = key[i][j] >= Tc;
                if (sel) *(int32_t *)((uint8_t *)out + pos) = c0 + nhead + x0 + j;
                pos += sel ? 4u : 0u;
            }
            mbytes = (kept >> (4 * i) & 15u) * 0x00204081u & 0x01010101u;     // bit j to byte j
        } else {
            int gt_before = (int)(before & 0xffffu), eq_before = (int)(before >> 16);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool is_gt = key[i][j] > Tc, is_eq = key[i][j] == Tc;
                const bool sel = is_gt || (is_eq && eq_before < krem);
                if (sel) out[gt_before + min(eq_before, krem)] = c0 + nhead + x0 + j;
                gt_before += is_gt ? 1 : 0;
                eq_before += is_eq ? 1 : 0;
                mbytes |= sel ? (1u << (8 * j)) : 0u;
            }
        }
        if (mrow && x0 < nq_el) {
            uint8_t *mp = mrow + c0 + nhead + x0;
            if (mask_dwords && x0 + 3 < nq_el) *(uint32_t *)mp = mbytes;
            else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (x0 + j < nq_el) mp[j] = (uint8_t)((mbytes >> (8 * j)) & 1u);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Radix selection for rows longer than 32768 candidates (keys re-read from L2).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kSelThreads) void select_topk_kernel(const SelParams p)
{
    __shared__ uint32_t hist[256];
    __shared__ int32_t sh_bin, sh_above;
    __shared__ int32_t wave_gt[kSelWaves], wave_eq[kSelWaves];

    const int b = blockIdx.x, g = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int ks = min(max(p.cu_k[b], 0), p.total_k);
    const int ke = min(max(p.cu_k[b + 1], ks), p.total_k);
    const int nk = ke - ks;
    int c0 = p.cand_b ? p.cand_b[b] : 0;
    int c1 = p.cand_e ? p.cand_e[b] : nk;
    c0 = min(max(c0, 0), nk);
    c1 = min(max(c1, c0), nk);
    const int n = c1 - c0;
    const int keep0 = min(max(p.cu_keep[b], 0), p.total_keep);
    const int keep1 = min(max(p.cu_keep[b + 1], keep0), p.total_keep);
    const int slots = keep1 - keep0;
    const int kk = min(min(max(p.k_per[b], 0), n), slots);

    const float *seq = p.scores + (int64_t)g * p.total_k + ks;
    int32_t *out = p.out_idx + (int64_t)g * p.total_keep + keep0;
    uint8_t *mrow = p.out_mask ? p.out_mask + (int64_t)g * p.total_k + ks : nullptr;
    auto cand_key = [&](int x) {
        return order_key(pooled_score(seq, nk, c0 + x, p.pool_r, p.pool_mode, p.pool_inv));
    };

    if (p.pooled_out) {
        float *po = p.pooled_out + (int64_t)g * p.total_k + ks;
        for (int x = tid; x < nk; x += kSelThreads) po[x] = pooled_score(seq, nk, x, p.pool_r, p.pool_mode, p.pool_inv);
    }
    // mask outside the candidate range, unused index slots
    if (mrow) {
        for (int x = tid; x < c0; x += kSelThreads) mrow[x] = 0;
        for (int x = c1 + tid; x < nk; x += kSelThreads) mrow[x] = 0;
    }
    for (int x = kk + tid; x < slots; x += kSelThreads) out[x] = -1;
    if (kk == 0) {
        if (mrow)
            for (int x = c0 + tid; x < c1; x += kSelThreads) mrow[x] = 0;
        return;
    }

    // ---- the row's key range
    __shared__ uint32_t wave_min[kSelWaves], wave_max[kSelWaves];
    uint32_t kmin = 0xffffffffu, kmax = 0u;
#pragma unroll 8
    for (int x = tid; x < n; x += kSelThreads) {
        const uint32_t key = cand_key(x);
        kmin = min(kmin, key);
        kmax = max(kmax, key);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        kmin = min(kmin, (uint32_t)__shfl_xor((int)kmin, off, 64));
        kmax = max(kmax, (uint32_t)__shfl_xor((int)kmax, off, 64));
    }
    if (lane == 0) { wave_min[wave] = kmin; wave_max[wave] = kmax; }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kSelWaves; ++w) { kmin = min(kmin, wave_min[w]); kmax = max(kmax, wave_max[w]); }
    const uint32_t range = kmax - kmin;
    const int nbits = 32 - __builtin_clz(range | 1u);        // 1 .. 32
    const int passes = (nbits + 7) >> 3;                     // 1 .. 4
    const int lsh = 8 * passes - nbits;                      // scaled key = (key - kmin) << lsh < 2^(8 passes)
    const bool aggregate = nbits < 12;

    // ---- radix select on the scaled keys: afterwards `prefix` is the scaled key of the kk-th largest
    uint32_t prefix = 0;
    int krem = kk;
    for (int pass = 0; pass < passes; ++pass) {
        const int shift = 8 * (passes - 1 - pass);
        if (tid < 256) hist[tid] = 0;
        __syncthreads();
#pragma unroll 4
        for (int x0 = 0; x0 < n; x0 += kSelThreads) {
            const int x = x0 + tid;
            const bool in = x < n;
            const uint32_t sk = in ? (cand_key(x) - kmin) << lsh : 0u;
            // digits above the current one must equal the prefix found so far
            const bool part = in && (pass == 0 || (sk >> (shift + 8)) == prefix);
            const uint32_t bin = (sk >> shift) & 255u;
            if (!aggregate) {
                // wide key range: the scaled digits spread over the bins, plain LDS atomics
                if (part) atomicAdd(&hist[bin], 1u);
            } else {
                // narrow range (many equal keys): lanes that share the first participating
                // lane's bin are counted with a single atomic
                const uint64_t pm = __ballot(part);
                if (pm) {
                    const int leader = __ffsll((unsigned long long)pm) - 1;
                    const uint32_t lbin = __builtin_amdgcn_readlane(bin, leader);
                    const uint64_t same = __ballot(part && bin == lbin);
                    if (lane == leader) atomicAdd(&hist[lbin], (uint32_t)__popcll(same));
                    if (part && bin != lbin) atomicAdd(&hist[bin], 1u);
                }
            }
        }
        __syncthreads();
        if (wave == 0) {
            // lane L owns bins 4L .. 4L+3 ; `above` = count in bins greater than d
            uint32_t c[4];
            uint32_t sum4 = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) { c[i] = hist[4 * lane + i]; sum4 += c[i]; }
            uint32_t incl = sum4;   // inclusive suffix sum over lanes >= L
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const uint32_t o = __shfl_down(incl, off, 64);
                if (lane + off < 64) incl += o;
            }
            uint32_t above = incl - sum4;
#pragma unroll
            for (int i = 3; i >= 0; --i) {
                if ((uint32_t)krem > above && (uint32_t)krem <= above + c[i]) {
                    sh_bin = 4 * lane + i;
                    sh_above = (int32_t)above;
                }
                above += c[i];
            }
        }
        __syncthreads();
        prefix = (prefix << 8) | (uint32_t)sh_bin;
        krem -= sh_above;
        __syncthreads();
    }
    const uint32_t T = kmin + (prefix >> lsh);   // threshold key; `krem` (>= 1) ties at T are kept, lowest index first

    // ---- stable compaction: each wave owns a contiguous slice of the candidates
    const int seg = ((n + kSelWaves - 1) / kSelWaves + 63) & ~63;
    const int s0 = min(wave * seg, n), s1 = min(s0 + seg, n);
    int cgt = 0, ceq = 0;
    for (int x0 = s0; x0 < s1; x0 += 64) {
        const int x = x0 + lane;
        const bool in = x < s1;
        const uint32_t key = in ? cand_key(x) : 0u;
        cgt += __popcll(__ballot(in && key > T));
        ceq += __popcll(__ballot(in && key == T));
    }
    if (lane == 0) { wave_gt[wave] = cgt; wave_eq[wave] = ceq; }
    __syncthreads();
    int gt_before = 0, eq_before = 0;
    for (int w = 0; w < wave; ++w) { gt_before += wave_gt[w]; eq_before += wave_eq[w]; }
    int sel_before = gt_before + min(eq_before, krem);
    const uint64_t lt_mask = (1ull << lane) - 1ull;
    for (int x0 = s0; x0 < s1; x0 += 64) {
        const int x = x0 + lane;
        const bool in = x < s1;
        const uint32_t key = in ? cand_key(x) : 0u;
        const bool is_gt = in && key > T, is_eq = in && key == T;
        const uint64_t be = __ballot(is_eq);
        const int eq_rank = eq_before + __popcll(be & lt_mask);
        const bool sel = is_gt || (is_eq && eq_rank < krem);
        const uint64_t bs = __ballot(sel);
        if (sel) out[sel_before + __popcll(bs & lt_mask)] = c0 + x;
        if (mrow && in) mrow[c0 + x] = sel ? 1 : 0;
        sel_before += __popcll(bs);
        eq_before += __popcll(be);
    }
}

}  // namespace pdd
