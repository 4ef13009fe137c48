// Top-k selection with the candidates of a row divided over workgroups (paper Section 3.2, "Prompt
// Refiner"; the same outputs as select_topk.hpp, byte for byte), for rows that one workgroup is
// too little for.
//
// One workgroup of 1024 threads per (row, chunk of 4096 QPT candidates); two launches with a caller
// workspace between them, and no workgroup that waits for another one.
//   select_bracket_kernel   Every workgroup draws the same sample of the row, one key from each of 1024
//                           equal pieces, and takes from its histogram two edges that enclose the threshold's
//                           place by four and a half standard deviations of its rank.  Of the chunk's keys those above,
//                           those equal to the upper edge, those between and those equal to the lower edge are
//                           counted; those between, a tenth of the row, go to the workspace by 256 bins.
//   select_divided_kernel   The chunks' counts give the threshold's class and bin, the bin's keys (some
//                           tens) are ranked, and the chunk's indices and mask written.
// Where the histogram has a bin of many keys, the edges' bins are divided anew: a value that many keys share
// becomes an edge, whose equals are counted and never listed.  A bin of more than kDivListMax keys (a value between the
// edges that a twentieth of a long row shares) is read where it lies: if its smallest and largest key are one, that is the
// threshold, else its digits give it.  Where the threshold lies outside the edges all the same (one row in a hundred
// thousand), every workgroup searches the row by itself.
// Bound by the latency of its steps (loads, scans, barriers, launches) up to some 10 rows, by
// instruction issue beyond.  By a radix search of three digits, a launch for each and one for the output, 8 rows of
// 131072 candidates took 21.7 us, 16 of 400000 81, 128 of 131072 162; now 16.5, 37.6 and 79 (k = 10 %).  Of the first
// kernel's 11500 cycles 1100 go to the row's bounds, 4500 to the sample and the keys, 1100 to the sample's range, 2300 to its
// histogram, 1800 to the classes and 700 to the lists; the second takes as long.  (The edges from exact order
// statistics of the sample, by single probes of one wave, took 12000 cycles.)
#pragma once
#include "select_topk.hpp"

namespace pdd {

constexpr int kSplitSelChunk = 4 * kSelThreads;       // candidates per workgroup and step, four per thread
constexpr int kDivSample = kSelThreads;               // keys of the sample, one per thread
constexpr uint32_t kDivBinMany = 24;                  // keys of the sample in one of its 1024 bins that are no even spread
constexpr int kDivBins = 256;                         // of the keys between the edges
constexpr int kDivGroups = kSelThreads / 32;          // half waves of a workgroup
constexpr int kDivListMax = 12 * kSelThreads;         // keys of one bin that a workgroup ranks in LDS

// What a workgroup leaves in the workspace: its keys above the upper edge `hi`, equal to it, strictly between
// the edges, equal to the lower one `lo` (0 where lo == hi), 16384 at most.
struct DivCounts { uint16_t above, at_hi, between, at_lo; };

struct SplitSelParams {
    SelParams s;
    int32_t n_chunks, n_units;  // of the longest sequence: workgroups, three at least; 4096 candidates
    uint16_t *list;             // [rows][n_units][4096]: a workgroup's keys between the edges, by bins
    uint16_t *before;           // [rows][n_chunks][kDivBins]: where a bin starts among them
    DivCounts *counts;          // [rows][n_chunks]
    uint2 *row;                 // [rows][n_chunks], of the row: {lo, hi}, {first key of bin 1 less its width, log2 of the width}
};
constexpr size_t kSplitSelChunkBytes = (kSplitSelChunk + kDivBins) * sizeof(uint16_t) + sizeof(DivCounts) + sizeof(uint2);   // of 4096 candidates

// Whether a bin's list holds the low bits of its keys, or else the candidates' numbers in their workgroup
// (the outer bins take what lies beyond them too).
__device__ __forceinline__ bool div_by_value(uint32_t bin, int shift) { return shift <= 16 && bin > 0 && bin < (uint32_t)kDivBins - 1u; }

typedef float sel_f32x4 __attribute__((ext_vector_type(4), aligned(4)));        // four scores at any score's address
typedef uint32_t sel_u32_any __attribute__((aligned(1)));                       // four mask bytes at any address

struct SelRow {
    const float *cand;         // the row's candidates
    int nk, c0, n, chunks, kk, slots, keep0;
    int64_t row, at;           // row = head * B + sequence; first mask element of the sequence
};

template <int QPT>
__device__ __forceinline__ SelRow split_sel_row(const SelParams &p, int n_units)
{
    SelRow r;
    const int b = blockIdx.y, g = blockIdx.z;
    const int ks = min(max(p.cu_k[b], 0), p.total_k);
    const int ke = min(max(p.cu_k[b + 1], ks), p.total_k);
    r.nk = ke - ks;
    const int c0 = min(max(p.cand_b ? p.cand_b[b] : 0, 0), r.nk);
    const int c1 = min(max(p.cand_e ? p.cand_e[b] : r.nk, c0), r.nk);
    r.c0 = c0;
    r.n = min(c1 - c0, n_units * kSplitSelChunk);                // what the workspace has room for
    r.chunks = (r.n + kSplitSelChunk * QPT - 1) / (kSplitSelChunk * QPT);
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

// The fourth largest of the sixteen values a workgroup's waves left in LDS, every wave for itself.
__device__ __forceinline__ uint32_t fourth_largest(const uint32_t *of_wave, int lane)
{
    const uint32_t mine = of_wave[lane & 15];
    uint32_t larger = 0;                                         // and equal ones of a lower number
#pragma unroll
    for (int q = 0; q < kSelWaves / 4; ++q) {
        const uint4 o = ((const uint4 *)of_wave)[q];
        const uint32_t v[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) larger += v[e] > mine || (v[e] == mine && 4 * q + e < (lane & 15)) ? 1u : 0u;
    }
    const int at = __ffsll((unsigned long long)__ballot(larger == 3u)) - 1;
    return (uint32_t)__builtin_amdgcn_readlane((int)mine, at);
}

// Registers for eight waves per SIMD, so that two workgroups share a compute unit.
template <int QPT>
__global__ __launch_bounds__(kSelThreads) __attribute__((amdgpu_waves_per_eu(8, 8))) void select_bracket_kernel(const SplitSelParams p)
{
    __shared__ __attribute__((aligned(16))) uint32_t hist[2][kSelBins], bins[kDivBins], top_of[kSelWaves], bottom_of[kSelWaves];
    __shared__ uint32_t sh_min, sh_max, sh_uneven, sh_count[3];
    __shared__ struct { uint32_t bin, keys, above; } place[2];   // a bin of the sample's histogram, its keys, those above it
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int chunk = blockIdx.x;
    const SelRow r = split_sel_row<QPT>(p.s, p.n_units);
    if (chunk >= r.chunks || r.kk == 0) return;
    // one key from each of m equal pieces of the row, at a place that only the piece's number decides
    const int m = min(r.n, kDivSample);
    uint32_t mine = 0;
    if (tid < m) {
        const uint32_t mix = (uint32_t)tid * 2654435761u;
        const uint32_t at = m < kDivSample ? (uint32_t)tid
                                           : (uint32_t)((uint64_t)((uint32_t)tid << 16 | mix >> 16) * (uint32_t)r.n >> 26);    // kDivSample = 2^10
        mine = order_key(r.cand[at]);
    }
    uint32_t key[QPT][4];
#pragma unroll
    for (int i = 0; i < QPT; ++i) split_sel_keys(r, (chunk * QPT + i) * kSplitSelChunk + 4 * tid, key[i]);
    hist[0][tid] = hist[1][tid] = 0;
    if (tid < kDivBins) bins[tid] = 0;
    if (tid < 3) sh_count[tid] = 0;
    if (tid == 0) { sh_min = 0xffffffffu; sh_max = 0; }
    __syncthreads();
    {
        uint32_t mn = mine - 1u, mx = mine;                       // an empty slot is never the minimum
        wave_min_max(mn, mx);
        if (lane == 63) { atomicMin(&sh_min, mn); atomicMax(&sh_max, mx); }
    }
    __syncthreads();
    // The sample in bins of equal width: the two edges are the outer bounds of the bins in which their ranks lie.
    const float share = (float)r.kk / (float)r.n, rank = share * (float)m;
    const float dev = 4.5f * __builtin_amdgcn_sqrtf(rank * fmaxf(1.f - share, 0.f)) + 1.f;
    const int above = (int)floorf(rank - dev), below = (int)(rank + dev) + 2;         // in the sample, from the top
    const bool has[2] = {above >= 1, below <= m};
    const uint32_t bottom = sh_min + 1u, top = sh_max;
    const int width0 = max(32 - __builtin_clz((top - bottom) | 1u) - 10, 0);             // kSelBins = 2^10
    if (mine != 0) atomicAdd(&hist[0][(mine - bottom) >> width0], 1u);
    // wave 0 looks for the upper edge, wave 1 for the lower one
    auto look = [&](const uint32_t *h, int want) {
        uint32_t sum, over, most;
        hist_total(h, lane, sum, over, most);
        const SelBin at = hist_find(h, lane, sum, over, want);
        if (lane == 0 && at.bin >= 0) place[wave] = {(uint32_t)at.bin, at.own, at.above};
        return most;
    };
    __syncthreads();
    if (wave < 2) {
        const uint32_t most = look(hist[0], wave == 0 ? above : below);
        if (wave == 0 && lane == 0) sh_uneven = 0;
        if (wave == 0 && most > kDivBinMany) sh_uneven = 1;
    }
    __syncthreads();
    uint32_t lo = has[1] ? bottom + (place[1].bin << width0) - 1u : 0u;
    uint32_t hi = has[0] ? bottom + min((place[0].bin + 1u) << width0, 0xffffffffu - bottom) : 0xffffffffu;
    uint32_t base = has[1] ? lo + 1u : bottom, end = has[0] ? hi : top;       // what the bins of the keys between cover
    if (sh_uneven) {                                              // the same in every workgroup of the row
        // Some bin holds many keys, which may be equal ones: the edges' bins are divided anew until they do not, or
        // until they are one key value, which is then the edge itself and its keys are counted as equal to it.
        uint32_t low[2] = {bottom + (place[0].bin << width0), bottom + (place[1].bin << width0)};
        int width[2] = {width0, width0}, want[2] = {above - (int)place[0].above, below - (int)place[1].above};
        for (;;) {
            const bool again[2] = {has[0] && place[0].keys > kDivBinMany && width[0] > 0, has[1] && place[1].keys > kDivBinMany && width[1] > 0};
            if (!again[0] && !again[1]) break;                    // ten bits each time: four times at most
            hist[0][tid] = hist[1][tid] = 0;
            __syncthreads();
#pragma unroll
            for (int e = 0; e < 2; ++e)
                if (again[e]) {
                    const bool in = mine >= low[e] && mine - low[e] < 1u << width[e];
                    width[e] = max(width[e] - 10, 0);
                    if (in) atomicAdd(&hist[e][(mine - low[e]) >> width[e]], 1u);
                }
            __syncthreads();
            if (wave < 2 && again[wave]) look(hist[wave], want[wave]);
            __syncthreads();
#pragma unroll
            for (int e = 0; e < 2; ++e)
                if (again[e]) {
                    low[e] += place[e].bin << width[e];
                    want[e] -= (int)place[e].above;
                }
        }
        if (has[0]) hi = width[0] == 0 ? low[0] : low[0] + min(1u << width[0], 0xffffffffu - low[0]);
        if (has[1]) lo = width[1] == 0 ? low[1] : low[1] - 1u;
        // and the bins cover all but the outermost of the sample between the edges: what lies beyond falls into
        // the first and the last one
        const bool in = mine > lo && mine < hi;
        uint32_t mn = in ? mine : 0xffffffffu, mx = in ? mine : 0u;
        wave_min_max(mn, mx);
        if (lane == 63) { bottom_of[wave] = ~mn; top_of[wave] = mx; }
        __syncthreads();
        base = ~fourth_largest(bottom_of, lane);
        end = fourth_largest(top_of, lane);
        if (base > end) { base = lo + 1u; end = hi; }             // next to nothing between
    }
    const uint32_t span = max(end, base) - base;
    const int shift = max(32 - __builtin_clz(max(span, 1u)) - 8, 0);         // kDivBins = 2^8
    uint32_t n_above = 0, n_hi = 0, n_lo = 0, bin[QPT][4], slot[QPT][4];
#pragma unroll
    for (int i = 0; i < QPT; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t k = key[i][j];                         // an empty slot, key 0, is in no class
            n_above += (uint32_t)__popcll(__ballot(k > hi));
            n_hi += (uint32_t)__popcll(__ballot(k == hi));
            n_lo += (uint32_t)__popcll(__ballot(k == lo && lo < hi && k != 0));
            bin[i][j] = kDivBins;
            if (k > lo && k < hi) {
                bin[i][j] = min((max(k, base) - base) >> shift, (uint32_t)kDivBins - 1u);
                slot[i][j] = atomicAdd(&bins[bin[i][j]], 1u);
            }
        }
    if (lane == 0) {
        if (n_above) atomicAdd(&sh_count[0], n_above);
        if (n_hi) atomicAdd(&sh_count[1], n_hi);
        if (n_lo) atomicAdd(&sh_count[2], n_lo);
    }
    __syncthreads();
    const int64_t at = r.row * p.n_chunks + chunk;
    if (wave == 0) {
        const uint4 h = ((const uint4 *)bins)[lane];
        const uint32_t sum = (h.x + h.y) + (h.z + h.w), incl = wave_incl_scan(sum);
        const uint32_t b0 = incl - sum, b1 = b0 + h.x, b2 = b1 + h.y, b3 = b2 + h.z;
        ((uint4 *)bins)[lane] = make_uint4(b0, b1, b2, b3);
        ((uint2 *)(p.before + at * kDivBins))[lane] = make_uint2(b0 | b1 << 16, b2 | b3 << 16);
        if (lane == 63)
            p.counts[at] = DivCounts{(uint16_t)sh_count[0], (uint16_t)sh_count[1], (uint16_t)incl, (uint16_t)sh_count[2]};
        if (chunk == 0 && lane < 2) p.row[at + lane] = lane == 0 ? make_uint2(lo, hi) : make_uint2(base, (uint32_t)shift);
    }
    __syncthreads();
    uint16_t *const list = p.list + (r.row * p.n_units + chunk * QPT) * kSplitSelChunk;
#pragma unroll
    for (int i = 0; i < QPT; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (bin[i][j] < kDivBins)
                list[bins[bin[i][j]] + slot[i][j]] =
                    (uint16_t)(div_by_value(bin[i][j], shift) ? (key[i][j] - base) & ((1u << shift) - 1u) : (uint32_t)(i * kSplitSelChunk + 4 * tid + j));
}

// The key of rank `rank` from the top among at most kSelFinish keys in LDS (zeros behind them), eight
// lanes to a key, written to *out by the lanes whose key it is.
__device__ __forceinline__ void short_key_of_rank(const uint32_t *keys, int m, uint32_t rank, int tid, uint32_t *out)
{
    constexpr int PER = kSelThreads / kSelFinish;
    const uint32_t mine = keys[tid / PER];
    uint32_t both = 0;                                           // keys above it | at or above it << 16
#pragma unroll
    for (int q = 0; q < kSelFinish / (4 * PER); ++q) {
        if (4 * q * PER >= m) break;
        const uint4 o = *(const uint4 *)(keys + 4 * (q * PER + (tid & (PER - 1))));
        both += (o.x > mine ? 1u : 0u) + (o.x >= mine ? 0x10000u : 0u) + (o.y > mine ? 1u : 0u) + (o.y >= mine ? 0x10000u : 0u) +
                (o.z > mine ? 1u : 0u) + (o.z >= mine ? 0x10000u : 0u) + (o.w > mine ? 1u : 0u) + (o.w >= mine ? 0x10000u : 0u);
    }
#pragma unroll
    for (int off = 1; off < PER; off <<= 1) both += (uint32_t)__shfl_xor((int)both, off, 64);
    if (tid / PER < m && (both & 0xffffu) < rank && rank <= both >> 16) *out = mine;      // equal keys only
}

// The key of rank `rank` from the top among the m keys of an LDS list (1 <= rank <= m, zeros behind them up to
// kSelFinish), by the whole workgroup.  Keys are not 0.
__device__ __forceinline__ uint32_t list_key_of_rank(const uint32_t *list, int m, uint32_t rank, int tid, int lane)
{
    __shared__ __attribute__((aligned(16))) uint32_t fin_keys[kSelFinish];
    __shared__ uint32_t probe_tot[kSelMaxProbes], fin_count, fin_T;
    __shared__ uint2 range[kSelMaxProbes];
    if (m <= kSelFinish) {                                       // the same in every thread
        short_key_of_rank(list, m, rank, tid, &fin_T);
        __syncthreads();
        return fin_T;
    }
    uint32_t lo = 1, hi = 0xffffffffu, c_lo = (uint32_t)m, c_above = 0;
    if (tid < kSelFinish) fin_keys[tid] = 0;
    if (tid == 0) fin_count = 0;
    if (tid < kSelMaxProbes) {
        probe_tot[tid] = 0;
        range[tid] = make_uint2(0xffffffffu, 0u);
    }
    __syncthreads();
    bool interp = true, narrow = true;
    for (int probe = 0; lo < hi && c_lo - c_above > (uint32_t)kSelFinish; ++probe) {
        if (narrow) {                                            // to the keys that the bracket holds
            uint32_t mn = 0xffffffffu, mx = 0;
            for (int x = tid; x < m; x += kSelThreads) range_of_key(list[x], lo, hi, mn, mx);
            narrow_bracket(&range[probe], mn, mx, lane, lo, hi);
            if (lo >= hi) break;
        }
        const uint32_t inside = c_lo - c_above;
        const uint32_t mid = next_probe(lo, hi, inside, rank - c_above, interp);
        uint32_t c = 0;
        for (int x = tid; x < m; x += kSelThreads) c += list[x] >= mid ? 1u : 0u;
        c = wave_incl_scan(c);
        if (lane == 63) atomicAdd(&probe_tot[probe], c);
        __syncthreads();
        c = probe_tot[probe];
        if (c >= rank) { lo = mid; c_lo = c; }
        else { hi = mid - 1u; c_above = c; }
        const bool halved = !interp;
        interp = halved || 4u * (c_lo - c_above) <= inside;
        narrow = halved && c_lo - c_above == inside;
    }
    if (lo >= hi) return lo;                                     // the same in every thread
    for (int x = tid; x < m; x += kSelThreads)
        if (list[x] - lo <= hi - lo) fin_keys[atomicAdd(&fin_count, 1u)] = list[x];
    __syncthreads();
    short_key_of_rank(fin_keys, (int)(c_lo - c_above), rank - c_above, tid, &fin_T);
    __syncthreads();
    return fin_T;
}

// The same threshold without a bracket: keys by four digits of eight bits, read anew for each.  `each` calls its
// argument with (key, whether the lane has one), all lanes of a wave together.
template <typename Each>
__device__ __forceinline__ uint32_t any_key_of_rank(Each &&each, uint32_t rank, int tid, int lane, int wave)
{
    __shared__ uint32_t hist[256], sh_bin, sh_rank;
    uint32_t prefix = 0;
    for (int shift = 24; shift >= 0; shift -= 8) {
        if (tid < 256) hist[tid] = 0;
        __syncthreads();
        each([&](uint32_t k, bool has) {
            const uint32_t bin = k >> shift & 255u;
            const bool part = has && (shift == 24 || k >> (shift + 8) == prefix);
            const uint64_t parts = __ballot(part);
            if (parts) {                                         // the lanes of the first one's bin add as one
                const int first = __ffsll((unsigned long long)parts) - 1;
                const uint32_t common = (uint32_t)__builtin_amdgcn_readlane((int)bin, first);
                const uint64_t same = __ballot(part && bin == common);
                if (lane == first) atomicAdd(&hist[common], (uint32_t)__popcll(same));
                if (part && bin != common) atomicAdd(&hist[bin], 1u);
            }
        });
        __syncthreads();
        if (wave == 0) {
            const uint4 h = make_uint4(hist[4 * lane], hist[4 * lane + 1], hist[4 * lane + 2], hist[4 * lane + 3]);
            const uint32_t own[4] = {h.x, h.y, h.z, h.w}, sum = (h.x + h.y) + (h.z + h.w), incl = wave_incl_scan(sum);
            uint32_t run = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63) - incl;
#pragma unroll
            for (int e = 3; e >= 0; --e) {
                if (run < rank && rank <= run + own[e]) { sh_bin = (uint32_t)(4 * lane + e); sh_rank = rank - run; }
                run += own[e];
            }
        }
        __syncthreads();
        prefix = prefix << 8 | sh_bin;
        rank = sh_rank;
    }
    return prefix;
}

template <int QPT>
__global__ __launch_bounds__(kSelThreads) __attribute__((amdgpu_waves_per_eu(8, 8))) void select_divided_kernel(const SplitSelParams p)
{
    __shared__ __attribute__((aligned(16))) uint32_t bin_part[kSelWaves][kDivBins], bin_sum[kDivBins], list[kDivListMax];
    __shared__ uint2 bin_own[kDivGroups];              // keys of the bin and of higher ones in a chunk
    __shared__ uint32_t step_own[kSelWaves * QPT], list_above, list_before, row_count[3];
    __shared__ uint2 heavy;                            // smallest and largest key of a bin
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int chunk = blockIdx.x;
    const SelRow r = split_sel_row<QPT>(p.s, p.n_units);
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

    const int64_t row0 = r.row * p.n_chunks;
    const DivCounts *counts = p.counts + row0;
    const uint16_t *before = p.before + row0 * kDivBins;
    // ---- what the chunks hold: a lane has a chunk's classes, a half wave where the bins of a chunk start, eight a lane
    uint2 cls = lane < r.chunks ? *(const uint2 *)&counts[lane] : make_uint2(0, 0);
    const uint2 edges = p.row[row0], binning = p.row[row0 + 1];
    const uint32_t lo = edges.x, hi = edges.y, kk = (uint32_t)r.kk;
    const int group = tid >> 5, l32 = tid & 31;
    uint4 starts = make_uint4(0, 0, 0, 0);
    uint32_t group_between = 0;
    if (group < r.chunks) {
        starts = *(const uint4 *)(before + group * kDivBins + 8 * l32);
        group_between = counts[group].between;
    }
    uint32_t key[QPT][4];
#pragma unroll
    for (int i = 0; i < QPT; ++i) split_sel_keys(r, (chunk * QPT + i) * kSplitSelChunk + 4 * tid, key[i]);
    uint32_t sum[8] = {starts.x & 0xffffu, starts.x >> 16, starts.y & 0xffffu, starts.y >> 16,
                       starts.z & 0xffffu, starts.z >> 16, starts.w & 0xffffu, starts.w >> 16};
    for (int c = group + kDivGroups; c < r.chunks; c += kDivGroups) {
        const uint4 t = *(const uint4 *)(before + c * kDivBins + 8 * l32);
        sum[0] += t.x & 0xffffu;  sum[1] += t.x >> 16;  sum[2] += t.y & 0xffffu;  sum[3] += t.y >> 16;
        sum[4] += t.z & 0xffffu;  sum[5] += t.z >> 16;  sum[6] += t.w & 0xffffu;  sum[7] += t.w >> 16;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) sum[e] += (uint32_t)__shfl_xor((int)sum[e], 32, 64);
    if (lane < 32) {
        *(uint4 *)&bin_part[wave][8 * lane] = make_uint4(sum[0], sum[1], sum[2], sum[3]);
        *(uint4 *)&bin_part[wave][8 * lane + 4] = make_uint4(sum[4], sum[5], sum[6], sum[7]);
    }
    if (tid < kSelFinish) list[tid] = 0;
    if (tid == 0) list_above = list_before = 0;
    __syncthreads();
    if (tid < kDivBins) {
        uint32_t t = 0;
#pragma unroll
        for (int w = 0; w < kSelWaves; ++w) t += bin_part[w][tid];
        bin_sum[tid] = t;
    }
    // the classes over all chunks, and over those before this one; every wave for itself
    uint32_t all[4] = {}, pre[4] = {};
    for (int c0 = 0; c0 < r.chunks; c0 += 64) {
        if (c0 > 0) cls = c0 + lane < r.chunks ? *(const uint2 *)&counts[c0 + lane] : make_uint2(0, 0);
        uint32_t sc[4] = {cls.x & 0xffffu, cls.x >> 16, cls.y & 0xffffu, cls.y >> 16};
        wave_incl_scan_n(sc);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            all[e] += (uint32_t)__builtin_amdgcn_readlane((int)sc[e], 63);
            if (chunk > c0) pre[e] += (uint32_t)__builtin_amdgcn_readlane((int)sc[e], min(chunk - c0, 64) - 1);
        }
    }
    // T; the keys above it in the row, the keys above and at it in the chunks before, but for those counted in `list`
    uint32_t T = 0, above = 0, gt_before = 0, eq_before = 0;
    bool found = true, listed = false;                           // the same in every thread of the row's workgroups
    if (kk <= all[0]) found = false;
    else if (kk <= all[0] + all[1]) { T = hi; above = all[0]; gt_before = pre[0]; eq_before = pre[1]; }
    else if (kk > all[0] + all[1] + all[2]) {
        found = kk <= all[0] + all[1] + all[2] + all[3];
        T = lo;
        above = all[0] + all[1] + all[2];
        gt_before = pre[0] + pre[1] + pre[2];
        eq_before = pre[3];
    } else {
        __syncthreads();
        // the bin: of the keys between the edges, all[2], those in it and in higher ones reach the rank, those in higher ones do not
        const uint4 t = *(const uint4 *)&bin_sum[4 * lane];
        const uint32_t next = (uint32_t)__shfl_down((int)t.x, 1, 64), s[5] = {t.x, t.y, t.z, t.w, lane == 63 ? all[2] : next};
        const uint32_t want = kk - all[0] - all[1];
        uint32_t bin = 0, over = 0, upto = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint64_t hit = __ballot(all[2] - s[e + 1] < want && want <= all[2] - s[e]);
            if (hit) {
                const int l = __builtin_amdgcn_readfirstlane(__ffsll((unsigned long long)hit) - 1);
                bin = (uint32_t)(4 * l + e);
                over = all[2] - (uint32_t)__builtin_amdgcn_readlane((int)s[e + 1], l);
                upto = all[2] - (uint32_t)__builtin_amdgcn_readlane((int)s[e], l);
            }
        }
        const bool by_value = div_by_value(bin, (int)binning.y);
        const uint32_t low = binning.x + (bin << binning.y);
        above = all[0] + all[1] + over;
        // AHEAD keys of a chunk's part of the bin, on from number x < n, requested together (the workspace goes on behind the last list)
        constexpr int AHEAD = QPT > 2 ? 4 : 8;
        typedef uint16_t Ahead __attribute__((ext_vector_type(AHEAD), aligned(2)));
        const auto keys_at = [&](const uint16_t *src, int c, uint32_t x, uint32_t n, uint32_t (&k)[AHEAD]) __attribute__((always_inline)) {
            const Ahead at = *(const Ahead *)(src + x);
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) k[u] = by_value ? low + at[u] : order_key(r.cand[c * (kSplitSelChunk * QPT) + (x + u < n ? at[u] : 0)]);
        };
        if (__builtin_expect(upto - over <= (uint32_t)kDivListMax, 1)) {
            // its keys from all chunks, in the order of the chunks, a half wave per chunk and kDivGroups of them at a time
            uint32_t total = 0, own_at = 0, higher = 0;              // `higher`: keys of the chunks before in higher bins
            for (int c0 = 0; c0 < r.chunks; c0 += kDivGroups) {
                const int c = c0 + group;
                uint32_t b0 = 0, n = 0;
                if (c0 > 0) {
                    starts = make_uint4(0, 0, 0, 0);
                    group_between = 0;
                    if (c < r.chunks) {
                        starts = *(const uint4 *)(before + c * kDivBins + 8 * l32);
                        group_between = counts[c].between;
                    }
                }
                const auto start_of = [&](uint32_t x) {
                    const uint32_t pair = (x & 7u) < 2 ? starts.x : (x & 7u) < 4 ? starts.y : (x & 7u) < 6 ? starts.z : starts.w;
                    return (uint32_t)__shfl((int)(x & 1u ? pair >> 16 : pair & 0xffffu), (int)(x >> 3), 32);
                };
                b0 = start_of(bin);
                const uint32_t b1 = bin + 1 < kDivBins ? start_of(bin + 1) : group_between;
                n = b1 - b0;
                const uint16_t *src = p.list + (r.row * p.n_units + c * QPT) * kSplitSelChunk + b0;
                const auto key_at = [&](uint32_t x) {
                    return by_value ? low + src[x] : order_key(r.cand[c * (kSplitSelChunk * QPT) + src[x]]);
                };
                const uint32_t first = l32 < (int)n ? key_at(l32) : 0u;
                if (c0 > 0) __syncthreads();                         // the last round's reads are done
                if (l32 == 0) bin_own[group] = make_uint2(n, group_between - b1);
                __syncthreads();
                const uint2 mine = lane < kDivGroups ? bin_own[lane] : make_uint2(0u, 0u);
                uint32_t sc[2] = {mine.x, mine.y};
                wave_incl_scan_n(sc);
                if (chunk > c0) {
                    const int l = min(chunk - c0, kDivGroups) - 1;
                    own_at = total + (uint32_t)__builtin_amdgcn_readlane((int)sc[0], l);
                    higher += (uint32_t)__builtin_amdgcn_readlane((int)sc[1], l);
                }
                const uint32_t to = total + (uint32_t)__shfl((int)sc[0], group, 64) - n;
                if (l32 < (int)n) list[to + l32] = first;
                if (__builtin_expect(__any(n > 32), 0)) {
                    for (uint32_t x = l32 + 32; x < min(n, 128u); x += 32) list[to + x] = key_at(x);
                    for (uint32_t x = 128 + AHEAD * l32; x < n; x += 32 * AHEAD) {
                        uint32_t k[AHEAD];
                        keys_at(src, c, x, n, k);
#pragma unroll
                        for (int u = 0; u < AHEAD; ++u)
                            if (x + u < n) list[to + x + u] = k[u];
                    }
                }
                total += (uint32_t)__builtin_amdgcn_readlane((int)sc[0], 63);
            }
            __syncthreads();
            T = list_key_of_rank(list, (int)total, want - over, tid, lane);
            uint32_t sc[2] = {0u, 0u};                               // of the bin: keys above T in the row; above it | at it << 16 before this chunk
            for (int x = tid; x < (int)total; x += kSelThreads) {
                const uint32_t k = list[x];
                sc[0] += k > T ? 1u : 0u;
                sc[1] += x < (int)own_at ? (k > T ? 1u : 0u) + (k == T ? 0x10000u : 0u) : 0u;
            }
            if (wave * 64 < (int)total) {
                wave_incl_scan_n(sc);
                if (lane == 63) {
                    atomicAdd(&list_above, sc[0]);
                    atomicAdd(&list_before, sc[1]);
                }
            }
            listed = true;
            gt_before = pre[0] + pre[1] + higher;
        } else {
            // Too many for LDS: most often they are one value, else the rank is found by digits, the keys read where they are.
            // (8 rows of 131072 of seven values, k = half: 20.9 us, by a search of the row in every workgroup 82.8; one of
            // 500000, a millionth apart: 39 against 730.  The code beside the path above costs that 0.2 us of 14.)
            const auto bin_keys = [&](auto &&f) __attribute__((always_inline)) {
                for (int c0 = 0; c0 < r.chunks; c0 += kDivGroups) {
                    const int c = c0 + group;
                    uint32_t b0 = 0, n = 0;
                    if (c < r.chunks) {
                        b0 = before[c * kDivBins + bin];
                        n = (bin + 1 < kDivBins ? (uint32_t)before[c * kDivBins + bin + 1] : (uint32_t)counts[c].between) - b0;
                    }
                    const uint16_t *src = p.list + (r.row * p.n_units + c * QPT) * kSplitSelChunk + b0;
                    for (uint32_t x = AHEAD * l32; __any(x < n); x += 32 * AHEAD) {
                        uint32_t k[AHEAD] = {};
                        if (x < n) keys_at(src, c, x, n, k);
#pragma unroll
                        for (int u = 0; u < AHEAD; ++u) f(k[u], x + u < n, c < chunk);
                    }
                }
            };
            if (tid == 0) heavy = make_uint2(0xffffffffu, 0u);
            if (tid < 3) row_count[tid] = 0;
            __syncthreads();
            uint32_t mn = 0xffffffffu, mx = 0;
            bin_keys([&](uint32_t k, bool has, bool) { mn = min(mn, has ? k : 0xffffffffu); mx = max(mx, has ? k : 0u); });
            wave_min_max(mn, mx);
            if (lane == 63) { atomicMin(&heavy.x, mn); atomicMax(&heavy.y, mx); }
            // what the chunks before hold of the bin and of higher ones, every wave for itself
            uint32_t own_at = 0;
            gt_before = pre[0] + pre[1];
            for (int c = lane; c - lane < chunk; c += 64) {
                uint32_t sc[2] = {0u, 0u};
                if (c < chunk) {
                    const uint32_t all_c = counts[c].between, b1 = bin + 1 < kDivBins ? before[c * kDivBins + bin + 1] : all_c;
                    sc[0] = b1 - before[c * kDivBins + bin];
                    sc[1] = all_c - b1;
                }
                wave_incl_scan_n(sc);
                own_at += (uint32_t)__builtin_amdgcn_readlane((int)sc[0], 63);
                gt_before += (uint32_t)__builtin_amdgcn_readlane((int)sc[1], 63);
            }
            __syncthreads();
            T = heavy.x;
            eq_before = own_at;
            if (heavy.x != heavy.y) {                            // the same in every thread
                T = any_key_of_rank([&](auto &&f) { bin_keys([&](uint32_t k, bool has, bool) { f(k, has); }); }, want - over, tid, lane, wave);
                uint32_t sc[3] = {0u, 0u, 0u};                   // of the bin: keys above T in the row, above it and at it before this chunk
                bin_keys([&](uint32_t k, bool has, bool earlier) {
                    sc[0] += has && k > T ? 1u : 0u;
                    sc[1] += has && earlier && k > T ? 1u : 0u;
                    sc[2] += has && earlier && k == T ? 1u : 0u;
                });
                wave_incl_scan_n(sc);
                if (lane == 63)
#pragma unroll
                    for (int e = 0; e < 3; ++e) atomicAdd(&row_count[e], sc[e]);
                __syncthreads();
                above += row_count[0];
                gt_before += row_count[1];
                eq_before = row_count[2];
            }
#pragma unroll
            for (int i = 0; i < QPT; ++i) split_sel_keys(r, (chunk * QPT + i) * kSplitSelChunk + 4 * tid, key[i]);     // (not held through all that)
        }
    }
    if (__builtin_expect(!found, 0)) {                           // the same in every thread
        __syncthreads();
        T = any_key_of_rank([&](auto &&f) {
#pragma unroll 4
            for (int x0 = 0; x0 < r.n; x0 += kSelThreads) f(x0 + tid < r.n ? order_key(r.cand[x0 + tid]) : 0u, x0 + tid < r.n);
        }, kk, tid, lane, wave);
        if (tid < 3) row_count[tid] = 0;
        __syncthreads();
        uint32_t c[3] = {};
        const int own0 = chunk * kSplitSelChunk * QPT;
        for (int x = tid; x < r.n; x += kSelThreads) {
            const uint32_t k = order_key(r.cand[x]);
            c[0] += k > T ? 1u : 0u;
            c[1] += k > T && x < own0 ? 1u : 0u;
            c[2] += k == T && x < own0 ? 1u : 0u;
        }
        wave_incl_scan_n(c);
        if (lane == 63)
#pragma unroll
            for (int e = 0; e < 3; ++e) atomicAdd(&row_count[e], c[e]);
        __syncthreads();
        above = row_count[0];
        gt_before = row_count[1];
        eq_before = row_count[2];
    }
    // ---- the chunk's own keys > T | == T << 16, in index order (step, wave, lane, key)
    uint32_t incl[QPT], own[QPT];
#pragma unroll
    for (int i = 0; i < QPT; ++i) {
        own[i] = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {                            // empty slots hold key 0, below every score
            own[i] += key[i][j] > T ? 1u : 0u;
            own[i] += key[i][j] == T ? 0x10000u : 0u;
        }
        incl[i] = own[i];
    }
    wave_incl_scan_n(incl);
#pragma unroll
    for (int i = 0; i < QPT; ++i)
        if (lane == 63) step_own[i * kSelWaves + wave] = incl[i];
    __syncthreads();
    if (listed) {
        above += list_above;
        gt_before += list_before & 0xffffu;
        eq_before = list_before >> 16;
    }
    const int krem = (int)(kk - above);                          // ties at T to keep (>= 1), lowest index first
    uint32_t steps[1] = {lane < kSelWaves * QPT ? step_own[lane] : 0u};
    const uint32_t step_mine = steps[0];
    wave_incl_scan_n(steps);
#pragma unroll
    for (int i = 0; i < QPT; ++i) {
        const uint32_t first = (uint32_t)__builtin_amdgcn_readlane((int)(steps[0] - step_mine), i * kSelWaves + wave) + incl[i] - own[i];
        int gt = (int)(gt_before + (first & 0xffffu)), eq = (int)(eq_before + (first >> 16));
        const int x0 = (chunk * QPT + i) * kSplitSelChunk + 4 * tid;
        uint32_t mbytes = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool is_gt = key[i][j] > T, is_eq = key[i][j] == T;
            const bool sel = is_gt || (is_eq && eq < krem);
            if (sel) out[gt + min(eq, krem)] = r.c0 + x0 + j;
            gt += is_gt ? 1 : 0;
            eq += is_eq ? 1 : 0;
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
}

}  // namespace pdd
