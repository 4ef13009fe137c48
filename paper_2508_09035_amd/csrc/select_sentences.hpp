// Sentence-level selection (paper Section 3.2, "Prompt Refiner": the KV cache
// entries of one sentence are combined and treated as a whole, so that
// selecting KV cache entries means selecting sentences; Section 1: sentence-
// level selection keeps the refined prompt semantically coherent).
//
// Per (sequence, head row): sentences are contiguous token ranges that tile the
// content part [cand_begin, sent_end[last]).  A sentence's score is the sum or
// the mean of its tokens' scores; sentences are ranked by (score descending,
// index ascending) and the longest prefix of that ranking whose token count
// fits the budget is kept.  Outputs: keep flag per sentence, 0/1 mask per
// token, number of kept tokens.
//
// One 1024-thread workgroup per row; a thread owns up to eight consecutive
// sentences, whose bounds, scores and lengths stay in registers.
//   * The row's scores come through LDS in pieces of up to 32768 (whole-row loads,
//     the next piece requested while one is summed); a sentence is summed by its
//     owner in token order, one fp32 chain.  (Read by the owner straight from
//     memory, one score after the other, the longest sentence alone cost 60 us.)
//   * No ranks are formed: the kept prefix of the ranking is every sentence above a
//     threshold key and the first of those that tie with it, and the threshold
//     is found like the k-th score of a short token row, with the lengths as weights:
//     a histogram over the row's range, probes (see next_probe) where its bin holds
//     more than 64 sentences.
//   * The token mask: kept sentences flip a bit at their start and at their end,
//     and a prefix parity over the bits gives the mask 32768 tokens at a time.
// Bound by the latency of its steps on the one compute unit the row runs on:
// 1 row of 32768 tokens in 1362 sentences 149 -> 15.5 us (serial reads, S^2 ranks and
// a binary search per token before; 21 with the scores in two pieces and five to seven probes
// instead of the histogram), a third of it the sums, whose LDS reads of 64 sentences
// at a time conflict.
#pragma once
#include "select_topk.hpp"
#include <type_traits>

namespace pdd {

enum { kSentSum = 0, kSentMean = 1 };
constexpr int kSentMax = 8192;    // sentences per sequence

struct SentParams {
    const float *scores;
    const int32_t *cu_k, *cu_sent, *sent_end, *cand_b, *budget;
    uint8_t *sent_keep, *mask;
    int32_t *kept_tokens;
    float *sent_scores;
    int32_t n_heads, B, total_k, total_sent, s_cap, mode;
    int32_t seg;              // scores in LDS at a time, a multiple of 4 * kSelThreads up to kSentSeg
};

constexpr int kSentOwn = kSentMax / kSelThreads;     // sentences per thread at most
constexpr int kSentSeg = 32 * kSelThreads;            // scores in LDS at a time, at most
constexpr int kSentChunk = 32 * kSelThreads;          // mask tokens at a time: one 32-bit word per thread
// a probe either cuts the tokens inside the bracket to a quarter (at most 16 times), or is
// followed by one that halves the bracket (at most 32 pairs)
constexpr int kSentMaxProbes = 96;
constexpr int kSentFinish = 64;                       // sentences left in the bracket that are compared directly

typedef float sent_f32x4 __attribute__((ext_vector_type(4), aligned(4)));    // four scores at any score's address

// inclusive prefix maximum of values >= 0 over the 64 lanes of a wave (see wave_incl_scan)
__device__ __forceinline__ uint32_t wave_incl_max(uint32_t x)
{
    x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, true));
    x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, true));
    x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, true));
    x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, true));
    x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false));
    x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false));
    return x;
}

__global__ __launch_bounds__(kSelThreads) void select_sentences_kernel(const SentParams p)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t sent_smem[];    // p.seg scores, later mask words
    float *const stage = (float *)sent_smem;
    uint32_t *const bits = (uint32_t *)sent_smem;
    __shared__ int32_t sh_end[kSelWaves];
    __shared__ uint32_t sh_tie[kSelWaves];
    __shared__ uint32_t wave_min[kSelWaves], wave_max[kSelWaves], wave_par[kSelWaves];
    __shared__ unsigned long long probe_tot[kSentMaxProbes];       // tokens | sentences << 32 at or above a probe
    __shared__ __attribute__((aligned(16))) unsigned long long hist[kSelBins];     // tokens | sentences << 32 of a bin
    __shared__ __attribute__((aligned(16))) uint2 fin[kSentFinish];              // key, length
    __shared__ struct { uint32_t bin, tokens, sentences, above, n_above; } place;
    __shared__ uint32_t fin_count, fin_T, fin_above, sh_kept;
    __shared__ uint2 range[kSentMaxProbes];                       // of probe number p, see narrow_bracket

    const int b = blockIdx.x, g = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int ks = min(max(p.cu_k[b], 0), p.total_k);
    const int ke = min(max(p.cu_k[b + 1], ks), p.total_k);
    const int nk = ke - ks;
    const int s0 = min(max(p.cu_sent[b], 0), p.total_sent);
    const int s1 = min(max(p.cu_sent[b + 1], s0), p.total_sent);
    const int S = min(s1 - s0, p.s_cap);
    const int c0 = min(max(p.cand_b ? p.cand_b[b] : 0, 0), nk);
    const uint32_t budget = (uint32_t)max(p.budget[b], 0);
    const float *seq = p.scores + (int64_t)g * p.total_k + ks;
    uint8_t *mrow = p.mask ? p.mask + (int64_t)g * p.total_k + ks : nullptr;

    if (tid < kSentMaxProbes) {
        probe_tot[tid] = 0;
        range[tid] = make_uint2(0xffffffffu, 0u);
    }
    hist[tid] = 0;
    if (tid < kSentFinish) fin[tid] = make_uint2(0, 0);
    if (tid == 0) { fin_count = 0; sh_kept = 0; }

    // ---- sentence bounds: ends forced into [c0, nk] and non-decreasing (running maximum)
    const int ch = (S + kSelThreads - 1) / kSelThreads;          // sentences per thread, <= kSentOwn
    const int s_lo = tid * ch;
    int end[kSentOwn];
    int mx = c0;
#pragma unroll
    for (int i = 0; i < kSentOwn; ++i) {
        if (i < ch && s_lo + i < S) mx = max(mx, min(max(p.sent_end[s0 + s_lo + i], c0), nk));
        end[i] = mx;
    }
    const int mx_incl = (int)wave_incl_max((uint32_t)mx);
    if (lane == 63) sh_end[wave] = mx_incl;
    __syncthreads();
    int content_end = c0, begin = c0;                             // running maximum of all threads, of those before this one
#pragma unroll
    for (int w = 0; w < kSelWaves; ++w) {
        content_end = max(content_end, sh_end[w]);
        begin = w < wave ? max(begin, sh_end[w]) : begin;
    }
    {
        const int up = __shfl_up(mx_incl, 1, 64);
        begin = lane > 0 ? max(begin, up) : begin;
    }
#pragma unroll
    for (int i = 0; i < kSentOwn; ++i) end[i] = max(end[i], begin);

    // ---- sentence scores.  Sentence i covers [start of i, end[i]), start = end of the one before
    float acc[kSentOwn];
#pragma unroll
    for (int i = 0; i < kSentOwn; ++i) acc[i] = 0.f;
    constexpr int QUADS = kSentSeg / (4 * kSelThreads);
    sent_f32x4 pre[QUADS];
    auto request = [&](int at) {
#pragma unroll
        for (int q = 0; q < QUADS; ++q) {
            const int o = 4 * (q * kSelThreads + tid), x = at + o;
            if (o < p.seg) {
                if (x + 4 <= content_end) pre[q] = *(const sent_f32x4 *)(seq + x);
                else
#pragma unroll
                    for (int j = 0; j < 4; ++j) pre[q][j] = x + j < content_end ? seq[x + j] : 0.f;
            }
        }
    };
    request(c0);
    for (int seg0 = c0; seg0 < content_end; seg0 += p.seg) {
#pragma unroll
        for (int q = 0; q < QUADS; ++q) {
            const int o = 4 * (q * kSelThreads + tid);
            if (o < p.seg) *(float4 *)(stage + o) = make_float4(pre[q][0], pre[q][1], pre[q][2], pre[q][3]);
        }
        __syncthreads();
        if (seg0 + p.seg < content_end) request(seg0 + p.seg);
#pragma unroll
        for (int i = 0; i < kSentOwn; ++i) {
            if (i < ch) {
                const int x = max(i == 0 ? begin : end[i - 1], seg0) - seg0;
                const int z = min(end[i] - seg0, p.seg);
                float a = acc[i];
                // eight scores from two quads at a time, added in token order; in the first and the last
                // eight, what lies outside the sentence counts as zero (the masks are what a step costs
                // most, and the reads stay inside the stage: p.seg is a multiple of 8)
                auto eight = [&](int y, auto masked) {
                    const float4 q0 = *(const float4 *)(stage + y), q1 = *(const float4 *)(stage + y + 4);
                    const float v[8] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w};
#pragma unroll
                    for (int j = 0; j < 8; ++j)
                        a += !decltype(masked)::value || (y + j >= x && y + j < z) ? v[j] : 0.f;
                };
                if (x < z) {
                    int y = x & ~7;
                    eight(y, std::true_type{});
                    for (y += 8; y + 8 <= z; y += 8) eight(y, std::false_type{});
                    if (y < z) eight(y, std::true_type{});
                }
                acc[i] = a;
            }
        }
        __syncthreads();
    }
    // slots without a sentence: key 0, length 0
    uint32_t key[kSentOwn], len[kSentOwn];
    uint32_t kmin = 0xffffffffu, kmax = 0;
#pragma unroll
    for (int i = 0; i < kSentOwn; ++i) {
        key[i] = len[i] = 0;
        if (i < ch && s_lo + i < S) {
            const int n = end[i] - (i == 0 ? begin : end[i - 1]);
            const float sc = (p.mode == kSentMean) ? acc[i] / (float)max(n, 1) : acc[i];
            key[i] = order_key(sc);
            len[i] = (uint32_t)n;
            kmin = min(kmin, key[i]);
            kmax = max(kmax, key[i]);
            if (p.sent_scores) p.sent_scores[(int64_t)g * p.total_sent + s0 + s_lo + i] = sc;
        }
    }

    // ---- threshold: the largest T whose sentences (key >= T) hold more tokens than the budget.  The
    // ranking then keeps every sentence above T and, in index order, those at T that still fit.
    const uint32_t total = (uint32_t)(content_end - c0);
    uint32_t T = 0, above = 0;                                   // above = tokens of the sentences > T
    const bool all = total <= budget;                            // the same in every thread
    if (!all) {
        wave_min_max(kmin, kmax);
        if (lane == 63) { wave_min[wave] = kmin; wave_max[wave] = kmax; }
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kSelWaves; ++w) {
            kmin = w == 0 ? wave_min[0] : min(kmin, wave_min[w]);
            kmax = w == 0 ? wave_max[0] : max(kmax, wave_max[w]);
        }
        const uint32_t need = budget + 1u;
        uint32_t lo = kmin, hi = kmax, w_lo = total, n_lo = (uint32_t)S, n_above = 0;
        bool interp = true;
        if (lo < hi && S > kSentFinish) {
            // the bin of the row's range that holds T
            const int shift = max(32 - __builtin_clz(hi - lo) - 10, 0);       // kSelBins = 2^10
#pragma unroll
            for (int i = 0; i < kSentOwn; ++i)
                if (i < ch && s_lo + i < S) atomicAdd(&hist[(key[i] - lo) >> shift], 1ull << 32 | len[i]);
            __syncthreads();
            if (wave == 0) {
                unsigned long long bin[16], sum = 0;              // lane: 16 consecutive bins
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    bin[e] = hist[16 * lane + e];
                    sum += bin[e];
                }
                uint32_t sc[2] = {(uint32_t)sum, (uint32_t)(sum >> 32)};
                wave_incl_scan_n(sc);
                uint32_t w = total - sc[0], n = (uint32_t)S - sc[1];
#pragma unroll
                for (int e = 15; e >= 0; --e) {
                    const uint32_t wb = (uint32_t)bin[e], nb = (uint32_t)(bin[e] >> 32);
                    if (w < need && need <= w + wb) place = {(uint32_t)(16 * lane + e), wb, nb, w, n};
                    w += wb;
                    n += nb;
                }
            }
            __syncthreads();
            const uint32_t first = place.bin << shift;
            hi = lo + min(first + ((1u << shift) - 1u), hi - lo);
            lo += first;
            above = place.above;
            w_lo = above + place.tokens;
            n_above = place.n_above;
            n_lo = n_above + place.sentences;
        }
        for (int probe = 0; lo < hi && n_lo - n_above > (uint32_t)kSentFinish; ++probe) {
            const uint32_t inside = w_lo - above;
            const uint32_t mid = next_probe(lo, hi, inside, need - above, interp);
            uint32_t w = 0, n = 0;
#pragma unroll
            for (int i = 0; i < kSentOwn; ++i) {                  // mid > lo >= kmin: empty slots never count
                w += key[i] >= mid ? len[i] : 0u;
                n += key[i] >= mid ? 1u : 0u;
            }
            uint32_t sc[2] = {w, n};
            wave_incl_scan_n(sc);
            if (lane == 63) atomicAdd(&probe_tot[probe], (unsigned long long)sc[0] | (unsigned long long)sc[1] << 32);
            __syncthreads();
            const unsigned long long t = probe_tot[probe];
            if ((uint32_t)t >= need) { lo = mid; w_lo = (uint32_t)t; n_lo = (uint32_t)(t >> 32); }
            else { hi = mid - 1u; above = (uint32_t)t; n_above = (uint32_t)(t >> 32); }
            const bool halved = !interp;
            interp = halved || 4u * (w_lo - above) <= inside;
            // sentences of one score (2 x 2112 tokens, 845 sentences, most of score 0: 32 -> 10.4 us; 21 by ranks)
            if (__builtin_expect(halved && w_lo - above == inside && lo < hi, 0)) {
                uint32_t mn = 0xffffffffu, mx = 0;
#pragma unroll
                for (int i = 0; i < kSentOwn; ++i) range_of_key(key[i], lo, hi, mn, mx);
                narrow_bracket(&range[probe], mn, mx, lane, lo, hi);
            }
        }
        T = lo;
        if (lo < hi) {
            // at most kSentFinish sentences lie in [lo, hi]
#pragma unroll
            for (int i = 0; i < kSentOwn; ++i)
                if (i < ch && s_lo + i < S && key[i] - lo <= hi - lo) {
                    const uint32_t at = atomicAdd(&fin_count, 1u);
                    fin[at] = make_uint2(key[i], len[i]);
                }
            __syncthreads();
            if (wave == 0) {
                const int m = (int)fin_count;
                const uint32_t mine = fin[lane].x;                // slots past m: key 0, length 0
                uint32_t gt = above, ge = above;
#pragma unroll 4
                for (int j = 0; j < m; j += 2) {
                    const uint4 o = *(const uint4 *)(fin + j);
                    gt += (o.x > mine ? o.y : 0u) + (o.z > mine ? o.w : 0u);
                    ge += (o.x >= mine ? o.y : 0u) + (o.z >= mine ? o.w : 0u);
                }
                if (lane < m && gt < need && ge >= need) { fin_T = mine; fin_above = gt; }   // one key at most
            }
            __syncthreads();
            T = fin_T;
            above = fin_above;
        }
    }

    // ---- keep flags
    uint32_t kept = 0;
    {
        uint32_t tie = 0;
#pragma unroll
        for (int i = 0; i < kSentOwn; ++i) tie += (i < ch && s_lo + i < S && key[i] == T) ? len[i] : 0u;
        const uint32_t tie_incl = wave_incl_scan(tie);
        if (lane == 63) sh_tie[wave] = tie_incl;
        __syncthreads();
        uint32_t run = tie_incl - tie;
#pragma unroll
        for (int w = 0; w < kSelWaves; ++w) run += w < wave ? sh_tie[w] : 0u;
        uint32_t tokens = 0;
#pragma unroll
        for (int i = 0; i < kSentOwn; ++i) {
            if (i < ch && s_lo + i < S) {
                bool k = all || key[i] > T;
                if (!all && key[i] == T) {
                    run += len[i];
                    k = run <= budget - above;
                }
                kept |= k ? 1u << i : 0u;
                tokens += k ? len[i] : 0u;
                if (p.sent_keep) p.sent_keep[(int64_t)g * p.total_sent + s0 + s_lo + i] = k ? 1 : 0;
            }
        }
        if (p.kept_tokens) {
            tokens = wave_incl_scan(tokens);
            if (lane == 63) atomicAdd(&sh_kept, tokens);
            __syncthreads();
            if (tid == 0) p.kept_tokens[(int64_t)g * p.B + b] = (int32_t)sh_kept;
        }
    }

    // ---- token mask
    if (mrow) {
        uint32_t carry = 0;                                       // parity of the flips before the chunk
        const bool dwords = ((uint32_t)(uintptr_t)mrow & 3u) == 0;
        for (int x0 = 0; x0 < nk; x0 += kSentChunk) {
            __syncthreads();
            bits[tid] = 0;
            __syncthreads();
#pragma unroll
            for (int i = 0; i < kSentOwn; ++i) {
                if (kept >> i & 1u) {
                    const uint32_t a = (uint32_t)((i == 0 ? begin : end[i - 1]) - x0), z = (uint32_t)(end[i] - x0);
                    if (a < (uint32_t)kSentChunk) atomicXor(&bits[a >> 5], 1u << (a & 31u));
                    if (z < (uint32_t)kSentChunk) atomicXor(&bits[z >> 5], 1u << (z & 31u));
                }
            }
            __syncthreads();
            uint32_t v = bits[tid];
#pragma unroll
            for (int off = 1; off < 32; off <<= 1) v ^= v << off;
            const uint64_t par = __ballot(v >> 31);
            if (lane == 0) wave_par[wave] = (uint32_t)__popcll(par) & 1u;
            __syncthreads();
            uint32_t odd = carry ^ ((uint32_t)__popcll(par & ((1ull << lane) - 1ull)) & 1u);
#pragma unroll
            for (int w = 0; w < kSelWaves; ++w) {
                odd ^= w < wave ? wave_par[w] : 0u;
                carry ^= wave_par[w];
            }
            bits[tid] = v ^ (0u - odd);
            __syncthreads();
            for (int o = 4 * tid; o < kSentChunk && x0 + o < nk; o += 4 * kSelThreads) {
                const uint32_t nib = bits[o >> 5] >> (o & 31) & 15u;
                const uint32_t v4 = nib * 0x00204081u & 0x01010101u;     // bit j of the nibble to byte j
                uint8_t *mp = mrow + x0 + o;
                if (dwords && x0 + o + 4 <= nk) *(uint32_t *)mp = v4;
                else
                    for (int j = 0; j < 4; ++j)
                        if (x0 + o + j < nk) mp[j] = (uint8_t)(v4 >> (8 * j));
            }
        }
    }
}

}  // namespace pdd
