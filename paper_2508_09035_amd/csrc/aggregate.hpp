// Aggregation of token-importance scores over attention layers and heads
// (paper Section 4.4: several layers take part in the selection, their weight
// distributions differ in magnitude, and the choice of layers is left open).
//
//   out[h, j] (+)= sum_l w_l * scores[l, h, j]              (per head row)
//   out[0, j] (+)= sum_l w_l * sum_h scores[l, h, j]        (heads reduced)
//
// Streaming, HBM bound: every score is read once, every output written once
// (read first when accumulating).  A wave owns 64 * VEC consecutive tokens of an
// output row; where the rows alone do not give the chip enough waves, several waves
// of a workgroup take the same tokens, each with a run of consecutive layers, and
// their sums are added in the order of the layers through LDS.  fp32, a fixed
// order for a given shape: deterministic.  The loads of a wave are contiguous and
// only as aligned as a score is (gfx950 loads 16 bytes from any 4-byte address),
// so every row length takes the wide form.  A workgroup has four waves at least.
// 32 layers x 8 heads x 32768 tokens into one row (34 MB, held by the last-level cache):
// 48 -> 6.0 us (one thread per four tokens walked all 256 scores, 32 workgroups);
// 32 x 8 x 27090 per head 13.1 -> 6.1 us (7.7 and 7.6 where every call has other scores).  From memory: 1 layer x 8 x 1048576 12.8 us (5.3 TB/s; 22.6 in
// workgroups of one wave), 32 x 8 x 1048576 184 per head, 161 into one row (5.8 and 6.7 TB/s).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

namespace pdd {

struct AggParams {
    const float *scores;     // [n_layers, n_heads, total_k], layer stride in elements
    const float *weights;    // [n_layers] or nullptr (= 1)
    float *out;              // [n_heads or 1, total_k]
    int64_t layer_stride;
    int32_t n_layers, n_heads, total_k, reduce_heads, accumulate;
    int32_t share_log2;      // 2^share_log2 waves share the layers of the same tokens
};

constexpr int kAggMaxWaves = 16, kAggMinWaves = 4;

// blockDim.x = 64 * waves, a multiple of 2^share_log2 up to kAggMaxWaves.  AHEAD loads of a wave in flight:
// the order of the additions does not depend on it.
template <int VEC, int AHEAD>
__global__ __launch_bounds__(64 * kAggMaxWaves) void aggregate_scores_kernel(const AggParams p)
{
    typedef float vec __attribute__((ext_vector_type(VEC)));
    typedef float vec_any __attribute__((ext_vector_type(VEC), aligned(4)));
    extern __shared__ __attribute__((aligned(16))) uint8_t agg_smem[];      // sums of the waves, where they share
    vec *const part_sum = (vec *)agg_smem;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int share = 1 << p.share_log2, part = wave & (share - 1);          // waves on these tokens, and which of them
    const int64_t group = (int64_t)blockIdx.x * (blockDim.x >> (6 + p.share_log2)) + (wave >> p.share_log2);
    const int64_t j0 = (group * 64 + lane) * VEC;
    const int row = blockIdx.y;                       // output row
    const int h_lo = p.reduce_heads ? 0 : row, n_h = p.reduce_heads ? p.n_heads : 1;
    const int l_lo = (int)((int64_t)p.n_layers * part >> p.share_log2), l_hi = (int)((int64_t)p.n_layers * (part + 1) >> p.share_log2);
    float *op = p.out + (int64_t)row * p.total_k;
    // A lane past the row's end reads the last token again, so that no load hangs on a branch; the waves inside
    // the row, almost all of them, load VEC tokens at once.
    const bool whole = (group + 1) * 64 * VEC <= p.total_k;           // of the wave

    // AHEAD rows in flight: layers, or the heads of a layer, which are added up first.
    auto sum = [&](auto whole_c) {
        auto load = [&](const float *sp) {
            vec t;
            if constexpr (decltype(whole_c)::value) t = __builtin_nontemporal_load((const vec_any *)(sp + j0));
            else
#pragma unroll
                for (int c = 0; c < VEC; ++c) t[c] = sp[min(j0 + c, (int64_t)p.total_k - 1)];
            return t;
        };
        // calls add(i, row i), the rows `stride` apart; several loads in flight in the last, incomplete batch too
        auto each = [&](const float *sp, int n, int64_t stride, auto &&add) {
            int i0 = 0;
            for (; i0 + AHEAD <= n; i0 += AHEAD, sp += AHEAD * stride) {
                vec t[AHEAD];
#pragma unroll
                for (int i = 0; i < AHEAD; ++i) t[i] = load(sp + i * stride);
#pragma unroll
                for (int i = 0; i < AHEAD; ++i) add(i0 + i, t[i]);
            }
            if constexpr (AHEAD > 1) {
                const int m = n - i0;
                vec t[AHEAD - 1];
#pragma unroll
                for (int i = 0; i < AHEAD - 1; ++i)
                    if (i < m) t[i] = load(sp + i * stride);
#pragma unroll
                for (int i = 0; i < AHEAD - 1; ++i)
                    if (i < m) add(i0 + i, t[i]);
            }
        };
        vec acc = 0.f;
        if (p.accumulate && part == 0) acc = load(op);
        const float *sp = p.scores + (int64_t)l_lo * p.layer_stride + (int64_t)h_lo * p.total_k;
        auto weighted = [&](int l, const vec &t) { acc += (p.weights ? p.weights[l] : 1.f) * t; };
        if (n_h == 1) {
            each(sp, l_hi - l_lo, p.layer_stride, [&](int i, const vec &t) { weighted(l_lo + i, t); });
        } else {
            for (int l = l_lo; l < l_hi; ++l, sp += p.layer_stride) {
                vec heads = 0.f;
                each(sp, n_h, p.total_k, [&](int, const vec &t) { heads += t; });
                weighted(l, heads);
            }
        }
        return acc;
    };
    vec acc = whole ? sum(std::true_type{}) : sum(std::false_type{});
    if (share > 1) {
        if (part > 0) part_sum[64 * wave + lane] = acc;
        __syncthreads();
        if (part > 0) return;
        for (int w = 1; w < share; ++w) acc += part_sum[64 * (wave + w) + lane];
    }
    if (whole) *(vec_any *)(op + j0) = acc;
    else
#pragma unroll
        for (int c = 0; c < VEC; ++c)
            if (j0 + c < p.total_k) op[j0 + c] = acc[c];
}

}  // namespace pdd
