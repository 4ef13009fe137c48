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
// so every row length takes the wide form.  A workgroup has four waves at least, also
// where they share nothing: the LDS of the sums lets ten workgroups onto a compute unit.
// 32 layers x 8 heads x 32768 tokens into one row (34 MB, held by the last-level cache):
// 48 -> 6.6 us (one thread per four tokens walked all 256 scores, 32 workgroups);
// 32 x 8 x 27090 per head 13.1 -> 8.5 us.  From memory: 1 layer x 8 x 1048576 12.8 us (5.3 TB/s; 22.6 in
// workgroups of one wave), 32 x 8 x 1048576 184 per head, 161 into one row (5.8 and 6.7 TB/s).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

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
    __shared__ vec part_sum[kAggMaxWaves][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int share = 1 << p.share_log2, part = wave & (share - 1);          // waves on these tokens, and which of them
    const int64_t group = (int64_t)blockIdx.x * (blockDim.x >> (6 + p.share_log2)) + (wave >> p.share_log2);
    const int64_t j0 = (group * 64 + lane) * VEC;
    const int row = blockIdx.y;                       // output row
    const int h_lo = p.reduce_heads ? 0 : row, n_h = p.reduce_heads ? p.n_heads : 1;
    const int l_lo = (int)((int64_t)p.n_layers * part >> p.share_log2), l_hi = (int)((int64_t)p.n_layers * (part + 1) >> p.share_log2);
    float *op = p.out + (int64_t)row * p.total_k + j0;
    const int width = (int)min((int64_t)VEC, (int64_t)p.total_k - j0);       // tokens of this lane, <= 0 past the row

    auto load = [&](const float *sp) {
        vec t = 0.f;
        if (width == VEC) t = __builtin_nontemporal_load((const vec_any *)sp);
        else
#pragma unroll
            for (int c = 0; c < VEC; ++c) t[c] = c < width ? sp[c] : 0.f;
        return t;
    };
    vec acc = 0.f;
    if (p.accumulate && part == 0) acc = load(op);
    if (width > 0) {
        const float *sp = p.scores + (int64_t)l_lo * p.layer_stride + (int64_t)h_lo * p.total_k + j0;
        if (n_h == 1) {
            int l = l_lo;
            for (; l + AHEAD <= l_hi; l += AHEAD, sp += AHEAD * p.layer_stride) {
                vec t[AHEAD];
#pragma unroll
                for (int i = 0; i < AHEAD; ++i) t[i] = load(sp + i * p.layer_stride);
#pragma unroll
                for (int i = 0; i < AHEAD; ++i) acc += (p.weights ? p.weights[l + i] : 1.f) * t[i];
            }
            for (; l < l_hi; ++l, sp += p.layer_stride) acc += (p.weights ? p.weights[l] : 1.f) * load(sp);
        } else {
            for (int l = l_lo; l < l_hi; ++l, sp += p.layer_stride) {
                const float *hp = sp;
                vec heads = 0.f;
                int h = 0;
                for (; h + AHEAD <= n_h; h += AHEAD, hp += AHEAD * (int64_t)p.total_k) {
                    vec t[AHEAD];
#pragma unroll
                    for (int i = 0; i < AHEAD; ++i) t[i] = load(hp + i * (int64_t)p.total_k);
#pragma unroll
                    for (int i = 0; i < AHEAD; ++i) heads += t[i];
                }
                for (; h < n_h; ++h, hp += p.total_k) heads += load(hp);
                acc += (p.weights ? p.weights[l] : 1.f) * heads;
            }
        }
    }
    if (share > 1) {
        if (part > 0) part_sum[wave][lane] = acc;
        __syncthreads();
        if (part > 0) return;
        for (int w = 1; w < share; ++w) acc += part_sum[wave + w][lane];
    }
    if (width == VEC) *(vec_any *)op = acc;
    else
#pragma unroll
        for (int c = 0; c < VEC; ++c)
            if (c < width) op[c] = acc[c];
}

}  // namespace pdd
