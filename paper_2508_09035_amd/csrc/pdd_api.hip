// C ABI of libpdd (declared in include/pdd.h): host-side argument validation
// and kernel launches.  No device memory is allocated or freed here and no
// device data is read from the host.
#include "../../include/pdd.h"

#include <hip/hip_runtime.h>
#include <atomic>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>

#include "attn_fwd.hpp"
#include "attn_wide.hpp"
#include "attn_rows.hpp"
#include "importance.hpp"
#include "select_topk.hpp"
#include "select_split.hpp"
#include "pack_mask.hpp"
#include "select_sentences.hpp"
#include "aggregate.hpp"
#include <mutex>

// Scratch of the allocation-free entry point: one copy per GPU the library runs on, held until
// the process ends.  In host code this name is only a handle for hipGetSymbolAddress; the address
// that kernels and memory calls use is the one that call returns for the current device.
#define PDD_STATIC_SCRATCH_BYTES (16u << 20)
static __device__ __align__(256) unsigned char scratch[PDD_STATIC_SCRATCH_BYTES];

namespace {

thread_local char g_err[512] = "";
std::atomic<int> g_attn_waves{0};  // 0 = choose per problem
std::atomic<int> g_imp_keys{0};    // keys per importance workgroup, 0 = choose per problem

pdd_status fail(pdd_status st, const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof g_err, fmt, ap);
    va_end(ap);
    return st;
}

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

pdd_status check_cu_host(const char *what, const int32_t *cu, int B, int total, int max_len)
{
    if (!cu) return PDD_OK;
    if (cu[0] != 0) return fail(PDD_ERR_INVALID_ARG, "%s[0] must be 0", what);
    for (int b = 0; b < B; ++b) {
        if (cu[b + 1] < cu[b]) return fail(PDD_ERR_INVALID_ARG, "%s is not non-decreasing at %d", what, b);
        if (cu[b + 1] - cu[b] > max_len)
            return fail(PDD_ERR_INVALID_ARG, "%s: sequence %d longer than max_seqlen (%d > %d)", what, b,
                        cu[b + 1] - cu[b], max_len);
    }
    if (cu[B] != total) return fail(PDD_ERR_INVALID_ARG, "%s[B] = %d differs from the total %d", what, cu[B], total);
    return PDD_OK;
}

enum Mode { MODE_PREFILL, MODE_CHUNKED, MODE_IMPORTANCE };

pdd_status check_desc(const pdd_attn_desc *d, Mode mode)
{
    if (!d) return fail(PDD_ERR_INVALID_ARG, "desc is NULL");
    if (d->batch < 1) return fail(PDD_ERR_INVALID_ARG, "batch must be >= 1");
    if (d->n_q_heads < 1 || d->n_kv_heads < 1) return fail(PDD_ERR_INVALID_ARG, "head counts must be >= 1");
    if (d->n_q_heads % d->n_kv_heads) return fail(PDD_ERR_INVALID_ARG, "n_q_heads %% n_kv_heads != 0");
    if (d->head_dim != 64 && d->head_dim != 128)
        return fail(PDD_ERR_UNSUPPORTED, "head_dim %d not supported (64 or 128)", d->head_dim);
    if (d->total_q < 0 || d->total_k < 0) return fail(PDD_ERR_INVALID_ARG, "negative totals");
    if (d->max_seqlen_q < 0 || d->max_seqlen_k < 0 || d->max_seqlen_q > d->total_q || d->max_seqlen_k > d->total_k)
        return fail(PDD_ERR_INVALID_ARG, "max_seqlen out of range");
    if (d->total_q > 0 && d->max_seqlen_q < 1) return fail(PDD_ERR_INVALID_ARG, "max_seqlen_q must be >= 1");
    if (d->total_k > 0 && d->max_seqlen_k < 1) return fail(PDD_ERR_INVALID_ARG, "max_seqlen_k must be >= 1");
    if (!d->cu_seqlens_q || !d->cu_seqlens_k) return fail(PDD_ERR_INVALID_ARG, "cu_seqlens pointers are NULL");
    if (mode == MODE_PREFILL && d->total_q != d->total_k)
        return fail(PDD_ERR_INVALID_ARG, "prefill needs total_q == total_k (use the chunked entry point)");
    if (d->total_k < d->total_q) return fail(PDD_ERR_INVALID_ARG, "total_k < total_q");
    const int64_t hd = d->head_dim;
    const int64_t st[8] = {d->q_stride_tok, d->q_stride_head, d->k_stride_tok, d->k_stride_head,
                           d->v_stride_tok, d->v_stride_head, d->o_stride_tok, d->o_stride_head};
    const int n_st = mode == MODE_IMPORTANCE ? 4 : 8;
    for (int i = 0; i < n_st; ++i) {
        if (st[i] < hd) return fail(PDD_ERR_INVALID_ARG, "stride %d smaller than head_dim", i);
        if (st[i] % 8) return fail(PDD_ERR_INVALID_ARG, "stride %d is not a multiple of 8 elements (16 bytes)", i);
    }
    if (mode == MODE_PREFILL && d->window < 0) return fail(PDD_ERR_INVALID_ARG, "window must be >= 0");
    if (mode == MODE_IMPORTANCE && d->window == 0) return fail(PDD_ERR_INVALID_ARG, "window must not be 0");
    pdd_status s = check_cu_host("cu_seqlens_q_host", d->cu_seqlens_q_host, d->batch, d->total_q, d->max_seqlen_q);
    if (s) return s;
    s = check_cu_host("cu_seqlens_k_host", d->cu_seqlens_k_host, d->batch, d->total_k, d->max_seqlen_k);
    if (s) return s;
    if (d->cu_seqlens_q_host && d->cu_seqlens_k_host) {
        for (int b = 0; b < d->batch; ++b) {
            const int nq = d->cu_seqlens_q_host[b + 1] - d->cu_seqlens_q_host[b];
            const int nk = d->cu_seqlens_k_host[b + 1] - d->cu_seqlens_k_host[b];
            if (nk < nq) return fail(PDD_ERR_INVALID_ARG, "sequence %d has fewer keys than queries", b);
            if (mode == MODE_PREFILL && nk != nq)
                return fail(PDD_ERR_INVALID_ARG, "sequence %d: prefill needs Nq == Nk", b);
        }
    }
    return PDD_OK;
}

float scale_log2(const pdd_attn_desc *d)
{
    const float s = d->softmax_scale > 0.f ? d->softmax_scale : 1.0f / std::sqrt((float)d->head_dim);
    return s * 1.4426950408889634f;
}

constexpr int kLdsBytes = 160 * 1024;    // of a compute unit, and the most one workgroup can have

// The dynamic-LDS limit of a kernel is raised once per (kernel, device), not on every launch.
pdd_status raise_lds_limit(const void *kern, int bytes)
{
    struct Done { const void *kern; int dev; };
    static Done done[64];
    static int n_done = 0;
    static std::mutex mu;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(PDD_ERR_HIP, "hipGetDevice: %s", hipGetErrorString(e));
    std::lock_guard<std::mutex> lock(mu);
    for (int i = 0; i < n_done; ++i)
        if (done[i].kern == kern && done[i].dev == dev) return PDD_OK;
    e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e != hipSuccess) return fail(PDD_ERR_HIP, "hipFuncSetAttribute: %s", hipGetErrorString(e));
    if (n_done < 64) done[n_done++] = {kern, dev};
    return PDD_OK;
}

template <typename Kern>
pdd_status launch_attn_kernel(Kern kern, int smem, int threads, const pdd::AttnParams &p, int64_t blocks,
                              hipStream_t st)
{
    const pdd_status s = raise_lds_limit(reinterpret_cast<const void *>(kern), kLdsBytes);      // (launches differ in what they take)
    if (s) return s;
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(threads), smem, st, p);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(PDD_ERR_HIP, "attention launch: %s", hipGetErrorString(e));
    return PDD_OK;
}

// spread: with the LDS of an 8-wave workgroup, so that no more than two share a compute unit
template <int D, int NW>
pdd_status launch_attn_t(const pdd::AttnParams &p, int64_t blocks, bool spread, hipStream_t st)
{
    if (p.imp_part)
        return launch_attn_kernel(pdd::attn_fwd_kernel<D, NW, true>, pdd::AttnSmem<D>::SWEEP_BYTES, NW * 64, p, blocks, st);
    return launch_attn_kernel(pdd::attn_fwd_kernel<D, NW>, pdd::AttnSmem<D>::bytes(spread ? 8 : NW), NW * 64, p, blocks, st);
}

int compute_units();

constexpr int kSplitRows = 128;          // packed (token, head) rows per workgroup of the key-split form
constexpr size_t kSplitWorkspaceMax = (size_t)256 << 20;
struct SplitPlan { int tiles, n_split; size_t bytes; double us; };        // tiles == 0: the form does not apply; us: its estimate

template <int D>
pdd_status launch_attn_split(const pdd::AttnParams &p, int64_t blocks, hipStream_t st)
{
    const pdd_status s = launch_attn_kernel(pdd::attn_fwd_kernel<D, kSplitRows / 32, false, true>,
                                            pdd::AttnSmem<D>::SPLIT_BYTES, 2 * kSplitRows, p, blocks, st);
    if (s) return s;
    const int64_t n = ((int64_t)p.total_q * p.Hq + 3) / 4;       // one wave per (token, head)
    hipLaunchKernelGGL(pdd::attn_combine_kernel<D>, dim3((unsigned)n), dim3(256), 0, st, p, kSplitRows);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(PDD_ERR_HIP, "attention combine launch: %s", hipGetErrorString(e));
    return PDD_OK;
}

// Queries per attention workgroup.  8 waves (256 queries, one workgroup per compute unit) halve the
// K/V traffic into LDS per flop and win wherever the compute units stay evenly busy; 4 waves (128
// queries: twice as many workgroups of half the rows, which spread more evenly) win on small grids.  Measured on 256 compute units, T = number of 256-query tiles:
// chunks behind a prefix at least as long (workgroups of nearly equal length) prefer 8 waves from
// T = 192 on (1.0 against 0.8 PFLOP/s) and 4 waves at T = 128 (0.87 against 0.76); causal prefill,
// whose workgroups differ in length by the number of query tiles, needs more than one 8-wave
// workgroup per compute unit before their dynamic placement evens out: 4 waves up to T = 256
// (0.76 against 0.70 PFLOP/s at 4096 tokens x 16 heads), 8 waves from T = 288 on.
int attn_rows_per_workgroup(const pdd_attn_desc *d)
{
    int nw = g_attn_waves;
    if (nw == 0) {
        const int64_t tiles256 = (int64_t)((d->max_seqlen_q + 255) / 256) * d->batch * d->n_q_heads;
        const bool even_lengths = d->max_seqlen_k - d->max_seqlen_q >= d->max_seqlen_q;
        const int64_t cus = compute_units();
        nw = tiles256 > (even_lengths ? cus / 2 : cus) ? 8 : 4;
    }
    return nw * 32;
}

// Query tiles that exist in a batch, at most, and whether the grid of 4-wave workgroups lists them (tile_of), longest walks first,
// instead of holding the longest sequence's tiles for each sequence: where a fifth of those at least would be empty.  (The place of the empty
// ones settles which shader engines the others go to: 653 + 6936 tokens x 8/8 heads 4 waves 188 us, 8 waves 124, 4 waves listed 116.
// Launches of many larger workgroups even out by themselves and lose half a per cent by the search.)
int64_t existing_tiles(const pdd_attn_desc *d, int bm) { return (d->total_q + (int64_t)d->batch * (bm - 1)) / bm; }
bool lists_tiles(const pdd_attn_desc *d)
{
    return d->batch > 1 && d->batch <= pdd::kListedMax &&
           4 * (int64_t)((d->max_seqlen_q + 127) / 128) * d->batch > 5 * existing_tiles(d, 128);
}

// Prompts of head_dim 128: uneven batches whose 256-query tiles do not go round the chip twice take 4 waves, however many the
// longest sequence's tiles for each sequence would be (8 waves or wide | 4 waves, listed: T = tiles by their mean number 173
// 380 + 2136 x 16/2 heads 49.9 | 41 us, 240 3308 + 4000 + 5809 + 1320 + 269 x 4/2 114 | 95, 333 7879 + 7 x 263 to 4548 x 4/2 157 | 127, 396
// 4924 + 1160 x 16/2 117 | 131, 479 4895 + 4 x 292 to 4048 x 8/8 122 | 146).  Below 0.69 of a tile to a compute unit one long walk decides, in
// which attn_wide_kernel is the faster (200 7726 + 4 x 464 to 2132 x 4/2 111 | 115).
// Of head_dim 64: 4 waves at every size (the largest go on to 64 queries to a wave, takes_wide): against 8 waves, two to a compute
// unit, 16384 tokens x 32/8 heads 1188 -> 1143 us, 8192 x 64/8 630 -> 597, 3000 + 1111 + 6100 x 32/8 253 -> 236, 8000 + 3 x 300 x 8/8
// 244 -> 205; only where the 8-wave workgroups just fill the chip once do they stay (3500 x 32/8, 448 of 512 places: 75.4
// against 77.0).  The chunked call keeps the rule above, by which its importance sweep and its scratch are sized.
int attn_prefill_rows_per_workgroup(const pdd_attn_desc *d)
{
    if (g_attn_waves != 0) return attn_rows_per_workgroup(d);
    if (d->head_dim == 128) {
        const double tiles = d->n_q_heads * (d->total_q / 256.0 + 0.5 * d->batch), cus = (double)compute_units();
        const bool few = tiles <= 1.3 * cus && (d->max_seqlen_q < 36 * pdd::kBN || tiles >= 0.6875 * cus);
        return few && lists_tiles(d) ? 128 : attn_rows_per_workgroup(d);
    }
    const int64_t tiles256 = (int64_t)((d->max_seqlen_q + 255) / 256) * d->batch * d->n_q_heads, slots = 2 * (int64_t)compute_units();
    return 32 * (8 * tiles256 > 6 * slots && tiles256 <= slots ? 8 : 4);
}

// Whether all query tiles of a call take the chip longer than the longest walk over the keys takes one of them; the sequences but
// the longest are taken for equally long.  Then three 4-wave workgroups of head_dim 64 share a compute unit (266 launches 1.04 to
// 1.19 times as fast as 8 waves; from a tenth longer on 64 queries to a wave).  Else no more than two: a long walk is the slower for two neighbours (1456 + 704 + 663 + 615 + 632 + 770 +
// 3482 + 5753 x 4/2 heads 87 us by threes, 71 by twos and 82 with 8 waves; 574 + 1335 + 7269 + 253 + 801 x 16/2 152, 139 and 139; 440 such prompts 1.04 times
// as fast by twos as by threes, 0.93 to 1.43, break even where both times are alike).
double fill_of_the_chip(const pdd_attn_desc *d)
{
    const double cus = (double)compute_units(), longest = d->max_seqlen_q, others = d->batch - 1.0, mean = others > 0 ? (d->total_q - longest) / others : 0.0;
    return d->n_q_heads * (longest * longest + others * mean * mean) / (512.0 * cus * longest);      // tiles of 256 rows, half their walk
}
bool tiles_fill_the_chip(const pdd_attn_desc *d) { return fill_of_the_chip(d) >= 1.0; }

// Launches that take attn_wide_kernel, 64 queries to a wave (bm: queries per workgroup of the other forms).
//   * head_dim 128: where the 8-wave workgroups were chosen and the longest walk (behind longer prefixes: the mean one) has 36
//     tiles or more.  A workgroup spends more cycles outside its loop than one of attn_fwd_kernel and 8 % fewer in it
//     (8 waves | wide: 2414 tokens x 64/8 heads 102.8 | 103.0 us, 2413 x 32/8 60.9 | 60.0, 2959 x 32/8 79.4 | 76.0, 2346 + 1560 x 32/8 72.4 | 73.9,
//     30 such prompts of 2300 to 3300 tokens 1.01 in the mean, 0.98 to 1.05; 403 x 4 behind 2598, 32/8 heads 77.7 | 76.5, 512 x 3 behind 3500
//     94.7 | 91.7, 64/8 187.9 | 179.0; below, with 2 % less in the loop than now: 1611 tokens x 64/8 55.1 | 56.2).
//   * Prompts of head_dim 64 that took 4 waves: where the tiles take the chip a tenth longer than the longest walk takes one, by the measure of
//     tiles_fill_the_chip.  Two of these workgroups share a compute unit where three of 128 queries do otherwise (4 waves | wide, that
//     measure in front: 0.90 1848 x 64/8 43.2 | 44.5, 0.99 8104 x 16/2 153 | 160, 1.19 2438 x 64/8 67.8 | 66.4, 1.41 2878 x 64/8 85.3 | 79.5,
//     1.61 6597 x 32/8 197.8 | 183.1.  One long sequence among short ones loses up to there: 1.11 3490 + 616 + 1965 + 734 x 32/8 89 | 101,
//     1.38 5603 + 599 x 32/8 144 | 152; 34 drawn batches from 1.1 to 1.7 1.01 in the mean, 0.88 to 1.08).
bool takes_wide(const pdd_attn_desc *d, int bm)
{
    if (g_attn_waves != 0) return false;
    if (d->head_dim == 128) {
        const bool prefixes = d->max_seqlen_k - d->max_seqlen_q >= d->max_seqlen_q;
        return bm == 256 && (prefixes ? d->total_k / d->batch : d->max_seqlen_k) >= 36 * pdd::kBN;
    }
    return bm == 128 && fill_of_the_chip(d) >= 1.1;
}

// The plain form of a call whose tiles would have bm queries: `sweeps` with the importance sweep.
int plain_form(const pdd_attn_desc *d, int bm, bool sweeps)
{
    if (takes_wide(d, bm) && (!sweeps || d->head_dim == 128)) return PDD_ATTN_WIDE;
    if (bm == 256) return PDD_ATTN_8_WAVES;
    return !sweeps && d->head_dim == 128 && lists_tiles(d) ? PDD_ATTN_4_WAVES_LISTED : PDD_ATTN_4_WAVES;
}

// Chunked mode can take the token importance from a second sweep inside the
// attention kernel (every query of the call is a window query there).  Its partial sums need one
// float per (query head, query tile, key); 0 = this shape does not use the sweep.
constexpr size_t kSweepWorkspaceMax = (size_t)256 << 20;
size_t sweep_workspace(const pdd_attn_desc *d)
{
    if (d->total_q == 0 || d->total_k == 0) return 0;
    const int bm = attn_rows_per_workgroup(d);
    const size_t n_qtiles = (size_t)((d->max_seqlen_q + bm - 1) / bm);
    // The sweep costs what full query tiles cost, the separate kernel what the rows present
    // cost: chunks that fill their tiles to less than 70 % take the separate kernel (measured on
    // 4 x (q + 8192) x 64 heads, sweep against separate kernel: 335 / 348 us at q = 192,
    // 327 / 301 at q = 160, 287 / 168 at q = 64).
    if (10 * (int64_t)d->max_seqlen_q < 7 * (int64_t)n_qtiles * bm) return 0;
    const size_t need = n_qtiles * d->n_q_heads * (size_t)d->total_k * sizeof(float);
    return need <= kSweepWorkspaceMax ? need : 0;
}

void launch_importance_reduce(const float *part, float *imp, int64_t n, int n_split, hipStream_t st)
{
    hipLaunchKernelGGL(pdd::importance_reduce_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st,
                       part, imp, n, n_split);
}

// What keeps the importance kernel from taking this shape (32-bit byte offsets inside one
// sequence's Q rows and inside the log-sum-exp tensor), or NULL
const char *importance_limits(const pdd_attn_desc *d)
{
    const int64_t span = 2 * ((int64_t)d->max_seqlen_q * d->q_stride_tok + (int64_t)d->n_q_heads * d->q_stride_head);
    if (span >= (1LL << 32)) return "a sequence's Q span must stay below 4 GiB";
    if ((int64_t)d->n_q_heads * d->total_q * 4 >= (1LL << 32)) return "the log-sum-exp tensor must stay below 4 GiB";
    return nullptr;
}

// What a chunk's attention costs in the plain form, in microseconds, from the sizes alone.  Fitted on 256 compute units to the
// times of 1400 chunks and prompts (inputs of their own in every call), half of them within 5 %, nine in ten within 20; a launch
// lasts as long as its longest sequence's walk over the key tiles or as its tiles take the whole chip.
// (Uneven batches are priced as if the longest query sequence met all keys; the 400 chunks that take attn_wide_kernel have 0.74 to 1.2
// of it, half of them 0.87 to 1.15.)
double plain_attention_us(const pdd_attn_desc *d, int bm)
{
    const double cus = (double)compute_units(), max_q = d->max_seqlen_q;
    const int64_t n_qt = (d->max_seqlen_q + bm - 1) / bm, tiles_max = (d->max_seqlen_k + pdd::kBN - 1) / pdd::kBN;
    const double fill = max_q / (double)(n_qt * bm), seen = 1.0 - 0.5 * max_q / d->max_seqlen_k;
    const double work = (double)n_qt * d->n_q_heads * ((double)d->total_k / pdd::kBN + 0.5 * d->batch) * seen / cus;
    const double us = bm == 256 ? std::fmax(tiles_max * (0.75 + 0.5 * fill), work * (0.75 + 1.05 * fill))
                                : std::fmax((double)tiles_max, work) * (0.75 + 0.15 * fill);
    return 5.0 + (d->head_dim == 64 ? 0.68 : 0.95) * us;
}

// `of` a sequence's tokens, summed over a prompt batch whose sequences but the longest are taken for equally long, for a compute unit.
template <typename F>
double per_compute_unit(const pdd_attn_desc *d, F of)
{
    const double longest = d->max_seqlen_q, others = d->batch - 1.0, mean = others > 0 ? (d->total_q - longest) / others : 0.0;
    return (of(longest) + (mean > 0 ? others * of(mean) : 0.0)) / compute_units();
}
double with_part(double a, double b, double share) { return std::fmax(a, b) + share * std::fmin(a, b); }

// What a prompt batch's attention costs in the plain form that it would run in, in microseconds, from the sizes alone: the longest
// walk in key tiles, and the key tiles that all tiles walk for a compute unit.  Fitted on 256 compute units to 6000 prompt batches of 1
// to 8 sequences of 200 to 16384 tokens, every form on those that it is chosen for: half of them within 1 to 5 %, nine in ten within 4
// to 20 (attn_wide_kernel up to 250 us; beyond, the clock decides and no other form is near).
double plain_prompt_us(const pdd_attn_desc *d)
{
    struct Price { double base, walk, all, less; };      // [head_dim 64][4 waves, 8 waves, 4 waves listed, wide]
    static const Price prices[2][4] = {{{6.87, 0.771, 0.955, 0.244}, {9.05, 1.31, 1.88, 0.0}, {7.55, 0.766, 1.01, 0.244}, {10.1, 0.968, 1.56, 0.273}},
                                       {{6.02, 0.585, 0.498, 0.377}, {7.52, 0.764, 0.829, 0.334}, {}, {14.6, 1.18, 0.846, 0.223}}};
    const int form = plain_form(d, attn_prefill_rows_per_workgroup(d), false);
    const Price &p = prices[d->head_dim == 64][form];
    const double bm = form == PDD_ATTN_8_WAVES || form == PDD_ATTN_WIDE ? 256.0 : 128.0, walk = (d->max_seqlen_q + pdd::kBN - 1) / pdd::kBN;
    const double all = d->n_q_heads * per_compute_unit(d, [&](double n) {
        const double t = std::ceil(n / bm);
        return t * (n / pdd::kBN + 0.5) - 0.5 * t * (t - 1.0) * bm / pdd::kBN;
    });
    return p.base + with_part(p.walk * walk, p.all * all, p.less);
}

// Key tiles that a prompt batch's tiles of `rows` packed (token, head of the group) rows walk, for a compute unit.
double packed_prompt_walks(const pdd_attn_desc *d, int rows)
{
    return d->n_q_heads * per_compute_unit(d, [&](double n) { return n / rows * (n / pdd::kBN + 1.0) / 2.0; });
}

// Whether the sizes are inside what every form but the plain one can take: the kernels divide a row by G with one 32-bit
// multiplication and address `rows` rows of Q, 32 or 128, with 32-bit byte offsets.
bool packed_rows_fit(const pdd_attn_desc *d, int rows)
{
    // (the scratch query comes here with whatever its caller's descriptor holds)
    if (g_attn_waves != 0 || d->total_q <= 0 || d->total_k <= 0 || d->max_seqlen_q <= 0 || d->max_seqlen_k <= 0 ||
        (d->head_dim != 64 && d->head_dim != 128) || d->n_q_heads % d->n_kv_heads)
        return false;
    const int64_t G = d->n_q_heads / d->n_kv_heads, max_q = d->max_seqlen_q;
    if (G > 65535 || max_q * G >= (1LL << 31) || max_q * G * G >= (1LL << 32)) return false;
    return rows * d->q_stride_tok < (1LL << 30) && G * d->q_stride_head < (1LL << 30);
}

// Whether and how the keys of a prompt are split over workgroups (attn_fwd_kernel's SPLIT form).
// The plain form gives a workgroup all keys of 128 or 256 queries of one head, so a call lasts at
// least as long as its longest sequence's walk over the key tiles, however few workgroups there
// are.  The split form packs the (token, head) rows of a KV group into its tiles and cuts the walk into pieces of `tiles` key
// tiles; it pays with 32-bit partial rows, written once and read back by a second kernel.
// The choice compares estimates in microseconds, fitted to times on 256 compute units of 3700 prompt batches that could be split (half
// of them within 8 %), with plain_prompt_us: 2048 tokens x 1 head 31 -> 18 and 8192 x 4/2 heads 117 -> 94; the plain form is better on
// prompts that fill the chip (8192 tokens x 8 heads 135 against 165).
// Depends on the descriptor and the device only.
SplitPlan split_plan(const pdd_attn_desc *d)
{
    const SplitPlan none = {0, 0, 0, 0.0};
    if (!packed_rows_fit(d, 32)) return none;
    const int64_t G = d->n_q_heads / d->n_kv_heads, Hkv = d->n_kv_heads, B = d->batch, max_q = d->max_seqlen_q;
    const double cus = (double)compute_units();
    const int64_t n_qt = (max_q * G + kSplitRows - 1) / kSplitRows;
    const int64_t tiles_max = (d->max_seqlen_k + pdd::kBN - 1) / pdd::kBN;
    const double tiles_all = (double)d->total_k / pdd::kBN + 0.5 * B;
    const double seen = 1.0 - 0.5 * max_q / d->max_seqlen_k;    // share of the keys an average query tile walks

    // Key tiles per workgroup: about one workgroup per compute unit, 8 to 24 tiles (fewer and the
    // start of a workgroup and the partial rows cost more than they spread), evened out over the longest sequence, and
    // as many more as the scratch asks for.
    const double base = (double)(n_qt * Hkv);
    double T = 24;
    if (cus > base * B) T = std::ceil(tiles_all * base / (cus - base * B));
    T = T < 8 ? 8 : T > 24 ? 24 : T;
    if ((double)d->total_q * d->n_q_heads > (double)kSplitWorkspaceMax) return none;
    const size_t per_split = (size_t)d->total_q * d->n_q_heads * (d->head_dim + 1) * sizeof(float);
    const size_t room = kSplitWorkspaceMax / per_split;
    int64_t n_split = (tiles_max + (int64_t)T - 1) / (int64_t)T;
    if (n_split > (int64_t)room) n_split = (int64_t)room;
    if (n_split < 2) return none;
    const int64_t tiles = (tiles_max + n_split - 1) / n_split;
    n_split = (tiles_max + tiles - 1) / tiles;
    if ((double)n_split * base * B >= 2147483647.0) return none;

    const double partial = (double)n_split * per_split * seen * 1e-6 / 4.0;     // written and read back, at 4 TB/s each
    const double all = packed_prompt_walks(d, kSplitRows);
    // As long as its pieces, or as the chip takes for all of them.  (8/8 heads, head_dim 128, plain against
    // split: 1500 tokens 26 and 30 us, 2441 39 and 46, 694 + 2020 33 and 43, 4000 63 and 66; 4/2 heads 2441 37 and 29.)
    const double us = d->head_dim == 64 ? std::fmax(9.1 + 0.627 * tiles + 0.228 * all + 5.95 * partial, 0.668 * all + 2.72 * partial)
                                        : std::fmax(11.4 + 0.635 * tiles + 0.55 * all + 3.48 * partial, 14.7 + 1.11 * all + 0.988 * partial);
    if (us > 0.97 * plain_prompt_us(d)) return none;
    return {(int)tiles, (int)n_split, (size_t)n_split * per_split, us};
}

size_t importance_workspace(const pdd_attn_desc *d, int window);

// The form of attn_rows.hpp that a call takes: row groups per workgroup (0: none, the plain form or split_plan's), workgroups
// per KV head and partial rows where the keys are divided (workers == 0: they are not).
//   * Whole (RG = 1): a workgroup per tile of 32 packed rows walks all of its keys, eight blocks at a time.
//   * Divided (RG = 1 or 4): pieces of the key tiles over about one workgroup per compute unit and a second kernel
//     that joins them; RG = 4 reads K and V once for 128 rows.
// The choice compares estimates in microseconds with the plain form's, fitted like those (half of the whole prompts within 4 %, else
// a median error of 7 to 15 %), and wants some of the plain time off.  Attention alone, plain or split as before | whole | RG = 1 | RG = 4:
// 512 tokens x 1/1 head of 64 9.6 | 6.3 us, 2000 x 8/8 of 128 31 | 21; 1 token behind 1126 keys, 4/2 heads of 128 17.3 | 9.7 |
// 11.3 | 12.7, 8 x 1 behind 512 to 7900, 32/8 heads 32.1 | 85 | 26 | 28; 5 to 64 tokens x 4 behind 700 to 12345, 32/8 heads 54 | - | 77 |
// 41.5; 7 chunks of 3 to 230 behind 200 to 12700, 16/2 heads 88 | - | 79 | 48; 256 behind 8192, 64/8 heads (243 plain) 240 | - | 190 | 172.
// (Beyond 100 us the whole form was not once the better one in 250 launches: K and V come once per 32 rows.)
// The divided forms' scratch of a chunked call stays within the built-in scratch, so that the call without a workspace
// argument takes the same form where it has importance to return.  Depends on the descriptor, the device and `scratch`, the
// bytes that there are (a prompt: 0 where the key-split form has no room).
constexpr int kWholeTiles = 45;
struct RowsPlan { int rg; int64_t workers; int min_tiles; int64_t part_rows; size_t bytes; };

RowsPlan rows_plan(const pdd_attn_desc *d, bool chunked, size_t scratch)
{
    RowsPlan best = {0, 0, 0, 0, 0};
    if (!packed_rows_fit(d, 32)) return best;
    const int64_t G = d->n_q_heads / d->n_kv_heads, Hkv = d->n_kv_heads, B = d->batch, max_q = d->max_seqlen_q, total_q = d->total_q;
    if (chunked) {      // the importance kernel has to be able to follow (the sweep has wider limits)
        if (importance_workspace(d, -1) > PDD_STATIC_SCRATCH_BYTES || importance_limits(d)) return best;
    }
    const double cus = (double)compute_units();
    const bool d64 = d->head_dim == 64;
    const double tiles_max = (double)((d->max_seqlen_k + pdd::kBN - 1) / pdd::kBN);
    const double tiles_mean = ((double)d->total_k / pdd::kBN + 0.5 * B) / B, seen = 1.0 - 0.5 * max_q / d->max_seqlen_k;
    auto row_tiles = [&](int rg) {      // of all sequences
        return std::fmin((double)total_q * G / (32 * rg) + 0.5 * B, (double)((max_q * G + 32 * rg - 1) / (32 * rg)) * B);
    };
    const double plain = chunked ? plain_attention_us(d, attn_rows_per_workgroup(d)) : plain_prompt_us(d), share = chunked || d64 ? 0.9 : 0.95;
    double us = share * plain;
    if (!chunked && scratch)
        if (const SplitPlan split = split_plan(d); split.tiles) {
            // A prompt that the key-split form takes a tenth off keeps to it beyond kWholeTiles, where the whole form waits for keys that no
            // cache holds (1/1 head of 128, whole and split with keys from memory: 6350 tokens 47.6 and 37.2 us, 3350 + 300 30.0 and 25.9).
            if (tiles_max > kWholeTiles && split.us < 0.9 * plain) return best;
            us = std::fmin(us, share * split.us);
        }
    {
        // rounds of the longest walk, what all walks take the chip, and a start for each workgroup behind the first of a compute unit
        const double rounds = std::ceil(tiles_max / 4.0);
        const int64_t blocks = (max_q * G + 31) / 32 * B * Hkv;
        double est, empty = 0.0;
        if (chunked) {
            const double rt = row_tiles(1), tiles = rt * Hkv * seen * (0.4 * tiles_mean + 0.6 * tiles_max) / cus, per_cu = rt * Hkv / cus;
            // (head_dim 128: whole rounds, because a workgroup has its compute unit to itself, and the unit waits for workgroups without
            // a row tile too, 1.5 us each for the first few: 24 to 257 new tokens x 7, 32/8 heads, 20.7 us, plain 14.7; 143 + 8 + 3 x 64/8 12.1 and 8.7)
            const double over = std::fmax((!d64 && per_cu < 3.0 ? std::ceil(per_cu - 0.03) : per_cu) - 1.0, 0.0);
            if (!d64) empty = std::fmin(1.5 * std::fmax((double)blocks / cus - per_cu - 0.5, 0.0), 3.0);
            est = d64 ? 4.6 + with_part(0.73 * rounds, 0.18 * tiles + 3.0 * over, 0.3) : 5.0 + with_part(1.33 * rounds, 0.30 * tiles + 4.1 * over, 0.3);
        } else {
            const double all = packed_prompt_walks(d, 32), over = std::fmax(((double)total_q * G / 32 + 0.5 * B) * Hkv / cus - 1.0, 0.0);
            est = d64 ? 6.09 + with_part(0.518 * rounds, 0.142 * all + 1.97 * over, 0.738) : 7.67 + with_part(0.674 * rounds, 0.205 * all + 5.77 * over, 1.2);
        }
        if (est + empty < us && est < 100.0 && blocks <= 0x7fffffffLL) {
            us = est + empty;
            best = {1, 0, 0, 0, 0};
        }
    }
    if (!chunked || !scratch) return best;
    const int64_t scratch_bytes = scratch < PDD_STATIC_SCRATCH_BYTES ? (int64_t)scratch : (int64_t)PDD_STATIC_SCRATCH_BYTES;
    for (int rg = 1; rg <= 4; rg += 3) {
        if (!packed_rows_fit(d, 32 * rg)) continue;
        const int64_t per_head = compute_units() / Hkv > 1 ? compute_units() / Hkv : 1, rows = 32 * rg;
        const int64_t by_rows = total_q * G / rows + B, by_longest = (max_q * G + rows - 1) / rows * B, pairs = by_rows < by_longest ? by_rows : by_longest;
        // Workgroups for the pieces.  Few (sequence, row tile) pairs: what is on the chip at once, one to a compute unit (one token x 8 and the like).
        // Each pair has up to a piece more than its share, so many of them at one round's share run into a second round: then
        // three rounds of smaller pieces where each sequence is one row tile (41 x 2 tokens behind 113 to 14497 keys, 8/8 heads of 64 83.7 -> 71.7 us,
        // 19 such launches of 31 and more 1.07 to 1.19 times as fast), two workgroups to a compute unit at head_dim 64 (341 + 10 + 56 + 20 + 1 + 58 behind
        // 268 to 15973, 32/8 heads 108 -> 89; 73 launches 1.05, 0.94 to 1.31; at shares of fewer than 16 key tiles 0.97), one round up to 0.7 pairs at head_dim 128 with 32 rows (17 launches 1.05).
        int64_t workers = per_head + pairs;
        if (2 * pairs <= per_head || (rg == 1 && !d64 && max_q * G > rows && 10 * pairs <= 7 * per_head)) workers = per_head;
        else if (max_q * G <= rows && pairs <= 2 * per_head) workers = 3 * per_head;
        else if (max_q * G > rows && d64 && 10 * pairs <= 9 * per_head && row_tiles(rg) * tiles_mean >= 16.0 * per_head) workers = 2 * per_head;
        const int64_t row_bytes = (int64_t)d->n_q_heads * (d->head_dim + 1) * (int64_t)sizeof(float);
        const int64_t table = total_q * d->n_q_heads * (int64_t)sizeof(uint4);
        const int64_t room = (scratch_bytes - table) / row_bytes;
        if (workers * Hkv > 0x7fffffffLL || room < total_q + (total_q + 3) / 4) continue;
        if ((double)(total_q > pairs ? total_q : pairs) * tiles_max >= 2147483648.0) continue;      // work_per's sums
        const int min_tiles = rg == 1 ? 8 : 4;
        // key tiles of a piece as the kernel will find them (work_per)
        const double rt = row_tiles(rg), tiles = rt * seen * (rg == 1 ? 0.3 * tiles_mean + 0.7 * tiles_max : 0.7 * tiles_mean + 0.3 * tiles_max);
        double per = std::ceil(rt * tiles_mean / std::fmax((double)workers - rt, 1.0));
        per = std::fmin(std::fmax(std::fmax(per, total_q * tiles_max / (double)(room - total_q)), (double)min_tiles), tiles_max);
        const double all = tiles * Hkv / cus;
        const double est = rg == 1 ? (d64 ? 10.7 + 0.024 * std::ceil(per / 4.0) + 0.20 * all : 12.2 + 0.42 * std::ceil(per / 4.0) + 0.30 * all)
                                   : (d64 ? 11.7 + 0.053 * per + 0.61 * all : 15.1 + 0.85 * all);
        // Where no cache nearer than the memory's own holds the keys and values, each tile of 32 rows reads them anew, at some
        // 9 TB/s: 128 rows are compared with that (67 tokens x 6 behind 13418, 8/8 heads of 64, 97 us, 72 with smaller pieces, in 128 rows 45;
        // 97 launches that this decides 1.31 times as fast, 0.89 to 1.97; from 64 to 80 MB 20 took 0.71 to 1.7).
        const double tile_mb = 2.0 * pdd::kBN * d->head_dim * 2e-6;
        if (rg == 4 && best.rg == 1 && max_q * G > 32 && tile_mb * tiles_mean * B * Hkv > 80.0)
            us = std::fmax(us, 5.0 + row_tiles(1) * tiles_mean * seen * Hkv * tile_mb / 9.0);
        if (est < 0.95 * us) {
            us = est;
            // what the pieces can take at most: each sequence one more than `min_tiles` goes into its key tiles
            const int64_t most = total_q * (((int64_t)tiles_max + min_tiles - 1) / min_tiles + 1), part_rows = most < room ? most : room;
            best = {rg, workers, min_tiles, part_rows, (size_t)(part_rows * row_bytes + table)};
        }
    }
    return best;
}

template <int D, int RG>
pdd_status launch_attn_rows(const RowsPlan &plan, pdd::AttnParams &p, int64_t max_q, void *scratch, hipStream_t st)
{
    p.g_magic = p.G > 1 ? (uint32_t)(((1ull << 32) + p.G - 1) / p.G) : 0u;
    if constexpr (RG == 1)                                       // the whole form has 32 rows to a workgroup
        if (plan.workers == 0) {
            p.n_qtiles = (int)((max_q * p.G + 31) / 32);
            p.turn = pdd::rows_per_turn(p.Hkv);
            return launch_attn_kernel(pdd::attn_rows_kernel<D, 1, false>, pdd::RowsSmem<D, 1>::BYTES, 64 * pdd::kRowsWaves, p,
                                      (int64_t)p.n_qtiles * p.B * p.Hkv, st);
        }
    p.workers = (int)plan.workers;  p.min_tiles = plan.min_tiles;  p.part_rows = (int)plan.part_rows;
    p.part_of = (uint4 *)scratch;
    p.part_o = (float *)(p.part_of + (int64_t)p.total_q * p.Hq);
    p.part_l = p.part_o + plan.part_rows * p.Hq * D;
    const pdd_status s = launch_attn_kernel(pdd::attn_rows_kernel<D, RG, true>, pdd::RowsSmem<D, RG>::BYTES, 64 * pdd::kRowsWaves, p,
                                            plan.workers * p.Hkv, st);
    if (s) return s;
    const int64_t n = ((int64_t)p.total_q * p.Hq + 3) / 4;       // one wave per (token, head)
    hipLaunchKernelGGL(pdd::attn_join_kernel<D>, dim3((unsigned)n), dim3(256), 0, st, p);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(PDD_ERR_HIP, "attention join launch: %s", hipGetErrorString(e));
    return PDD_OK;
}

// The attention form of a call.  bm: queries per workgroup of the plain forms but the wide one; split, rows: the plans of
// PDD_ATTN_SPLIT and PDD_ATTN_ROWS.
struct AttnForm { int kind, bm; SplitPlan split; RowsPlan rows; };

// imp_part != NULL: sweep_workspace(d) bytes; the importance sweep runs inside
// the attention kernel and leaves its partial sums there.
// scratch: split.bytes or rows.bytes of a form that divides the keys.
pdd_status launch_attn(const pdd_attn_desc *d, const AttnForm &form, const void *q, const void *k, const void *v, void *o, float *lse,
                       hipStream_t st, float *imp_part, void *scratch)
{
    if (d->total_q == 0) return PDD_OK;
    pdd::AttnParams p;
    p.imp_part = imp_part;
    p.split_tiles = p.n_split = 0;  p.g_magic = 0;  p.part_o = p.part_l = nullptr;
    p.q = (const uint16_t *)q;  p.k = (const uint16_t *)k;  p.v = (const uint16_t *)v;
    p.o = (uint16_t *)o;  p.lse = lse;
    p.cu_q = d->cu_seqlens_q;  p.cu_k = d->cu_seqlens_k;
    p.q_st = d->q_stride_tok;  p.q_sh = d->q_stride_head;
    p.k_st = d->k_stride_tok;  p.k_sh = d->k_stride_head;
    p.v_st = d->v_stride_tok;  p.v_sh = d->v_stride_head;
    p.o_st = d->o_stride_tok;  p.o_sh = d->o_stride_head;
    p.B = d->batch;  p.Hq = d->n_q_heads;  p.Hkv = d->n_kv_heads;  p.G = d->n_q_heads / d->n_kv_heads;
    p.total_q = d->total_q;  p.total_k = d->total_k;
    p.turn = 1;
    p.scale_log2 = scale_log2(d);

    const int bm = form.kind == PDD_ATTN_WIDE ? pdd::kWideRows : form.bm, nw = bm / 32;
    p.n_qtiles = (d->max_seqlen_q + bm - 1) / bm;
    int64_t blocks = (int64_t)p.n_qtiles * d->batch * d->n_q_heads;
    if (blocks > 0x7fffffffLL) return fail(PDD_ERR_INVALID_ARG, "launch grid too large");
    p.listed = 0;
    if (form.kind == PDD_ATTN_4_WAVES_LISTED) {
        p.listed = (d->max_seqlen_k > d->max_seqlen_q ? d->max_seqlen_k : d->max_seqlen_q) / bm + 1;
        blocks = existing_tiles(d, bm) * d->n_q_heads;
    }
    {   // 32-bit byte offsets inside one sequence's K / V span (buffer addressing); the kernels
        // request up to six tiles of 64 rows past a sequence's end, which read as zero
        const int64_t span = ((int64_t)d->max_seqlen_k + 512) * 2 *
                             (d->k_stride_tok > d->v_stride_tok ? d->k_stride_tok : d->v_stride_tok);
        if (span >= (1LL << 32)) return fail(PDD_ERR_UNSUPPORTED, "a sequence's K/V span must stay below 4 GiB");
        // and inside the 32 query rows of a wave
        if ((int64_t)d->q_stride_tok * 2 * 32 >= (1LL << 32))
            return fail(PDD_ERR_UNSUPPORTED, "32 rows of Q must span less than 4 GiB");
    }
    if (form.kind == PDD_ATTN_ROWS) {
        const RowsPlan &rows = form.rows;
        if (d->head_dim == 128)
            return rows.rg == 1 ? launch_attn_rows<128, 1>(rows, p, d->max_seqlen_q, scratch, st) : launch_attn_rows<128, 4>(rows, p, d->max_seqlen_q, scratch, st);
        return rows.rg == 1 ? launch_attn_rows<64, 1>(rows, p, d->max_seqlen_q, scratch, st) : launch_attn_rows<64, 4>(rows, p, d->max_seqlen_q, scratch, st);
    }
    if (form.kind == PDD_ATTN_SPLIT) {
        p.split_tiles = form.split.tiles;  p.n_split = form.split.n_split;
        p.n_qtiles = (int)(((int64_t)d->max_seqlen_q * p.G + kSplitRows - 1) / kSplitRows);
        p.g_magic = p.G > 1 ? (uint32_t)(((1ull << 32) + p.G - 1) / p.G) : 0u;
        p.part_o = (float *)scratch;
        p.part_l = p.part_o + (size_t)form.split.n_split * d->total_q * d->n_q_heads * d->head_dim;
        const int64_t n = (int64_t)p.n_qtiles * d->batch * d->n_kv_heads * form.split.n_split;
        return d->head_dim == 128 ? launch_attn_split<128>(p, n, st) : launch_attn_split<64>(p, n, st);
    }
    if (form.kind == PDD_ATTN_WIDE) {
        if (imp_part)
            return launch_attn_kernel(pdd::attn_wide_kernel<128, true>, pdd::WideSmem<128>::BYTES, 64 * pdd::kWideWaves, p, blocks, st);
        if (d->head_dim == 128)
            return launch_attn_kernel(pdd::attn_wide_kernel<128>, pdd::WideSmem<128>::BYTES, 64 * pdd::kWideWaves, p, blocks, st);
        return launch_attn_kernel(pdd::attn_wide_kernel<64>, pdd::WideSmem<64>::BYTES, 64 * pdd::kWideWaves, p, blocks, st);
    }
    if (d->head_dim == 128)
        return nw == 8 ? launch_attn_t<128, 8>(p, blocks, false, st) : launch_attn_t<128, 4>(p, blocks, false, st);
    return nw == 8 ? launch_attn_t<64, 8>(p, blocks, false, st) : launch_attn_t<64, 4>(p, blocks, !tiles_fill_the_chip(d), st);
}

template <int QPT>
void launch_select_reg(const pdd::SelParams &p, dim3 grid, hipStream_t st)
{
    if (p.pool_r == 0)
        hipLaunchKernelGGL((pdd::select_topk_reg_kernel<QPT, false>), grid, dim3(pdd::kSelThreads), 0, st, p);
    else
        hipLaunchKernelGGL((pdd::select_topk_reg_kernel<QPT, true>), grid, dim3(pdd::kSelThreads), 0, st, p);
}

// Chunks of 4096 candidates of the longest sequence where a selection divides its rows over workgroups, 0 where
// a row stays in one.  Longer rows than one workgroup's registers hold, 32768, are read again in every pass of the one
// workgroup: 8 x 65536 13.3 us divided against 117, 8 x 131072 16.5 against 225.  More than 5/4 of a row per compute unit keep the chip
// busy by themselves, two to a compute unit (512 x 33000 107 against 121 us), and stay whole for the scratch that they would
// take; so do rows of more than 512 chunks, whose sums would be long, and 8192 chunks bound the scratch to 68 MiB.
int select_chunks(int64_t n_heads, int64_t batch, int64_t max_seqlen_k)
{
    const int64_t chunks = (max_seqlen_k + pdd::kSplitSelChunk - 1) / pdd::kSplitSelChunk;
    if (max_seqlen_k <= pdd::kSelRegCap || chunks > 512 || batch > 8192 || n_heads > 8192) return 0;
    return 4 * n_heads * batch <= 5 * (int64_t)compute_units() && n_heads * batch * chunks <= 8192 ? (int)chunks : 0;
}

size_t select_workspace(int64_t n_heads, int64_t batch, int chunks)
{
    return (size_t)(n_heads * batch) * (size_t)chunks * pdd::kSplitSelChunkBytes;
}

template <int QPT>
void launch_select_split_t(const pdd::SelParams &s, int chunks, void *workspace, hipStream_t st)
{
    pdd::SplitSelParams p;
    p.s = s;
    p.n_chunks = (chunks + QPT - 1) / QPT;
    p.n_units = chunks;
    const int64_t rows = (int64_t)s.n_heads * s.B;
    p.list = (uint16_t *)workspace;
    p.before = p.list + rows * p.n_units * pdd::kSplitSelChunk;
    p.counts = (pdd::DivCounts *)(p.before + rows * p.n_chunks * pdd::kDivBins);
    p.row = (uint2 *)(p.counts + rows * p.n_chunks);
    const dim3 grid((unsigned)p.n_chunks, (unsigned)s.B, (unsigned)s.n_heads), block(pdd::kSelThreads);
    hipLaunchKernelGGL(pdd::select_bracket_kernel<QPT>, grid, block, 0, st, p);
    hipLaunchKernelGGL(pdd::select_divided_kernel<QPT>, grid, block, 0, st, p);
}

// Chunks of 4096 candidates to a workgroup: one while every compute unit gets at most one (8 x 131072 16 us, 17 with
// two, 21 with four), two up to two of them (32 x 65536 23, 20 and 21), four beyond (32 x 131072 41, 30 and 27), because each
// workgroup reads the row's sample and what all of its chunks hold.  The latter makes two the better choice for very long rows
// too (1 x 800000 22.5 and 19.9; 1 x 200000 13.8 and 14.8).
pdd_status launch_select_split(const pdd::SelParams &s, int chunks, void *workspace, hipStream_t st)
{
    const int64_t all = (int64_t)s.n_heads * s.B * chunks, cus = compute_units();
    if (all <= cus && chunks <= 64) launch_select_split_t<1>(s, chunks, workspace, st);
    else if (all <= 2 * cus) launch_select_split_t<2>(s, chunks, workspace, st);
    else launch_select_split_t<4>(s, chunks, workspace, st);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(PDD_ERR_HIP, "select launch: %s", hipGetErrorString(e));
    return PDD_OK;
}

int compute_units()
{
    static std::atomic<int> cached{0};
    int n = cached.load();
    if (n > 0) return n;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1)
        return 256;                       // no device visible (host-only use): the MI355X figure
    cached.store(n);
    return n;
}

// Into how many workgroups the window rows of one 256-key slice are divided.  The importance
// kernel runs three 4-wave workgroups per compute unit; with one workgroup per slice the last
// round of a launch is often mostly empty and every workgroup walks all of its row blocks alone.
// The choice minimises rounds x (row blocks per workgroup + a start-up cost of about six row
// blocks), charges the extra reduction pass as three more, and only leaves the single-pass form
// for a gain above 15 % (measured: 246 -> 220 us on 4 x 8448 keys x 64 heads x 256 rows, nothing
// on the 32k-token prompt with its 128 window rows).  It depends only on the descriptor and the
// device.
template <typename Cost>
int best_importance_split(Cost &&cost, int64_t blocks)
{
    int best = 1;
    for (int r = 2; r <= 8 && blocks / r >= 4; ++r)
        if (cost(r) < (best == 1 ? 0.85 * cost(1) : cost(best))) best = r;
    return best;
}

// every sequence taken for the longest one
int importance_split_even(const pdd_attn_desc *d, int window)
{
    const int64_t slots = 3 * (int64_t)compute_units();
    const int64_t n_ktiles = (d->max_seqlen_k + pdd::kImpBK - 1) / pdd::kImpBK;
    const int64_t wgs = n_ktiles * d->batch * d->n_kv_heads;
    const int w = (window < 0 || window > d->max_seqlen_q) ? d->max_seqlen_q : window;
    const int64_t items = (int64_t)(d->n_q_heads / d->n_kv_heads) * ((w + 31) / 32);        // at whole blocks of a head
    return best_importance_split([&](int r) {
        const double rounds = (double)((wgs * r + slots - 1) / slots);
        return rounds * ((double)((items + r - 1) / r) + 6.0) + (r > 1 ? 3.0 : 0.0);
    }, items);
}

int importance_split(const pdd_attn_desc *d, int window)
{
    const int even = importance_split_even(d, window);
    const int w = (window < 0 || window > d->max_seqlen_q) ? d->max_seqlen_q : window;
    if ((int64_t)d->batch * d->max_seqlen_k == d->total_k && (w < d->max_seqlen_q || (int64_t)d->batch * w == d->total_q)) return even;
    // Sequences of different lengths: the longest walk over the row blocks, or what all slices take of the chip's places at
    // the mean window (only slices with keys are launched).  By the rule above the walks stayed whole: 1 to 383 tokens x 6 behind
    // 314 to 10880 keys, 16/2 heads 105 us, 68 divided; 6 to 315 x 7 behind
    // 117 to 2169, 32/8 heads 58.9 and 48.0; 277 tokens and seven sequences of few, where the long walk has few keys, 82.5 and 83.9.
    const double group = (double)(d->n_q_heads / d->n_kv_heads), slots = 3.0 * compute_units();
    const double mean_items = std::fmax(group * std::fmin((double)w, (double)d->total_q / d->batch) / 32.0, 1.0);
    const int64_t longest = ((int64_t)(d->n_q_heads / d->n_kv_heads) * w + 31) / 32;
    const int64_t by_keys = d->total_k / pdd::kImpBK + d->batch, by_longest = (int64_t)((d->max_seqlen_k + pdd::kImpBK - 1) / pdd::kImpBK) * d->batch;
    const double real_wgs = (double)(by_keys < by_longest ? by_keys : by_longest) * d->n_kv_heads;
    const int uneven = best_importance_split([&](int r) {
        return std::fmax((double)((longest + r - 1) / r) + 6.0, real_wgs * r / slots * (mean_items / r + 6.0)) + (r > 1 ? 3.0 : 0.0);
    }, longest);
    // (the built-in scratch holds what the rule above would ask for or this)
    const int64_t bytes = (int64_t)d->n_kv_heads * d->total_k * (int64_t)sizeof(float), fits = bytes > 0 ? PDD_STATIC_SCRATCH_BYTES / bytes : 8;
    return uneven <= even || uneven <= fits ? uneven : even > fits ? even : (int)fits;
}

// scratch for the partial sums of that many workgroups to a slice
size_t importance_split_bytes(const pdd_attn_desc *d, int r)
{
    return r > 1 ? (size_t)r * d->n_kv_heads * (size_t)d->total_k * sizeof(float) : 0;
}

// Whether the importance takes the form with all window rows in LDS, and its launch shape.
// The rows have to fit the 160 KB of a compute unit (19 blocks of 32 at head_dim 128).  Above 80 KB one
// 16-wave workgroup runs per compute unit: only for launches that fill the chip's 4096 wave slots with 32-key
// groups (64 tokens x 4 behind 8192 keys, 64/8 heads 46 us, 57 with the streaming kernel; 200 tokens behind 16000, 4/2
// heads, would take 15.3 us against 12.3 of the streaming kernel, which divides the rows).  A round of such
// workgroups takes 1.9 times as long with two groups per wave as with one, so the rounds decide: 32768 tokens, window of
// 128, 32/8 heads (one round or two) 38.2 us with two groups, 42.1 with one, 8 x 5000 (two or three) 64 and
// 61.5, 16 x 1000 (one either way) 29.3 and 22.1; 51.5, 59.5 and 27.0 with the streaming kernel.  Below 80 KB
// two or more run per compute unit; four waves each while all of them are resident at once (4096
// tokens, window of 64: 7.0 us, 8.5 with eight waves), else eight waves, which load the rows half as often,
// and two groups per wave from 4096 groups on (8 prompts of 512 to 7900 tokens, window of 64: 21.6 us with
// four waves, 17.7 / 19.4 with eight and one / two groups, the second the better one when the line was drawn; 27 with the
// streaming kernel), or four waves where there is one block of rows and so little to load (8 x 5000, 8 heads of head_dim 64,
// window of 32: 9.6 us, 11.6 with eight).  Sixteen blocks or more (head_dim 64) for few keys are a long walk, which the
// streaming kernel divides (300 tokens 7.6 us, 4096 x 16/2 heads 7.8; this form takes 7.0 and 7.3 since its loop was
// shortened, 8.7 and 9.2 before).
// uneven: the sequences may have different numbers of rows, and the launch is more than the chip holds at a group per wave.
struct ImpRowsPlan { int waves, groups; size_t lds; bool uneven; };       // waves == 0: the form does not apply
ImpRowsPlan importance_rows(const pdd_attn_desc *d, int window)
{
    const ImpRowsPlan none = {0, 0, 0, false};
    if (g_imp_keys != 0) return none;
    const int64_t w = (window < 0 || window > d->max_seqlen_q) ? d->max_seqlen_q : window;
    const int64_t blocks = (w * (d->n_q_heads / d->n_kv_heads) + 31) / 32;
    const int64_t lds = blocks * (d->head_dim == 128 ? pdd::importance_rows_block_bytes<128>() : pdd::importance_rows_block_bytes<64>());
    if (lds > kLdsBytes) return none;
    const bool uneven = w == d->max_seqlen_q && (int64_t)d->batch * w != d->total_q && blocks > 1;
    const int64_t tasks = (int64_t)(d->total_k / 32 + d->batch) * d->n_kv_heads, slots = 16 * (int64_t)compute_units();
    if (lds > kLdsBytes / 2) {
        if (tasks < slots) return none;
        const double rounds = (double)d->total_k * d->n_kv_heads / (1024.0 * compute_units());    // with two groups per wave
        const bool two = 1.9 * std::ceil(rounds - 0.05) <= std::ceil(2.0 * rounds - 0.05);
        return {16, two ? 2 : 1, (size_t)lds, uneven};
    }
    if (blocks >= 16 && (int64_t)d->batch * ((d->max_seqlen_k + 31) / 32) * d->n_kv_heads < 2 * compute_units()) return none;
    const int64_t resident = lds > kLdsBytes / 3 ? 2 : lds > kLdsBytes / 4 ? 3 : 4;     // 4-wave workgroups per compute unit
    if (tasks <= 4 * resident * compute_units()) return {4, 1, (size_t)lds, false};
    return {blocks == 1 && tasks >= slots ? 4 : 8, tasks >= slots ? 2 : 1, (size_t)lds, uneven};
}

// What the streaming kernel can use, also where the form above runs and needs none: the figure must not
// change with PDD_OPT_IMPORTANCE_KEYS, which a caller may set after sizing the scratch.
size_t importance_workspace(const pdd_attn_desc *d, int window)
{
    return importance_split_bytes(d, importance_split(d, window));
}

template <typename Kern>
pdd_status launch_importance_rows(Kern kern, pdd::ImpParams &p, const ImpRowsPlan &rows, int max_k, hipStream_t st)
{
    const pdd_status s = raise_lds_limit(reinterpret_cast<const void *>(kern), kLdsBytes);
    if (s) return s;
    const int keys = 32 * rows.waves * rows.groups;
    int64_t pieces = ((int64_t)max_k + keys - 1) / keys * p.B;
    // Sequences of different lengths: only pieces that exist, found by a scan over the lengths (see the kernel; it
    // costs 0.2 us, so only where the workgroups are not all at once on the chip anyway).
    p.scan = p.B <= pdd::kImpScanMax && (int64_t)p.B * max_k != p.total_k && pieces * p.Hkv > compute_units();
    if (p.scan && pieces > p.total_k / keys + p.B) pieces = p.total_k / keys + p.B;
    // Chunks of different lengths, with more keys than one group for every wave of the chip: as many pieces as
    // are on the chip at once (16 waves per compute unit), see the kernel.
    const int64_t places = 16 / rows.waves * (int64_t)compute_units() / p.Hkv;
    p.places = 0;
    if (rows.uneven && p.B <= pdd::kImpScanMax && 4 * p.B <= places) {
        p.scan = 1;
        p.places = (int)places;
        pieces = places;
    }
    const int64_t blocks = pieces * p.Hkv;
    if (blocks > 0x7fffffffLL) return fail(PDD_ERR_INVALID_ARG, "launch grid too large");
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(64 * rows.waves), rows.lds, st, p);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(PDD_ERR_HIP, "importance launch: %s", hipGetErrorString(e));
    return PDD_OK;
}

pdd_status launch_importance(const pdd_attn_desc *d, const void *q, const void *k, const float *lse, float *imp,
                             int window, void *workspace, size_t workspace_bytes, hipStream_t st)
{
    if (d->total_k == 0) return PDD_OK;
    pdd::ImpParams p;
    p.q = (const uint16_t *)q;  p.k = (const uint16_t *)k;  p.lse = lse;  p.imp = imp;
    p.cu_q = d->cu_seqlens_q;  p.cu_k = d->cu_seqlens_k;
    p.q_st = d->q_stride_tok;  p.q_sh = d->q_stride_head;
    p.k_st = d->k_stride_tok;  p.k_sh = d->k_stride_head;
    p.B = d->batch;  p.Hq = d->n_q_heads;  p.Hkv = d->n_kv_heads;  p.G = d->n_q_heads / d->n_kv_heads;
    p.total_q = d->total_q;  p.total_k = d->total_k;
    p.window = window;
    p.g_magic = p.G > 1 ? (uint32_t)(((1ull << 32) + p.G - 1) / p.G) : 0u;
    p.turn = pdd::rows_per_turn(p.Hkv);
    p.scale_log2 = scale_log2(d);
    if (const char *beyond = importance_limits(d)) return fail(PDD_ERR_UNSUPPORTED, "%s", beyond);
    // The row split needs room for its partial sums; where there is less, the rule for even lengths may fit, else the
    // single-pass form runs.  Scratch that has room for that rule's sums but not its alignment is refused whichever form runs;
    // other misaligned scratch is left unused.
    const int even = importance_split_even(d, window);
    const bool aligned = aligned16(workspace);
    if (even > 1 && workspace && workspace_bytes >= importance_split_bytes(d, even) && !aligned)
        return fail(PDD_ERR_WORKSPACE, "workspace must be 16-byte aligned");
    const size_t room = workspace && aligned ? workspace_bytes : 0;
    p.n_split = importance_split(d, window);
    if (importance_split_bytes(d, p.n_split) > room) p.n_split = importance_split_bytes(d, even) > room ? 1 : even;
    const bool split = p.n_split > 1;
    if (const ImpRowsPlan rows = importance_rows(d, window); rows.waves) {
        p.groups = rows.groups;
        // the LDS is sized from max_seqlen_q; a longer sequence of the device array keeps to it
        if (window < 0 || window > d->max_seqlen_q) p.window = d->max_seqlen_q;
        return d->head_dim == 128 ? launch_importance_rows(pdd::importance_rows_kernel<128>, p, rows, d->max_seqlen_k, st)
                                  : launch_importance_rows(pdd::importance_rows_kernel<64>, p, rows, d->max_seqlen_k, st);
    }
    p.part = split ? (float *)workspace : nullptr;
    // Up to four workgroups per compute unit the launch runs with half the keys per workgroup
    // (one 32-key group per wave instead of two): the same blocks of rows per workgroup at half
    // the work per block, and a workgroup's time is mostly its chain of blocks.  Measured against
    // 256 keys: 17 -> 12 us on 4096 tokens x 32 heads (128 workgroups become 256), 42 -> 37 us on
    // the batch of 8 mixed prompts (768 -> 1536), equal on the 32k-token prompt (1024 -> 2048);
    // beyond that the wide form re-reads the window rows half as often.  Same bits either way.
    // (Counted in workgroups that have keys: the grid is sized for the longest sequence.)
    // sequences of different lengths: only slices that exist, see the kernel
    p.scan = p.B <= pdd::kImpScanMax && (int64_t)p.B * d->max_seqlen_k != p.total_k;
    const int64_t working = (int64_t)d->total_k / pdd::kImpBK * d->n_kv_heads * p.n_split;
    const bool narrow = g_imp_keys ? g_imp_keys == pdd::kImpBK / 2 : working <= 4 * (int64_t)compute_units();
    const int keys = narrow ? pdd::kImpBK / 2 : pdd::kImpBK;
    p.n_ktiles = (d->max_seqlen_k + keys - 1) / keys;
    int64_t slices = (int64_t)p.n_ktiles * d->batch;
    if (p.scan && slices > p.total_k / keys + p.B) slices = p.total_k / keys + p.B;
    const int64_t blocks = slices * d->n_kv_heads * p.n_split;
    if (blocks > 0x7fffffffLL) return fail(PDD_ERR_INVALID_ARG, "launch grid too large");
    const dim3 grid((unsigned)blocks), block(pdd::kImpWaves * 64);
    if (d->head_dim == 128) {
        if (narrow) hipLaunchKernelGGL((pdd::importance_kernel<128, 1>), grid, block, 0, st, p);
        else hipLaunchKernelGGL((pdd::importance_kernel<128, 2>), grid, block, 0, st, p);
    } else {
        if (narrow) hipLaunchKernelGGL((pdd::importance_kernel<64, 1>), grid, block, 0, st, p);
        else hipLaunchKernelGGL((pdd::importance_kernel<64, 2>), grid, block, 0, st, p);
    }
    if (split) launch_importance_reduce(p.part, imp, (int64_t)d->n_kv_heads * d->total_k, p.n_split, st);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(PDD_ERR_HIP, "importance launch: %s", hipGetErrorString(e));
    return PDD_OK;
}

// What the chunked call can use: room for the in-kernel sweep where that applies, else for the
// row split of the separate importance kernel.
size_t plain_chunked_workspace(const pdd_attn_desc *d)
{
    const size_t sweep = sweep_workspace(d);
    return sweep ? sweep : importance_workspace(d, -1);
}

// The same with the form of attn_rows.hpp where that applies: its partial rows, and after them, in the
// same place, the partial sums of the importance kernel.
size_t chunked_workspace(const pdd_attn_desc *d)
{
    const RowsPlan rows = rows_plan(d, true, PDD_STATIC_SCRATCH_BYTES);
    if (!rows.rg) return plain_chunked_workspace(d);
    const size_t imp = importance_workspace(d, -1);
    return rows.bytes > imp ? rows.bytes : imp;
}

// The plan of rows_plan for the scratch that a chunked call is given.  Scratch that is too small for the plan it would take
// with all that it asks for still divides the keys, into fewer pieces.
RowsPlan rows_plan_with(const pdd_attn_desc *d, const void *workspace, size_t workspace_bytes)
{
    if (!workspace || !aligned16(workspace)) return rows_plan(d, true, 0);
    const RowsPlan rows = rows_plan(d, true, PDD_STATIC_SCRATCH_BYTES);
    return workspace_bytes >= rows.bytes ? rows : rows_plan(d, true, workspace_bytes);
}

// The forms that the two calls take for their scratch.
AttnForm prefill_form(const pdd_attn_desc *d, const void *workspace, size_t workspace_bytes)
{
    // (a prompt's rows plan takes no scratch; without scratch for the key-split form it is compared with the plain form alone)
    AttnForm f = {0, attn_prefill_rows_per_workgroup(d), split_plan(d), {}};
    const bool room = f.split.tiles && workspace && workspace_bytes >= f.split.bytes && aligned16(workspace);
    f.rows = rows_plan(d, false, room ? workspace_bytes : 0);
    f.kind = f.rows.rg ? PDD_ATTN_ROWS : room ? PDD_ATTN_SPLIT : plain_form(d, f.bm, false);
    return f;
}
// sweeps: there is importance to return, and scratch for the sweep
AttnForm chunk_form(const pdd_attn_desc *d, bool sweeps, const void *workspace, size_t workspace_bytes)
{
    AttnForm f = {0, attn_rows_per_workgroup(d), {}, rows_plan_with(d, workspace, workspace_bytes)};
    f.kind = f.rows.rg ? PDD_ATTN_ROWS : plain_form(d, f.bm, sweeps);
    return f;
}

// Device address of this GPU's copy of `scratch`, looked up once per device.
pdd_status static_scratch(void **out)
{
    static void *ptr[64];
    static bool known[64];
    static std::mutex mu;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(PDD_ERR_HIP, "hipGetDevice: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= 64) return fail(PDD_ERR_UNSUPPORTED, "device ordinal %d beyond 63", dev);
    std::lock_guard<std::mutex> lock(mu);
    if (!known[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) return fail(PDD_ERR_HIP, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
        ptr[dev] = p;
        known[dev] = true;
    }
    *out = ptr[dev];
    return PDD_OK;
}

pdd_status check_ptrs(const void *q, const void *k, const void *v, const void *o, const void *lse)
{
    if (!q || !k || !v || !o || !lse) return fail(PDD_ERR_INVALID_ARG, "NULL tensor pointer");
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o))
        return fail(PDD_ERR_INVALID_ARG, "tensor pointers must be 16-byte aligned");
    if (reinterpret_cast<uintptr_t>(lse) & 3u) return fail(PDD_ERR_INVALID_ARG, "lse must be 4-byte aligned");
    return PDD_OK;
}

}  // namespace

extern "C" {

const char *pdd_last_error(void) { return g_err; }
const char *pdd_version(void) { return "pdd 0.1 gfx950"; }

pdd_status pdd_set_option(int option, int value)
{
    if (option == PDD_OPT_ATTN_WAVES) {
        if (value != 0 && value != 4 && value != 8) return fail(PDD_ERR_INVALID_ARG, "attn waves must be 0, 4 or 8");
        g_attn_waves = value;
        return PDD_OK;
    }
    if (option == PDD_OPT_IMPORTANCE_KEYS) {
        if (value != 0 && value != pdd::kImpBK / 2 && value != pdd::kImpBK)
            return fail(PDD_ERR_INVALID_ARG, "importance keys per workgroup must be 0, 128 or 256");
        g_imp_keys = value;
        return PDD_OK;
    }
    return fail(PDD_ERR_INVALID_ARG, "unknown option %d", option);
}

size_t pdd_workspace_bytes(const pdd_attn_desc *desc, int which_call)
{
    if (!desc || desc->batch < 1 || desc->n_kv_heads < 1) return 0;
    if (which_call == PDD_CALL_SELECT_TOPK)         // the attention fields are not read
        return select_workspace(desc->n_kv_heads, desc->batch, select_chunks(desc->n_kv_heads, desc->batch, desc->max_seqlen_k));
    if (desc->n_q_heads < desc->n_kv_heads || desc->total_k < 0) return 0;
    switch (which_call) {
    case PDD_CALL_PREFILL_ATTN:
    {
        const size_t imp = desc->window > 0 ? importance_workspace(desc, desc->window) : 0;
        const size_t split = split_plan(desc).bytes;      // (also where a form of attn_rows.hpp needs none)
        return split > imp ? split : imp;
    }
    case PDD_CALL_PREFILL_ATTN_CHUNKED:
        return chunked_workspace(desc);
    case PDD_CALL_TOKEN_IMPORTANCE:
        return desc->window != 0 ? importance_workspace(desc, desc->window) : 0;
    default:
        return 0;
    }
}

int pdd_attn_form(const pdd_attn_desc *desc, int which_call, int importance, size_t workspace_bytes)
{
    if (which_call != PDD_CALL_PREFILL_ATTN && which_call != PDD_CALL_PREFILL_ATTN_CHUNKED) {
        fail(PDD_ERR_INVALID_ARG, "pdd_attn_form: not an attention call: %d", which_call);
        return PDD_ERR_INVALID_ARG;
    }
    const bool chunked = which_call == PDD_CALL_PREFILL_ATTN_CHUNKED;
    if (const pdd_status s = check_desc(desc, chunked ? MODE_CHUNKED : MODE_PREFILL)) return s;
    const void *scratch = workspace_bytes ? reinterpret_cast<const void *>(uintptr_t(16)) : nullptr;      // (not followed)
    if (!chunked) return prefill_form(desc, scratch, workspace_bytes).kind;
    const size_t sweep = importance ? sweep_workspace(desc) : 0;
    return chunk_form(desc, sweep && workspace_bytes >= sweep, scratch, workspace_bytes).kind;
}

pdd_status pdd_prefill_attn(const pdd_attn_desc *desc, const void *q, const void *k, const void *v, void *o,
                            float *lse, float *importance, void *workspace, size_t workspace_bytes,
                            pdd_stream stream)
{
    pdd_status s = check_desc(desc, MODE_PREFILL);
    if (s) return s;
    s = check_ptrs(q, k, v, o, lse);
    if (s) return s;
    if (desc->window > 0 && !importance)
        return fail(PDD_ERR_INVALID_ARG, "window > 0 needs an importance buffer");
    s = launch_attn(desc, prefill_form(desc, workspace, workspace_bytes), q, k, v, o, lse, (hipStream_t)stream, nullptr, workspace);
    if (s) return s;
    if (importance && desc->window > 0)
        return launch_importance(desc, q, k, lse, importance, desc->window, workspace, workspace_bytes,
                                 (hipStream_t)stream);
    return PDD_OK;
}

pdd_status pdd_prefill_attn_chunked(const pdd_attn_desc *desc, const void *q_chunk, const void *k_all,
                                    const void *v_all, void *o, float *lse, float *importance, void *workspace,
                                    size_t workspace_bytes, pdd_stream stream)
{
    pdd_status s = check_desc(desc, MODE_CHUNKED);
    if (s) return s;
    s = check_ptrs(q_chunk, k_all, v_all, o, lse);
    if (s) return s;
    // Scratch that has room for the sweep but not its alignment is refused whichever form runs.
    const size_t sweep = importance ? sweep_workspace(desc) : 0;
    const bool sweeps = sweep && workspace && workspace_bytes >= sweep;
    if (sweeps && !aligned16(workspace)) return fail(PDD_ERR_WORKSPACE, "workspace must be 16-byte aligned");
    const AttnForm form = chunk_form(desc, sweeps, workspace, workspace_bytes);
    if (sweeps && form.kind != PDD_ATTN_ROWS) {
        s = launch_attn(desc, form, q_chunk, k_all, v_all, o, lse, (hipStream_t)stream, (float *)workspace, nullptr);
        if (s) return s;
        const int n_slices = (desc->n_q_heads / desc->n_kv_heads) * ((desc->max_seqlen_q + form.bm - 1) / form.bm);
        launch_importance_reduce((const float *)workspace, importance, (int64_t)desc->n_kv_heads * desc->total_k,
                                 n_slices, (hipStream_t)stream);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return fail(PDD_ERR_HIP, "importance reduction launch: %s", hipGetErrorString(e));
        return PDD_OK;
    }
    s = launch_attn(desc, form, q_chunk, k_all, v_all, o, lse, (hipStream_t)stream, nullptr, workspace);
    if (s) return s;
    if (importance)
        return launch_importance(desc, q_chunk, k_all, lse, importance, -1, workspace, workspace_bytes,
                                 (hipStream_t)stream);
    return PDD_OK;
}

pdd_status pdd_prefill_attn_chunked_noalloc(const pdd_attn_desc *desc, const void *q_chunk, const void *k_all,
                                            const void *v_all, void *o, float *lse, float *importance,
                                            pdd_stream stream)
{
    pdd_status s = check_desc(desc, MODE_CHUNKED);
    if (s) return s;
    // Attention alone needs no scratch, so it takes none of the shared one: such calls may overlap.
    if (!importance) return pdd_prefill_attn_chunked(desc, q_chunk, k_all, v_all, o, lse, nullptr, nullptr, 0, stream);
    const size_t sweep = sweep_workspace(desc), plain = sweep ? sweep : importance_split_bytes(desc, importance_split_even(desc, -1));
    if (plain > PDD_STATIC_SCRATCH_BYTES)
        return fail(PDD_ERR_WORKSPACE, "this shape wants %zu bytes of scratch, the built-in scratch holds %u "
                    "(use pdd_prefill_attn_chunked with a workspace)", plain, (unsigned)PDD_STATIC_SCRATCH_BYTES);
    // (the forms of attn_rows.hpp never want more than the built-in scratch)
    const size_t need = chunked_workspace(desc);
    void *ws = nullptr;
    if (need > 0) {
        s = static_scratch(&ws);
        if (s) return s;
    }
    return pdd_prefill_attn_chunked(desc, q_chunk, k_all, v_all, o, lse, importance, ws, need, stream);
}

pdd_status pdd_token_importance(const pdd_attn_desc *desc, const void *q, const void *k, const float *lse,
                                float *importance, void *workspace, size_t workspace_bytes, pdd_stream stream)
{
    pdd_status s = check_desc(desc, MODE_IMPORTANCE);
    if (s) return s;
    if (!q || !k || !lse || !importance) return fail(PDD_ERR_INVALID_ARG, "NULL tensor pointer");
    if (!aligned16(q) || !aligned16(k)) return fail(PDD_ERR_INVALID_ARG, "tensor pointers must be 16-byte aligned");
    return launch_importance(desc, q, k, lse, importance, desc->window, workspace, workspace_bytes,
                             (hipStream_t)stream);
}

pdd_status pdd_select_topk_pooled(const float *scores, int32_t n_heads, int32_t batch, int32_t total_k,
                                  const int32_t *cu_seqlens_k, const int32_t *cu_seqlens_k_host,
                                  int32_t max_seqlen_k, const int32_t *cand_begin, const int32_t *cand_end,
                                  const int32_t *k_per_seq, const int32_t *cu_keep, int32_t total_keep,
                                  int32_t pool_kernel, int32_t pool_mode, float *pooled_out,
                                  int32_t *out_indices, uint8_t *out_mask, void *workspace,
                                  size_t workspace_bytes, pdd_stream stream)
{
    if (!scores || !cu_seqlens_k || !k_per_seq || !cu_keep) return fail(PDD_ERR_INVALID_ARG, "NULL pointer");
    if (n_heads < 1 || batch < 1) return fail(PDD_ERR_INVALID_ARG, "n_heads and batch must be >= 1");
    if (total_k < 0 || total_keep < 0 || max_seqlen_k < 0 || max_seqlen_k > total_k)
        return fail(PDD_ERR_INVALID_ARG, "bad sizes");
    if (total_keep > 0 && !out_indices) return fail(PDD_ERR_INVALID_ARG, "out_indices is NULL");
    if ((cand_begin == nullptr) != (cand_end == nullptr))
        return fail(PDD_ERR_INVALID_ARG, "cand_begin and cand_end must both be given or both be NULL");
    if (batch > 65535 * 32) return fail(PDD_ERR_INVALID_ARG, "batch too large");
    if (n_heads > 65535) return fail(PDD_ERR_INVALID_ARG, "n_heads too large");
    if (pool_mode != PDD_POOL_NONE && pool_mode != PDD_POOL_MAX && pool_mode != PDD_POOL_AVG)
        return fail(PDD_ERR_INVALID_ARG, "unknown pool_mode %d", pool_mode);
    if (pool_mode != PDD_POOL_NONE && (pool_kernel < 1 || pool_kernel % 2 == 0 || pool_kernel > 1025))
        return fail(PDD_ERR_INVALID_ARG, "pool_kernel must be odd and in [1, 1025]");
    pdd_status s = check_cu_host("cu_seqlens_k_host", cu_seqlens_k_host, batch, total_k, max_seqlen_k);
    if (s) return s;
    if (total_k == 0) return PDD_OK;

    pdd::SelParams p;
    p.scores = scores;  p.cu_k = cu_seqlens_k;  p.cand_b = cand_begin;  p.cand_e = cand_end;
    p.k_per = k_per_seq;  p.cu_keep = cu_keep;  p.out_idx = out_indices;  p.out_mask = out_mask;
    p.n_heads = n_heads;  p.B = batch;  p.total_k = total_k;  p.total_keep = total_keep;
    p.pool_r = pool_mode == PDD_POOL_NONE ? 0 : (pool_kernel - 1) / 2;
    p.pool_mode = pool_mode == PDD_POOL_MAX ? pdd::kPoolMax : pdd::kPoolAvg;
    p.pool_inv = pool_mode == PDD_POOL_AVG ? 1.0f / (float)pool_kernel : 1.0f;
    p.pooled_out = pooled_out;
    const dim3 grid((unsigned)batch, (unsigned)n_heads);
    hipStream_t st = (hipStream_t)stream;
    const int chunks = p.pool_r == 0 ? select_chunks(n_heads, batch, max_seqlen_k) : 0;
    if (chunks && workspace && aligned16(workspace) &&
        workspace_bytes >= select_workspace(n_heads, batch, chunks))
        return launch_select_split(p, chunks, workspace, st);
    // rows of up to 32768 candidates stay in registers (4096 per step and 1024 threads)
    if (max_seqlen_k <= 4 * pdd::kSelThreads)
        launch_select_reg<1>(p, grid, st);
    else if (max_seqlen_k <= 8 * pdd::kSelThreads)
        launch_select_reg<2>(p, grid, st);
    else if (max_seqlen_k <= 16 * pdd::kSelThreads)
        launch_select_reg<4>(p, grid, st);
    else if (max_seqlen_k <= 32 * pdd::kSelThreads)
        launch_select_reg<8>(p, grid, st);
    else
        hipLaunchKernelGGL(pdd::select_topk_kernel, grid, dim3(pdd::kSelThreads), 0, st, p);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(PDD_ERR_HIP, "select launch: %s", hipGetErrorString(e));
    return PDD_OK;
}

pdd_status pdd_select_topk(const float *scores, int32_t n_heads, int32_t batch, int32_t total_k,
                           const int32_t *cu_seqlens_k, const int32_t *cu_seqlens_k_host, int32_t max_seqlen_k,
                           const int32_t *cand_begin, const int32_t *cand_end, const int32_t *k_per_seq,
                           const int32_t *cu_keep, int32_t total_keep, int32_t *out_indices, uint8_t *out_mask,
                           void *workspace, size_t workspace_bytes, pdd_stream stream)
{
    return pdd_select_topk_pooled(scores, n_heads, batch, total_k, cu_seqlens_k, cu_seqlens_k_host, max_seqlen_k,
                                  cand_begin, cand_end, k_per_seq, cu_keep, total_keep, 1, PDD_POOL_NONE, nullptr,
                                  out_indices, out_mask, workspace, workspace_bytes, stream);
}

pdd_status pdd_select_sentences(const float *scores, int32_t n_heads, int32_t batch, int32_t total_k,
                                const int32_t *cu_seqlens_k, const int32_t *cu_seqlens_k_host, int32_t max_seqlen_k,
                                const int32_t *cu_sent, const int32_t *sent_end, int32_t total_sent,
                                int32_t max_sent_per_seq, const int32_t *cand_begin, const int32_t *token_budget,
                                int32_t agg_mode, float *out_sent_scores, uint8_t *out_sent_keep,
                                uint8_t *out_mask, int32_t *out_kept_tokens, pdd_stream stream)
{
    if (!scores || !cu_seqlens_k || !cu_sent || !token_budget) return fail(PDD_ERR_INVALID_ARG, "NULL pointer");
    if (total_sent > 0 && !sent_end) return fail(PDD_ERR_INVALID_ARG, "sent_end is NULL");
    if (n_heads < 1 || batch < 1) return fail(PDD_ERR_INVALID_ARG, "n_heads and batch must be >= 1");
    if (total_k < 0 || total_sent < 0 || max_seqlen_k < 0 || max_seqlen_k > total_k || max_sent_per_seq < 0 ||
        max_sent_per_seq > total_sent)
        return fail(PDD_ERR_INVALID_ARG, "bad sizes");
    if (max_sent_per_seq > pdd::kSentMax)
        return fail(PDD_ERR_UNSUPPORTED, "more than %d sentences in one sequence", pdd::kSentMax);
    if (agg_mode != PDD_SENT_SUM && agg_mode != PDD_SENT_MEAN) return fail(PDD_ERR_INVALID_ARG, "unknown agg_mode");
    if (batch > 65535 * 32 || n_heads > 65535) return fail(PDD_ERR_INVALID_ARG, "batch or n_heads too large");
    pdd_status s = check_cu_host("cu_seqlens_k_host", cu_seqlens_k_host, batch, total_k, max_seqlen_k);
    if (s) return s;
    if (total_k == 0) return PDD_OK;
    pdd::SentParams p;
    p.scores = scores;  p.cu_k = cu_seqlens_k;  p.cu_sent = cu_sent;  p.sent_end = sent_end;
    p.cand_b = cand_begin;  p.budget = token_budget;  p.sent_keep = out_sent_keep;  p.mask = out_mask;
    p.kept_tokens = out_kept_tokens;  p.sent_scores = out_sent_scores;
    p.n_heads = n_heads;  p.B = batch;  p.total_k = total_k;  p.total_sent = total_sent;
    p.s_cap = max_sent_per_seq > 0 ? ((max_sent_per_seq + 3) & ~3) : 4;
    p.mode = agg_mode == PDD_SENT_MEAN ? pdd::kSentMean : pdd::kSentSum;
    const int step = 4 * pdd::kSelThreads;
    p.seg = max_seqlen_k >= pdd::kSentSeg ? pdd::kSentSeg : (max_seqlen_k / step + 1) * step;
    const int smem = p.seg * (int)sizeof(float);
    s = raise_lds_limit(reinterpret_cast<const void *>(pdd::select_sentences_kernel), pdd::kSentSeg * (int)sizeof(float));
    if (s) return s;
    hipError_t e;
    hipLaunchKernelGGL(pdd::select_sentences_kernel, dim3((unsigned)batch, (unsigned)n_heads),
                       dim3(pdd::kSelThreads), smem, (hipStream_t)stream, p);
    e = hipGetLastError();
    if (e != hipSuccess) return fail(PDD_ERR_HIP, "sentence select launch: %s", hipGetErrorString(e));
    return PDD_OK;
}

pdd_status pdd_aggregate_scores(const float *scores, int32_t n_layers, int32_t n_heads, int32_t total_k,
                                int64_t layer_stride, const float *layer_weights, int32_t reduce_heads,
                                int32_t accumulate, float *out, pdd_stream stream)
{
    if (!scores || !out) return fail(PDD_ERR_INVALID_ARG, "NULL pointer");
    if (n_layers < 1 || n_heads < 1 || n_heads > 65535 || total_k < 0)
        return fail(PDD_ERR_INVALID_ARG, "bad sizes");
    if (layer_stride < (int64_t)n_heads * total_k)
        return fail(PDD_ERR_INVALID_ARG, "layer_stride smaller than n_heads * total_k");
    if (total_k == 0) return PDD_OK;
    pdd::AggParams p;
    p.scores = scores;  p.weights = layer_weights;  p.out = out;  p.layer_stride = layer_stride;
    p.n_layers = n_layers;  p.n_heads = n_heads;  p.total_k = total_k;
    p.reduce_heads = reduce_heads ? 1 : 0;  p.accumulate = accumulate ? 1 : 0;
    // Four tokens per lane, fewer where a row is too short to occupy every compute unit that way;
    // then waves that share the layers until there are 16 per compute unit (32 layers x 8 heads x
    // 32768 tokens into one row: 256 workgroups of 2 tokens per lane and 16 waves).
    const int64_t rows = reduce_heads ? 1 : n_heads, cus = compute_units();
    auto groups = [&](int v) { return ((total_k + 64LL * v - 1) / (64 * v)) * rows; };
    const int vec = groups(4) >= cus ? 4 : groups(2) >= cus ? 2 : 1;
    p.share_log2 = 0;
    while ((2 << p.share_log2) <= pdd::kAggMaxWaves && (2 << p.share_log2) <= n_layers && (groups(vec) << p.share_log2) < 16 * cus)
        ++p.share_log2;
    const int waves = (1 << p.share_log2) > pdd::kAggMinWaves ? 1 << p.share_log2 : pdd::kAggMinWaves;
    const int64_t tokens = 64LL * vec * (waves >> p.share_log2);        // of a workgroup
    const dim3 grid((unsigned)((total_k + tokens - 1) / tokens), (unsigned)rows), block(64 * waves);
    // Loads in flight: eight per wave where waves are few; where they fill every compute unit by
    // themselves that queues at the memory: two from 16 waves per compute unit on (32 layers x 8 heads x
    // 131072, 16 waves: 20.4 us against 25.0 with eight and 22.7 with one; x 1048576 into one row 161 against
    // 206), one from 32 on (32 layers x 2 heads x 1048576, 32 waves: 39.5 us against 43.6 with two; 32 x 8 per head,
    // 128 waves: 184 against 207 with two and 197 with eight).
    hipStream_t st = (hipStream_t)stream;
    const int smem = p.share_log2 > 0 ? waves * 64 * vec * (int)sizeof(float) : 0;
    if (p.share_log2 == 0 && groups(4) >= 32 * cus)      hipLaunchKernelGGL((pdd::aggregate_scores_kernel<4, 1>), grid, block, smem, st, p);
    else if (p.share_log2 == 0 && groups(4) >= 16 * cus) hipLaunchKernelGGL((pdd::aggregate_scores_kernel<4, 2>), grid, block, smem, st, p);
    else if (vec == 4) hipLaunchKernelGGL((pdd::aggregate_scores_kernel<4, 8>), grid, block, smem, st, p);
    else if (vec == 2) hipLaunchKernelGGL((pdd::aggregate_scores_kernel<2, 8>), grid, block, smem, st, p);
    else               hipLaunchKernelGGL((pdd::aggregate_scores_kernel<1, 8>), grid, block, smem, st, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(PDD_ERR_HIP, "aggregate launch: %s", hipGetErrorString(e));
    return PDD_OK;
}

/* Host-only scalar code: the closed form of the program that picks (r, L). */
pdd_status pdd_choose_r_L(const pdd_rl_model *m, int32_t l, double *r_out, int32_t *L_out)
{
    if (!m || !r_out || !L_out) return fail(PDD_ERR_INVALID_ARG, "NULL pointer");
    if (l < 1) return fail(PDD_ERR_INVALID_ARG, "prompt length must be >= 1");
    if (!(m->k_c >= 0) || !(m->k_d > 0) || !(m->delta >= 0) || !(m->tpot_c > 0) || !(m->tpot_d > 0) ||
        !(m->xi_scene >= 0 && m->xi_scene <= 1))
        return fail(PDD_ERR_INVALID_ARG, "model coefficients out of range");
    if (!(m->delta_cloud >= 0 && m->delta_cloud <= m->delta))
        return fail(PDD_ERR_INVALID_ARG, "delta_cloud must lie in [0, delta]");
    if (!(m->tau > m->tpot_d)) return fail(PDD_ERR_INFEASIBLE, "tau must exceed the device TPOT");
    const double len = (double)l;
    /* In terms of x = k_d*r*l (device prefill time of the refined prompt) and n = L - 1 >= 1:
     *   Eq. 5: x_min = k_d*xi*l <= x <= x_max = k_d*l - k_c*l - delta
     *   Eq. 6: n*tpot_c - (delta - delta_cloud) <= x <= n*(tau - tpot_d) + TTFT_c
     * The objective grows with x.  Below n0 = the smallest n whose upper bound reaches x_min
     * nothing is feasible; from n0 on the lower bound only grows with n, so the optimum is
     * n0 with x = max(x_min, n0*tpot_c - decompress), if that still respects both upper bounds. */
    const double ttft_c = m->k_c * len + m->delta_cloud;          /* prefill + compress + RTT */
    const double decompress = m->delta - m->delta_cloud;
    const double a = m->tau - m->tpot_d;
    const double x_min = m->k_d * m->xi_scene * len;
    const double x_max = m->k_d * len - m->k_c * len - m->delta;
    if (x_min > x_max) return fail(PDD_ERR_INFEASIBLE, "no ratio in [xi_scene, %.6g]", x_max / (m->k_d * len));
    double n0 = std::ceil((x_min - ttft_c) / a);
    if (n0 < 1.0) n0 = 1.0;
    if (n0 > 2147483646.0) return fail(PDD_ERR_INFEASIBLE, "L out of range");
    double x = n0 * m->tpot_c - decompress;
    double r = x / (m->k_d * len);
    if (x <= x_min) { x = x_min; r = m->xi_scene; }
    if (x > x_max || x > n0 * a + ttft_c)
        return fail(PDD_ERR_INFEASIBLE, "no (r, L): L - 1 = %.0f needs a device prefill of %.6g, allowed at most %.6g",
                    n0, x, x_max < n0 * a + ttft_c ? x_max : n0 * a + ttft_c);
    const double lm1 = n0;
    *r_out = r;
    *L_out = (int32_t)lm1 + 1;
    return PDD_OK;
}

int64_t pdd_pack_mask_layout(int32_t batch, const int32_t *cu_seqlens_k_host, int32_t *cu_bytes_host)
{
    if (batch < 1 || !cu_seqlens_k_host || !cu_bytes_host) {
        fail(PDD_ERR_INVALID_ARG, "pdd_pack_mask_layout: bad arguments");
        return -1;
    }
    int64_t total = 0;
    cu_bytes_host[0] = 0;
    for (int b = 0; b < batch; ++b) {
        const int64_t nk = (int64_t)cu_seqlens_k_host[b + 1] - cu_seqlens_k_host[b];
        if (nk < 0) {
            fail(PDD_ERR_INVALID_ARG, "pdd_pack_mask_layout: cu_seqlens_k_host decreases at %d", b);
            return -1;
        }
        total += (nk + 7) / 8;
        if (total > 0x7fffffffLL) {
            fail(PDD_ERR_INVALID_ARG, "pdd_pack_mask_layout: more than 2^31 bytes per row");
            return -1;
        }
        cu_bytes_host[b + 1] = (int32_t)total;
    }
    return total;
}

pdd_status pdd_pack_mask(const uint8_t *mask, int32_t n_rows, int32_t batch, int32_t total_k,
                         const int32_t *cu_seqlens_k, const int32_t *cu_seqlens_k_host, int32_t max_seqlen_k,
                         const int32_t *cu_bytes, int32_t total_bytes, uint8_t *out_bits, pdd_stream stream)
{
    if (!mask || !cu_seqlens_k || !cu_bytes) return fail(PDD_ERR_INVALID_ARG, "NULL pointer");
    if (n_rows < 1 || batch < 1) return fail(PDD_ERR_INVALID_ARG, "n_rows and batch must be >= 1");
    if (total_k < 0 || total_bytes < 0 || max_seqlen_k < 0 || max_seqlen_k > total_k)
        return fail(PDD_ERR_INVALID_ARG, "bad sizes");
    if (total_bytes > 0 && !out_bits) return fail(PDD_ERR_INVALID_ARG, "out_bits is NULL");
    if (batch > 65535 || n_rows > 65535) return fail(PDD_ERR_INVALID_ARG, "batch or n_rows too large");
    pdd_status s = check_cu_host("cu_seqlens_k_host", cu_seqlens_k_host, batch, total_k, max_seqlen_k);
    if (s) return s;
    if (total_k == 0 || total_bytes == 0) return PDD_OK;
    pdd::PackParams p;
    p.mask = mask;  p.bits = out_bits;  p.cu_k = cu_seqlens_k;  p.cu_bytes = cu_bytes;
    p.rows = n_rows;  p.B = batch;  p.total_k = total_k;  p.total_bytes = total_bytes;
    const int max_bytes = (max_seqlen_k + 7) / 8;
    const unsigned gx = (unsigned)((max_bytes + pdd::kPackThreads - 1) / pdd::kPackThreads);
    hipLaunchKernelGGL(pdd::pack_mask_kernel, dim3(gx, (unsigned)batch, (unsigned)n_rows), dim3(pdd::kPackThreads), 0,
                       (hipStream_t)stream, p);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(PDD_ERR_HIP, "pack launch: %s", hipGetErrorString(e));
    return PDD_OK;
}

}  // extern "C"
