// Prefix sum over a wave, for the kernels that place what their lanes or sequences hold.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pdd {

// inclusive prefix sum over the 64 lanes of a wave (DPP row shifts and row broadcasts)
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t x)
{
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, true);   // row_shr:1
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, true);   // row_shr:2
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, true);   // row_shr:4
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, true);   // row_shr:8
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1, 3
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2, 3
    return x;
}

// the same over N independent values per lane, one step over all of them at a time: consecutive
// instructions are independent, so none of them waits for the DPP hazard of its predecessor
template <int N>
__device__ __forceinline__ void wave_incl_scan_n(uint32_t (&x)[N])
{
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x[i], 0x111, 0xf, 0xf, true);
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x[i], 0x112, 0xf, 0xf, true);
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x[i], 0x114, 0xf, 0xf, true);
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x[i], 0x118, 0xf, 0xf, true);
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x[i], 0x142, 0xa, 0xf, false);
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x[i], 0x143, 0xc, 0xf, false);
}

}  // namespace pdd
