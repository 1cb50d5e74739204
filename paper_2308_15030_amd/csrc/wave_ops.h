// Reductions over the 64 lanes of a wavefront, shared by the kernels of libswapmoe.
#pragma once

#include <hip/hip_runtime.h>

// Reductions over the 16 lanes of a row by rotations within it (data-parallel primitives: one vector
// instruction each, no trip through the LDS crossbar).  Every lane ends up with the result; the order
// of the additions is the same in all of them up to commutation, so a sum has the same bits in every lane.
template <int N>
__device__ __forceinline__ int smoe_row_ror(int v) { return __builtin_amdgcn_update_dpp(v, v, 0x120 + N, 0xf, 0xf, false); }
template <int N>
__device__ __forceinline__ float smoe_row_ror(float v) { return __int_as_float(smoe_row_ror<N>(__float_as_int(v))); }

__device__ __forceinline__ float smoe_row_max(float v) {
    v = fmaxf(v, smoe_row_ror<8>(v));
    v = fmaxf(v, smoe_row_ror<4>(v));
    v = fmaxf(v, smoe_row_ror<2>(v));
    return fmaxf(v, smoe_row_ror<1>(v));
}
__device__ __forceinline__ int smoe_row_min(int v) {
    v = min(v, smoe_row_ror<8>(v));
    v = min(v, smoe_row_ror<4>(v));
    v = min(v, smoe_row_ror<2>(v));
    return min(v, smoe_row_ror<1>(v));
}
__device__ __forceinline__ float smoe_row_sum(float v) {
    v += smoe_row_ror<8>(v);
    v += smoe_row_ror<4>(v);
    v += smoe_row_ror<2>(v);
    return v + smoe_row_ror<1>(v);
}

// Inclusive prefix sum over the 64 lanes of a wave, all of them active: shifts within the rows of 16 lanes, then the rows'
// totals, six vector additions without a trip through the LDS crossbar.
__device__ __forceinline__ int smoe_wave_incl_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // the last lane of rows 0 and 2 to the rows behind them
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // lane 31 to the upper half
    return v;
}
