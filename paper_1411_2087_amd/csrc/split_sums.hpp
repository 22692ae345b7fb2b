// Sums of the kernels that give a 64-site tile to a workgroup (SplitTerms).
#pragma once

#include "dslash_core.hpp"

namespace hisq {

// v of another lane of the row of 16, by a DPP control
template <int CTRL> __device__ __forceinline__ double dpp_lane(double v)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double read_lane(double v, int l)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                            __builtin_amdgcn_readlane(__double2loint(v), l));
}
// Sum over the wavefront, the same in every lane and in a fixed order: the
// rows of 16 by DPP (neighbour, pair, half row, row), then the four rows.  The
// sums are on the critical path of kernels of a few microseconds, and the six
// cross-lane round trips through LDS of wave_sum are most of 1 us.
__device__ __forceinline__ double wave_sum_dpp(double v)
{
    v += dpp_lane<0xB1>(v);   // quad_perm 1 0 3 2
    v += dpp_lane<0x4E>(v);   // quad_perm 2 3 0 1
    v += dpp_lane<0x141>(v);  // row_half_mirror
    v += dpp_lane<0x140>(v);  // row_mirror
    return (read_lane(v, 0) + read_lane(v, 16)) + (read_lane(v, 32) + read_lane(v, 48));
}
// Sum over the workgroup, to every thread, in a fixed order.
__device__ __forceinline__ double split_total(double v, double *lds)
{
    v = wave_sum_dpp(v);
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < SPLIT; ++i) s += lds[i];
    return s;
}
// This tile's partial: only the TILE_REALS threads of the first wavefronts hold a value.
__device__ __forceinline__ void split_partial(double v, double *lds, double *out)
{
    constexpr int W = TILE_REALS / TILE;
    if (threadIdx.x < TILE_REALS) {
        v = wave_sum_dpp(v);
        if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < W; ++i) s += lds[i];
        *out = s;
    }
}

}  // namespace hisq
