// Fixed-order workgroup reduction shared by the bias kernels.
#pragma once
#include "sx_internal.h"

namespace sx {

// x + the value of the lane with bit 5, 4, .. 0 of its number flipped: the
// butterfly of __shfl_xor(x, 32), 16, .. 1 with its bits (each step's two
// sums are the same two values), without its trips through LDS (two reads and
// ~100 cycles a step).  The halves and 16-lane rows are exchanged by
// v_permlane32_swap and v_permlane16_swap; once lanes 8 apart agree, rotating
// a row by 4 reaches the value 4 lanes away.  Every lane of the wavefront must
// take part.  256 walkers' tiles 13.4 us with the shuffles, 12.9 with this;
// one tile's step 4.9 and 4.6; ABF's solve 4.8 and 4.3.  The pair kernel of the
// all-pairs coordination numbers keeps its shuffles: 10.3 us, 10.6 with this.
template <int CTRL>
__device__ __forceinline__ double dpp_lane(double x)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}

__device__ __forceinline__ double wave_sum(double x)
{
    {
        const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(x), __double2loint(x), false, false);
        const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(x), __double2hiint(x), false, false);
        x = __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
    }
    {
        const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(x), __double2loint(x), false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(x), __double2hiint(x), false, false);
        x = __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
    }
    x += dpp_lane<0x128>(x);  // row_ror:8
    x += dpp_lane<0x124>(x);  // row_ror:4
    x += dpp_lane<0x4E>(x);   // quad_perm [2, 3, 0, 1]
    x += dpp_lane<0xB1>(x);   // quad_perm [1, 0, 3, 2]
    return x;
}

// The sum over each 16 lanes, in the order 1, 2, 4, 8 of __shfl_xor and with
// its bits (once the lanes of a quad agree, mirroring eight lanes reaches the
// value 4 lanes away).  A training step's kernel 11.6 us with shuffles, 11.45
// with this.
template <int CTRL>
__device__ __forceinline__ float dpp_lane(float x)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, false));
}

__device__ __forceinline__ float row16_sum(float x)
{
    x += dpp_lane<0xB1>(x);   // quad_perm [1, 0, 3, 2]
    x += dpp_lane<0x4E>(x);   // quad_perm [2, 3, 0, 1]
    x += dpp_lane<0x141>(x);  // row_half_mirror
    x += dpp_lane<0x128>(x);  // row_ror:8
    return x;
}

// Sum N doubles over a workgroup of kBlock threads: a butterfly inside each
// wavefront, then the wavefronts in index order (the same order whatever
// the schedule); the result is in thread 0.  Ends with a barrier, so lds
// may be reused right after.
template <int N>
__device__ __forceinline__ void block_sum0(double (&v)[N], double *lds /* N * kBlock/64 */)
{
    // fixed tree: wave butterfly, then waves in index order; result in thread 0
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] = wave_sum(v[k]);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0)
#pragma unroll
        for (int k = 0; k < N; ++k) lds[wv * N + k] = v[k];
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < N; ++k) {
            double s = lds[k];
            for (int q = 1; q < kBlock / 64; ++q) s += lds[q * N + k];
            v[k] = s;
        }
    }
    __syncthreads();
}

}  // namespace sx
