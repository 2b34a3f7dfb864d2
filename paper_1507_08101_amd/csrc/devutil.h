// devutil.h -- small device helpers shared by the kernels of libsellcs.
#pragma once

#include <hip/hip_runtime.h>

namespace sellcs {

// Workgroup id -> position, so that XCD x (the hardware deals workgroups x, x+8, x+16, ... to it)
// works on one contiguous eighth of the positions: neighbouring rows share its L2.
__device__ __forceinline__ int xcd_block(int bid, int nblocks) {
    const int q = nblocks >> 3, r = nblocks & 7;
    const int x = bid & 7, k = bid >> 3;
    return (x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q) + k;
}

// One 64-bit value moved across the lanes of a wave in registers (two 32-bit moves).
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
    int w[2];
    __builtin_memcpy(w, &v, 8);
    w[0] = __builtin_amdgcn_update_dpp(0, w[0], CTRL, 0xf, 0xf, true);
    w[1] = __builtin_amdgcn_update_dpp(0, w[1], CTRL, 0xf, 0xf, true);
    __builtin_memcpy(&v, w, 8);
    return v;
}

// v of the lane 16 (ROWS = 1) or 32 (ROWS = 2) lanes away added to the lane's own. The swap
// exchanges the odd rows of one register with the even rows of another; with both holding v, each
// lane finds its own and the other row's value in the pair.
template <int ROWS>
__device__ __forceinline__ double add_rows(double v) {
    unsigned w[2], a[2], b[2];
    __builtin_memcpy(w, &v, 8);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const auto r = ROWS == 1 ? __builtin_amdgcn_permlane16_swap(w[h], w[h], false, false)
                                 : __builtin_amdgcn_permlane32_swap(w[h], w[h], false, false);
        a[h] = r[0];
        b[h] = r[1];
    }
    double x, y;
    __builtin_memcpy(&x, a, 8);
    __builtin_memcpy(&y, b, 8);
    return x + y;
}

// Sum over the lanes of a full wave that are congruent to this one modulo VL (a power of two, the
// same in all lanes), in a fixed order, by register moves: no LDS traffic, which in a workgroup's
// closing reductions (up to a dozen values per lane in every wave) was most of their time. Lanes
// of one class may differ in the last bits; callers take lanes 0 .. VL - 1.
__device__ __forceinline__ double class_sum(double v, int VL) {
    if (VL <= 1) v += dpp_move<0x121>(v);  // rows of 16 lanes rotated by 1, 2, 4 and 8
    if (VL <= 2) v += dpp_move<0x122>(v);
    if (VL <= 4) v += dpp_move<0x124>(v);
    if (VL <= 8) v += dpp_move<0x128>(v);
    if (VL <= 16) v = add_rows<1>(v);
    if (VL <= 32) v = add_rows<2>(v);
    return v;
}

// Sum of one value per thread of a 256-thread workgroup in a fixed order: inside each wave, then
// the four wave sums in order. The result is valid in thread 0.
__device__ __forceinline__ double block_sum_256(double v) {
    __shared__ double ws[4];
    v = class_sum(v, 1);
    if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x == 0) t = ((ws[0] + ws[1]) + ws[2]) + ws[3];
    __syncthreads();
    return t;
}

}  // namespace sellcs
