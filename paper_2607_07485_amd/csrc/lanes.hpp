// Small device helpers of the serial chains in the dense kernels.
#pragma once
#include <hip/hip_runtime.h>

namespace lsdd {

// 1 / x for normal x whose reciprocal is normal: the hardware's estimate and two Newton
// steps (each doubles its bits), about half the chain of a division
__device__ inline double quick_rcp(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    return fma(fma(-x, r, 1.0), r, r);
}

// v permuted among 16 lanes by the vector ALU itself (a shuffle goes through LDS, whose one
// pipe a CU's waves share: 44 ns a double against 20).  Every source lane must be active: not
// inside a branch or a conditional operand.
template <int CTRL>
__device__ inline double quad_perm(double v) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}

// v of lane s (0 .. 15) of the caller's group of 16 lanes, the same way; s is a constant after
// unrolling
__device__ inline double row_bcast(double v, int s) {
    switch (s) {
        case 0: return quad_perm<0x150>(v);
        case 1: return quad_perm<0x151>(v);
        case 2: return quad_perm<0x152>(v);
        case 3: return quad_perm<0x153>(v);
        case 4: return quad_perm<0x154>(v);
        case 5: return quad_perm<0x155>(v);
        case 6: return quad_perm<0x156>(v);
        case 7: return quad_perm<0x157>(v);
        case 8: return quad_perm<0x158>(v);
        case 9: return quad_perm<0x159>(v);
        case 10: return quad_perm<0x15a>(v);
        case 11: return quad_perm<0x15b>(v);
        case 12: return quad_perm<0x15c>(v);
        case 13: return quad_perm<0x15d>(v);
        case 14: return quad_perm<0x15e>(v);
        default: return quad_perm<0x15f>(v);
    }
}

// v (as 32-bit words) from the lane the control names, 0 in the rows of 16 lanes not in ROWS
template <int CTRL, int ROWS, typename T>
__device__ inline T row_from(T v) {
    if constexpr (sizeof(T) == 8) {
        const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xf, false);
        const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xf, false);
        return __hiloint2double(hi, lo);
    } else {
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROWS, 0xf, false));
    }
}
// v of lane 63, the same in the whole wave
template <typename T>
__device__ inline T from_last(T v) {
    if constexpr (sizeof(T) == 8)
        return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 63),
                                __builtin_amdgcn_readlane(__double2loint(v), 63));
    else
        return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// Sum of v over the caller's group of L lanes (a power of two), the same in every lane and in
// a fixed order, by the vector ALU's permutations: inside 16 lanes exchanging halves of 2, 4,
// 8 and 16 lanes (the last two mirror, which is the same once the smaller groups are equal);
// the four 16-lane sums of a wave pass on to the next row's lanes and end in the last lane.
// Ten sums over a wave by shuffles kept a CU's LDS pipe busy for 1 us at 8 waves.
template <int L, typename T>
__device__ inline T sum_lanes(T v) {
    if constexpr (L >= 2) v += row_from<0xb1, 0xf>(v);         // 1 0 3 2
    if constexpr (L >= 4) v += row_from<0x4e, 0xf>(v);         // 2 3 0 1
    if constexpr (L >= 8) v += row_from<0x141, 0xf>(v);        // mirror of 8 lanes
    if constexpr (L >= 16) v += row_from<0x140, 0xf>(v);       // mirror of 16 lanes
    if constexpr (L == 32) v += __shfl_xor(v, 16, 64);
    if constexpr (L == 64) {
        v += row_from<0x142, 0xa>(v);                          // rows 1, 3: lane 15 of the row before
        v += row_from<0x143, 0xc>(v);                          // rows 2, 3: lane 31
        v = from_last(v);
    }
    return v;
}

}  // namespace lsdd
