// Cholesky factor and triangular solves of one 64 x 64 tile by a workgroup of 256 threads
// (four waves), blocked by 16: the serial part of a column runs over 16 lanes of one wave,
// everything else on the FP64 matrix cores.
//
// What sets the time of a 64-column factorisation or substitution is its serial chain, and in
// it the trips through LDS: on gfx950 a barrier with an exchange costs 85 ns, an LDS read 8
// cycles of the CU's one pipe for every wave that issues it, a lane shuffle of a double 44 ns,
// a division 47 ns, but a dependent multiply-add 2 ns.  Four threads per vector with a
// division and a shuffle per row took 20 to 31 us a tile, one wave with a row per lane 48 us;
// here a panel or solve step takes 12 to 21 us (the longer ones with 800 and more tiles in the
// launch), the factor 17.5 us.
//
// The 16 x 16 x 4 instruction returns its result (register v of lane l: row l / 16 + 4 v, column
// l % 16) in the layout in which the next one takes its right operand, K step by K step, so a
// block substitution stays in registers: X_k = I_k (B_k - sum_m L_km X_m) with I_k the inverse
// of the 16 x 16 diagonal block.
#pragma once
#include <hip/hip_runtime.h>

#include "lanes.hpp"
#include "mgemm.hpp"

namespace lsdd {
namespace t64 {

constexpr int LD = 65;                 // row stride of the tile in LDS

struct Tile {
    double t[64][LD];                  // row-major, lower triangle
    double inv[4][16][17];             // inverses of the diagonal blocks, row-major
};

__device__ inline mg::d4 mma(double a, double b, mg::d4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }

// inverse of diagonal block kb by the calling wave: lane r % 16 holds row r of the block in a and
// the reciprocal of its diagonal entry in rd; lane c % 16 forms column c.  The factor's entries
// come by lane permutations, not from LDS, whose pipe the waves share.
__device__ inline void invert_block(Tile& s, int kb, const double (&a)[16], double rd) {
    const int c = (int)threadIdx.x & 15;
    double z[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        double v = r == c ? 1.0 : 0.0;
#pragma unroll
        for (int k = 0; k < r; ++k) v -= row_bcast(a[k], r) * z[k];
        z[r] = v * row_bcast(rd, r);
    }
    if (((int)threadIdx.x & 63) < 16)
#pragma unroll
        for (int r = 0; r < 16; ++r) s.inv[kb][r][c] = z[r];
}

// the four block inverses of the tile in s.t (after a barrier)
__device__ inline void prepare(Tile& s) {
    const int t = (int)threadIdx.x, kb = t >> 6, lm = t & 15;
    double a[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) a[k] = s.t[16 * kb + lm][16 * kb + k];
    invert_block(s, kb, a, 1.0 / s.t[16 * kb + lm][16 * kb + lm]);
    __syncthreads();
}

// X <- L^{-1} X for the wave's 16 columns: X[k] the rows 16 k .. 16 k + 15 in the result layout
__device__ inline void forward(const Tile& s, mg::d4 (&X)[4]) {
    const int l = (int)threadIdx.x & 63, lm = l & 15, lk = l >> 4;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
        mg::d4 v = X[kb];
#pragma unroll
        for (int m = 0; m < kb; ++m)
#pragma unroll
            for (int q = 0; q < 4; ++q) v = mma(-s.t[16 * kb + lm][16 * m + 4 * q + lk], X[m][q], v);
        mg::d4 y = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int q = 0; q < 4; ++q) y = mma(s.inv[kb][lm][4 * q + lk], v[q], y);
        X[kb] = y;
    }
}

// X <- L^{-T} X
__device__ inline void backward(const Tile& s, mg::d4 (&X)[4]) {
    const int l = (int)threadIdx.x & 63, lm = l & 15, lk = l >> 4;
#pragma unroll
    for (int kb = 3; kb >= 0; --kb) {
        mg::d4 v = X[kb];
#pragma unroll
        for (int m = 3; m > kb; --m)
#pragma unroll
            for (int q = 0; q < 4; ++q) v = mma(-s.t[16 * m + 4 * q + lk][16 * kb + lm], X[m][q], v);
        mg::d4 y = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int q = 0; q < 4; ++q) y = mma(s.inv[kb][4 * q + lk][lm], v[q], y);
        X[kb] = y;
    }
}

// reciprocal of a pivot, 1 for a failed one (the same value in every lane)
__device__ inline double pivot_rcp(double d) {
    if (d > 1e-290) return quick_rcp(d);
    return d > 0.0 ? 1.0 / d : 1.0;
}

// Cholesky factor of the tile in s.t (lower triangle, in place), its first nbk blocks of 16
// (the rest is taken to be an identity and left alone); piv[0 .. 63]: the pivots.  A pivot that
// is not positive is replaced by 1 so that the factorisation runs to the end.  Leaves s.inv of
// the blocks but the last; barriers on both sides.
__device__ inline void cholesky(Tile& s, double* piv, int nbk) {
    const int t = (int)threadIdx.x, w = t >> 6, l = t & 63, lm = l & 15, lk = l >> 4;
    for (int kb = 0; kb < nbk; ++kb) {
        const int o = 16 * kb;
        if (w == 0) {
            // lane r % 16 holds row r of the block; the columns carry d L until the end
            double a[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) a[k] = s.t[o + lm][o + k];
            double mine = 1.0;                         // pivot of column lm
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const double d = row_bcast(a[j], j);
                if (lm == j) mine = d;
                const double f = a[j] * pivot_rcp(d);
#pragma unroll
                for (int k = j + 1; k < 16; ++k) a[k] -= f * row_bcast(a[j], k);
            }
            const double root = mine > 0.0 ? sqrt(mine) : 1.0, rr = 1.0 / root;
            if (l < 16) piv[o + l] = mine;
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const double rk = row_bcast(rr, k);    // with every lane active
                a[k] = lm == k ? root : a[k] * rk;
                if (l < 16 && lm >= k) s.t[o + lm][o + k] = a[k];
            }
            if (kb + 1 < nbk) invert_block(s, kb, a, rr);
        }
        __syncthreads();
        if (kb + 1 == nbk) break;
        // the panel below, one block per wave: L_ib = A_ib I^T
        const int ib = kb + 1 + w;
        mg::d4 y = {0.0, 0.0, 0.0, 0.0};
        if (ib < nbk) {
#pragma unroll
            for (int q = 0; q < 4; ++q) y = mma(s.t[16 * ib + lm][o + 4 * q + lk], s.inv[kb][lm][4 * q + lk], y);
        }
        __syncthreads();
        if (ib < nbk) {
#pragma unroll
            for (int v = 0; v < 4; ++v) s.t[16 * ib + lk + 4 * v][o + lm] = y[v];
        }
        __syncthreads();
        // trailing blocks (i, j), i >= j > kb, dealt over the waves: A -= L_i L_j^T
        const int m = nbk - kb - 1;
        for (int job = w; job < m * (m + 1) / 2; job += 4) {
            int i = 0, r = job;
            while (r > i) r -= ++i;
            const int bi = 16 * (kb + 1 + i), bj = 16 * (kb + 1 + r);
            mg::d4 c;
#pragma unroll
            for (int v = 0; v < 4; ++v) c[v] = s.t[bi + lk + 4 * v][bj + lm];
#pragma unroll
            for (int q = 0; q < 4; ++q) c = mma(-s.t[bi + lm][o + 4 * q + lk], s.t[bj + lm][o + 4 * q + lk], c);
#pragma unroll
            for (int v = 0; v < 4; ++v) s.t[bi + lk + 4 * v][bj + lm] = c[v];
        }
        __syncthreads();
    }
}

}  // namespace t64
}  // namespace lsdd
