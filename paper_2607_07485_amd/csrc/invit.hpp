// Eigenvectors of a symmetric tridiagonal matrix by inverse iteration, one workgroup per call.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "consts.hpp"
#include "dense.hpp"
#include "lanes.hpp"
#include "mgemm.hpp"
#include "tile64.hpp"

namespace lsdd {

// ---------------------------------------------------------------- inverse iteration
// Every lane of a wave solves its own shifted system (T - lam I) y = b, scratch interleaved
// by lane (entry k of lane t at [64 k + t]).  The first solve factors with partial pivoting
// and keeps 1 / pivot, the two superdiagonals of U, the multipliers and the row exchanges;
// the later solves of the same shift only apply them.  A solve is one serial chain over the
// n rows: a division and two multiply-adds a row to factor, one multiply-add a row to apply,
// three to substitute back (the pivots' reciprocals are at hand, no division).
struct TriLane {
    double *ri, *u1, *u2, *y, *f;     // lane base pointers, stride 64
    uint32_t* sw;                     // word k >> 3, bit k & 7: rows k and k + 1 exchanged
};

__device__ inline TriLane tri_lane(double* ws, int n, int t) {
    TriLane L;
    L.ri = ws + t;
    L.u1 = L.ri + (int64_t)64 * n;
    L.u2 = L.u1 + (int64_t)64 * n;
    L.y = L.u2 + (int64_t)64 * n;
    L.f = L.y + (int64_t)64 * n;
    L.sw = reinterpret_cast<uint32_t*>(ws + (int64_t)5 * 64 * n) + t;
    return L;
}

// Rows go in blocks of 8: a full block has no branch, so that the compiler knows how many
// stores follow the loads of the next block, which it would otherwise wait for, rows and all.
constexpr int TB8 = 8;

__device__ inline void tri_factor_solve(const double* __restrict__ d, const double* __restrict__ e, int n, double lam,
                                        const TriLane& L, double tiny) {
    double a0 = d[0] - lam, a1 = e[0], bk = L.y[0];
    auto step = [&](int k, double sub, double nd, double ns, double bn, uint32_t& bits) {
        const bool sw = !(fabs(a0) >= fabs(sub));
        if (!sw && fabs(a0) < tiny) a0 = a0 >= 0.0 ? tiny : -tiny;
        const double r = quick_rcp(sw ? sub : a0);
        const double f = (sw ? a0 : sub) * r;
        const int64_t q = (int64_t)64 * k;
        L.ri[q] = r;
        L.u1[q] = sw ? nd : a1;
        L.u2[q] = sw ? ns : 0.0;
        L.f[q] = f;
        bits |= (uint32_t)sw << (k & 7);
        a0 = sw ? a1 - f * nd : nd - f * a1;
        a1 = sw ? -f * ns : ns;
        const double top = sw ? bn : bk, low = sw ? bk : bn;
        L.y[q] = top;
        bk = low - f * top;
    };
    // block k0: e[k0 .. k0 + 8], d and y [k0 + 1 .. k0 + 8] (past the end: the last entry)
    double E[TB8 + 1], D[TB8], B[TB8], En[TB8 + 1], Dn[TB8], Bn[TB8];
    auto fetch = [&](int k0, double (&e_)[TB8 + 1], double (&d_)[TB8], double (&b_)[TB8]) {
#pragma unroll
        for (int u = 0; u <= TB8; ++u) e_[u] = e[min(k0 + u, n - 2)];
#pragma unroll
        for (int u = 0; u < TB8; ++u) {
            d_[u] = d[min(k0 + u + 1, n - 1)];
            b_[u] = L.y[(int64_t)64 * min(k0 + u + 1, n - 1)];
        }
    };
    int k0 = 0;
    fetch(0, E, D, B);
    // the step of row k needs e[k + 1]: rows up to n - 3 here, the last ones below
    for (; k0 + TB8 < n - 1; k0 += TB8) {
        uint32_t bits = 0;
        fetch(k0 + TB8, En, Dn, Bn);
#pragma unroll
        for (int u = 0; u < TB8; ++u) step(k0 + u, E[u], D[u] - lam, E[u + 1], B[u], bits);
        L.sw[64 * (k0 >> 3)] = bits;
#pragma unroll
        for (int u = 0; u <= TB8; ++u) E[u] = En[u];
#pragma unroll
        for (int u = 0; u < TB8; ++u) D[u] = Dn[u], B[u] = Bn[u];
    }
    uint32_t bits = 0;
#pragma unroll
    for (int u = 0; u < TB8; ++u)
        if (k0 + u < n - 1) step(k0 + u, E[u], D[u] - lam, k0 + u + 1 < n - 1 ? E[u + 1] : 0.0, B[u], bits);
    L.sw[64 * (k0 >> 3)] = bits;
    if (fabs(a0) < tiny) a0 = a0 >= 0.0 ? tiny : -tiny;
    const int64_t q = (int64_t)64 * (n - 1);
    L.ri[q] = quick_rcp(a0);
    L.u1[q] = 0.0;
    L.u2[q] = 0.0;
    L.y[q] = bk;
}

__device__ inline void tri_apply_factor(int n, const TriLane& L) {
    double bk = L.y[0];
    auto step = [&](int k, double f, double bn, uint32_t bits) {
        const bool sw = (bits >> (k & 7)) & 1;
        const double top = sw ? bn : bk, low = sw ? bk : bn;
        L.y[(int64_t)64 * k] = top;
        bk = low - f * top;
    };
    double F[TB8], B[TB8], Fn[TB8], Bn[TB8];
    uint32_t S, Sn;
    auto fetch = [&](int k0, double (&f_)[TB8], double (&b_)[TB8], uint32_t& s_) {
        s_ = L.sw[64 * (k0 >> 3)];
#pragma unroll
        for (int u = 0; u < TB8; ++u) {
            f_[u] = L.f[(int64_t)64 * min(k0 + u, n - 2)];
            b_[u] = L.y[(int64_t)64 * min(k0 + u + 1, n - 1)];
        }
    };
    int k0 = 0;
    fetch(0, F, B, S);
    for (; k0 + TB8 < n - 1; k0 += TB8) {
        fetch(k0 + TB8, Fn, Bn, Sn);
#pragma unroll
        for (int u = 0; u < TB8; ++u) step(k0 + u, F[u], B[u], S);
#pragma unroll
        for (int u = 0; u < TB8; ++u) F[u] = Fn[u], B[u] = Bn[u];
        S = Sn;
    }
#pragma unroll
    for (int u = 0; u < TB8; ++u)
        if (k0 + u < n - 1) step(k0 + u, F[u], B[u], S);
    L.y[(int64_t)64 * (n - 1)] = bk;
}

// back substitution; returns the squared norm of the solution
__device__ inline double tri_back(int n, const TriLane& L) {
    double x1 = 0.0, x2 = 0.0, nr = 0.0;
    auto step = [&](int k, double y, double r, double p, double q) {
        const double xk = (y - q * x2 - p * x1) * r;
        L.y[(int64_t)64 * k] = xk;
        nr += xk * xk;
        x2 = x1;
        x1 = xk;
    };
    double Y[TB8], R[TB8], P[TB8], Q[TB8], Yn[TB8], Rn[TB8], Pn[TB8], Qn[TB8];
    auto fetch = [&](int k1, double (&y_)[TB8], double (&r_)[TB8], double (&p_)[TB8], double (&q_)[TB8]) {
#pragma unroll
        for (int u = 0; u < TB8; ++u) {
            const int64_t o = (int64_t)64 * max(k1 - u, 0);
            y_[u] = L.y[o];
            r_[u] = L.ri[o];
            p_[u] = L.u1[o];
            q_[u] = L.u2[o];
        }
    };
    int k1 = n - 1;
    fetch(k1, Y, R, P, Q);
    for (; k1 - TB8 >= 0; k1 -= TB8) {
        fetch(k1 - TB8, Yn, Rn, Pn, Qn);
#pragma unroll
        for (int u = 0; u < TB8; ++u) step(k1 - u, Y[u], R[u], P[u], Q[u]);
#pragma unroll
        for (int u = 0; u < TB8; ++u) Y[u] = Yn[u], R[u] = Rn[u], P[u] = Pn[u], Q[u] = Qn[u];
    }
#pragma unroll
    for (int u = 0; u < TB8; ++u)
        if (k1 - u >= 0) step(k1 - u, Y[u], R[u], P[u], Q[u]);
    return nr;
}

// LDS of the inverse iteration: the matrix cores' staging buffers, then the 64 x 64 tile.
union InvSmem {
    mg::Smem mm;
    t64::Tile tile;
    double s[64 * 65];
};

// Members of one cluster (cl[t] equal) are made orthonormal, members of different ones only
// normalised: with D the inverse column norms and the cross-cluster entries of the Gram
// matrix left out, D Y^T Y D = L L^T and Y <- Y D L^{-T}, the Q that Gram-Schmidt in index
// order gives per cluster (Y: n x bn, row-major, ld 64).  The Gram matrix runs on the matrix
// cores, its factor and the row-wise substitution through tile64.hpp (as 2016 dependent
// loads a row the substitution took about 1 ms a pass at n = 882).  0, with Y unchanged, when a
// pivot falls below 1e-12, where one pass would lose orthogonality; 2 when none falls below
// 1e-2 and no column has lost more than 99 % of its squared norm since norm[]: nothing that
// matters cancelled in this pass; else 1.
__device__ inline int batch_cholqr(InvSmem& sm, double* Y, int n, int bn, const int* cl, const double* norm) {
    __shared__ double s_d[64], s_piv[64];
    __shared__ bool s_kept[64];
    mg::d4 acc[2][2];
    mg::zero(acc);
    mg::tile_mma<mg::IMAJ, mg::IMAJ>(sm.mm, Y, 64, 0, bn, Y, 64, 0, bn, 0, n, acc);
    __syncthreads();
    t64::Tile& T = sm.tile;
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = mg::acc_row(p, v), j = mg::acc_col(q);
                T.t[i][j] = i < bn && j < bn ? (cl[i] == cl[j] ? acc[p][q][v] : 0.0) : (i == j ? 1.0 : 0.0);
            }
    __syncthreads();
    if (tid() < 64) {
        const double g = T.t[tid()][tid()];
        s_d[tid()] = g > 0.0 ? 1.0 / sqrt(g) : 0.0;
        s_piv[tid()] = 1.0;
        s_kept[tid()] = tid() >= bn || g > 1e-2 * norm[tid()];
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 16; ++u) {
        const int i = tid() & 63, j = (tid() >> 6) + 4 * u;
        T.t[i][j] *= s_d[i] * s_d[j];
    }
    __syncthreads();
    t64::cholesky(T, s_piv, (bn + 15) >> 4);
    const int l = tid() & 63;
    const bool ok = __all(s_piv[l] > 1e-12);            // the same in every wave
    if (ok) {
        t64::prepare(T);
        // 16 rows of Y per wave as right-hand sides: L z = D y
        for (int r0 = 16 * (tid() >> 6); r0 < n; r0 += 64) {
            const int r = r0 + (l & 15);
            double* y = Y + (int64_t)min(r, n - 1) * 64 + (l >> 4);
            mg::d4 X[4];
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int q = 0; q < 4; ++q) X[k][q] = y[16 * k + 4 * q] * s_d[16 * k + 4 * q + (l >> 4)];
            t64::forward(T, X);
            if (r < n)
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int q = 0; q < 4; ++q) y[16 * k + 4 * q] = X[k][q];
        }
    }
    const bool well = __all(s_piv[l] > 1e-2 && s_kept[l]);
    __syncthreads();
    return ok ? 1 + (int)well : 0;
}

struct InvShared {
    InvSmem sm;
    double red[LSDD_WG / 64];
    double dot[64];
    int cl[64];
    double norm[64];                                   // squared norms of the solves' results
    int conv;
};

// Eigenvectors of the tridiagonal (d, e) for the eigenvalues lam[0..kk) by inverse iteration,
// to the columns of V (n x kk, column-major).  Eigenvalues closer than 1e-4 ||T|| form a
// cluster; the workgroup takes the clusters that start at the indices [r0, r1), as many whole
// ones at a time as 64 lanes hold (symmetric aggregates have dozens of pairs and triples; one
// cluster at a time took 7 ms), a larger cluster 64 members at a time: solve every member's system on its own lane,
// make the batch orthogonal to the cluster's earlier members, then orthonormal (Cholesky QR;
// Gram-Schmidt member by member where that is refused).  The batch stays row-major in the
// scratch, interleaved by lane for the solves and an operand of the matrix cores as it is.
// Every iteration orthogonalises twice, but for the last only where something cancelled in the
// first pass: with one pass always, factors of element blocks with 96 equal eigenvalues of 128 were
// off by 7e-14 instead of 2e-15, and the modes of aggregates of 450 to 900 DOFs orthogonal to
// 1e-8 (geometric mean) instead of 1.1e-10 (the next solve multiplies what the pass leaves).
//
// Convergence: from the second solve on, the iterate entering a solve has unit norm, so the
// norm of the result is the solve's growth 1 / |lambda - shift| along the eigenvector; once it
// exceeds 1 / (1e-10 ||T||) (shift within 1e-10 ||T|| of an eigenvalue, at least 1e-4 ||T||
// from every other cluster) each further solve would shrink the error by at least 1e6, and
// the iteration stops when every member is there (at most 4 solves).
//
// Bound by the serial chains of the solves and of the 64-column factorisations, not by
// bytes: at n = 882 a factoring solve takes 187 us, a later one 104, an orthonormalisation
// 100.  Eight matrices of up to 882 with 179 vectors each: 15.4 -> 4.6 ms; 64 of up to 285
// with 40 each: 0.91 -> 0.31 ms.
// n >= 2; ws: invit_ws(n) doubles; first: LDS, kk + 1 bytes.
__device__ inline void wg_invit(const double* __restrict__ d, const double* __restrict__ e, int n, const double* lam,
                                int kk, int r0, int r1, double* V, double* ws, unsigned char* first, InvShared& S) {
    double tnorm = 0.0;
    for (int i = tid(); i < n; i += LSDD_WG)
        tnorm = fmax(tnorm, fabs(d[i]) + (i > 0 ? fabs(e[i - 1]) : 0.0) + (i + 1 < n ? fabs(e[i]) : 0.0));
    tnorm = fmax(wg_max(tnorm, S.red), 1e-300);
    double* dd = ws + (int64_t)INVIT_SLOTS * n + 64;   // 64 x 64
    double* Y = ws + (int64_t)3 * 64 * n;              // n x 64, row-major: the lanes' iterates
    for (int i = tid(); i <= kk; i += LSDD_WG)
        first[i] = i == 0 || i == kk || lam[i] - lam[i - 1] > 1e-4 * tnorm;
    __syncthreads();
    const double tiny = 2.220446049250313e-16 * tnorm;
    const double grow2 = 1.0 / ((1e-10 * tnorm) * (1e-10 * tnorm));
    auto start_value = [&](int i, int k) {
        unsigned h = (unsigned)(k * 2654435761u) ^ (unsigned)(i * 40503u);
        return 1.0 + 0.25 * ((double)(h & 0xffff) / 65536.0 - 0.5);
    };
    // members b0 .. b0 + bn - 1; q0 .. b0 - 1: the earlier members of their cluster
    auto batch = [&](int b0, int bn, int qa) {
        if (tid() < 64) {
            int c = min(b0 + tid(), b0 + bn - 1);
            while (!first[c]) --c;
            S.cl[tid()] = c;
        }
        for (int64_t q = tid(); q < (int64_t)64 * n; q += LSDD_WG) {
            const int t = (int)(q & 63), k = (int)(q >> 6);
            Y[q] = t < bn ? start_value(b0 + t, k) : 0.0;
        }
        __syncthreads();
        for (int it = 0; it < 4; ++it) {
            if (tid() == 0) S.conv = it >= 1;
            __syncthreads();
            if (tid() < bn) {
                const int i = b0 + tid();
                const TriLane L = tri_lane(ws, n, tid());
                if (it == 0) tri_factor_solve(d, e, n, lam[i] + (i - S.cl[tid()]) * 2.0 * tiny, L, tiny);
                else tri_apply_factor(n, L);
                const double nr = tri_back(n, L);
                if (!(nr >= grow2)) S.conv = 0;
                S.norm[tid()] = nr;
            }
            __syncthreads();
            const bool last = S.conv != 0 || it == 3;
            for (int pass = 0; pass < 2; ++pass) {
                // against the earlier members of the cluster, 64 at a time
                for (int q0 = qa; q0 < b0; q0 += 64) {
                    const double* Q = V + (int64_t)q0 * n;
                    const int qn = min(64, b0 - q0);
                    mg::d4 acc[2][2];
                    mg::zero(acc);
                    mg::tile_mma<mg::KMAJ, mg::IMAJ>(S.sm.mm, Q, n, 0, qn, Y, 64, 0, bn, 0, n, acc);
#pragma unroll
                    for (int p = 0; p < 2; ++p)
#pragma unroll
                        for (int q = 0; q < 2; ++q)
#pragma unroll
                            for (int v = 0; v < 4; ++v) {
                                const int i = mg::acc_row(p, v), j = mg::acc_col(q);
                                if (i < qn && j < bn) dd[i + j * qn] = acc[p][q][v];
                            }
                    __syncthreads();
                    for (int t0 = 0; t0 < n; t0 += mg::T) {
                        mg::zero(acc);
                        mg::tile_mma<mg::IMAJ, mg::KMAJ>(S.sm.mm, Q + t0, n, 0, n - t0, dd, qn, 0, bn, 0, qn, acc);
#pragma unroll
                        for (int p = 0; p < 2; ++p)
#pragma unroll
                            for (int q = 0; q < 2; ++q)
#pragma unroll
                                for (int v = 0; v < 4; ++v) {
                                    const int r = t0 + mg::acc_row(p, v), t = mg::acc_col(q);
                                    if (r < n && t < bn) Y[(int64_t)r * 64 + t] -= acc[p][q][v];
                                }
                    }
                    __syncthreads();
                }
                if (const int c = batch_cholqr(S.sm, Y, n, bn, S.cl, S.norm)) {
                    if (c == 2 && !last) break;
                    continue;
                }
                // member by member, each normalised before its use
                for (int t = 0; t < bn; ++t) {
                    const int w = tid() >> 6, l = tid() & 63, t0 = max(0, S.cl[t] - b0);
                    for (int s0 = t0 + w; s0 < t; s0 += LSDD_WG / 64) {
                        double s = 0.0;
                        for (int k = l; k < n; k += 64) s += Y[(int64_t)k * 64 + s0] * Y[(int64_t)k * 64 + t];
                        s = wave_sum(s);
                        if (l == 0) S.dot[s0] = s;
                    }
                    __syncthreads();
                    double nr = 0.0;
                    for (int k = tid(); k < n; k += LSDD_WG) {
                        double s = 0.0;
                        for (int s0 = t0; s0 < t; ++s0) s += Y[(int64_t)k * 64 + s0] * S.dot[s0];
                        const double v = Y[(int64_t)k * 64 + t] - s;
                        Y[(int64_t)k * 64 + t] = v;
                        nr += v * v;
                    }
                    nr = wg_sum(nr, S.red);
                    const double sc = 1.0 / sqrt(nr);
                    for (int k = tid(); k < n; k += LSDD_WG) Y[(int64_t)k * 64 + t] *= sc;
                    __syncthreads();
                }
            }
            if (last) break;
        }
        // to V, column-major, through LDS tiles: rows contiguous on both sides
        double* s = S.sm.s;
        for (int k0 = 0; k0 < n; k0 += 64) {
            __syncthreads();
            for (int q = tid(); q < 64 * 64; q += LSDD_WG)
                s[(q & 63) * 65 + (q >> 6)] = Y[(int64_t)min(k0 + (q >> 6), n - 1) * 64 + (q & 63)];
            __syncthreads();
            for (int q = tid(); q < 64 * 64; q += LSDD_WG) {
                const int t = q >> 6, k = q & 63;
                if (t < bn && k0 + k < n) V[(int64_t)(b0 + t) * n + k0 + k] = s[t * 65 + k];
            }
        }
        __syncthreads();
    };
    int b0 = r0;
    while (b0 < r1 && !first[b0]) ++b0;
    while (b0 < r1) {
        int end = b0, ce = b0;                         // whole clusters b0 .. end - 1
        while (end < r1) {
            ce = end + 1;
            while (!first[ce]) ++ce;                   // first[kk] is set
            if (ce - b0 > 64) break;
            end = ce;
        }
        const bool large = end == b0;                  // more than 64 members: 64 at a time
        const int stop = large ? ce : end;
        for (int m = b0; m < stop; m += 64) batch(m, min(64, stop - m), large ? b0 : m);
        b0 = stop;
    }
}

}  // namespace lsdd
