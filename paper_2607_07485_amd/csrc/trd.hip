// Blocked Householder tridiagonalisation of the larger local spectral problems
// (C = L^{-1} S~ L^{-T} of an aggregate), many matrices per launch and many
// workgroups per matrix.
//
// The reduction T = Q^T C Q is the one the single-workgroup path computes
// (reflector j from column j below the diagonal, tau_j, d, e), but the
// rank-2 updates of the trailing matrix are delayed over panels of TRD_NB
// columns: inside a panel, column j is corrected by the panel's earlier
// reflectors (V, W) and the matrix-vector product with the trailing block is
// corrected the same way; after the panel one symmetric rank-2k update
// C22 -= V W^T + W V^T runs on the FP64 matrix cores.  Per column:
//   k_trd_col   (one workgroup per matrix): finish the previous W column,
//               correct column j, form reflector v_j (stored in column j, with
//               an explicit 1 on the subdiagonal), dots W^T v and V^T v;
//   k_trd_symv  (many workgroups per matrix): w = tau (C22 v - V (W^T v)
//               - W (V^T v)), one wave per column of C22.
// Per panel: k_trd_fin (finish the last W column), k_trd_update.
//
// Storage per matrix: C (n x n, both triangles kept exactly symmetric), the
// tridiagonal d, e, tau in the T scratch, V and W (n x TRD_NB each,
// column-major, so row sweeps over one column are coalesced) and the dots in
// the v_buf slot (n^2 doubles, n > 2 TRD_NB).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <stdexcept>
#include <vector>

#include "dense.hpp"
#include "kernels.hpp"
#include "mgemm.hpp"

namespace lsdd {

namespace {

constexpr int WG = LSDD_WG;
constexpr int NB = TRD_NB;
constexpr int CPW = 4;               // columns per wave in k_trd_symv
constexpr int CPG = CPW * WG / 64;   // columns per workgroup

struct Mat {
    int n;
    double* a;
    double* d;
    double* e;
    double* tau;
    double* V;
    double* W;
    double* zw;
    double* zv;
};

__device__ inline Mat mat_of(const LocalArgs& A, int b) {
    Mat m;
    const int ag = A.first + b;
    m.n = (int)(A.agg_ptr[ag + 1] - A.agg_ptr[ag]);
    m.a = A.s_buf + A.sq_off[b];
    double* T = A.t_buf + A.t_off[b];
    m.d = T;
    m.e = T + m.n;
    m.tau = T + 2 * m.n;
    m.V = A.v_buf + A.sq_off[b];
    m.W = m.V + (int64_t)NB * m.n;
    m.zw = m.W + (int64_t)NB * m.n;
    m.zv = m.zw + NB;
    return m;
}

// W(:, q) <- w - (tau_jp / 2) (w . v) v for the raw w of reflector jp
__device__ inline void finish_w(const Mat& m, int jp, int q, double* red) {
    double s = 0.0;
    const double* vq = m.V + (int64_t)q * m.n;
    double* wq = m.W + (int64_t)q * m.n;
    for (int i = jp + 1 + tid(); i < m.n; i += WG) s += wq[i] * vq[i];
    s = wg_sum(s, red);
    const double K = 0.5 * m.tau[jp] * s;
    for (int i = jp + 1 + tid(); i < m.n; i += WG) wq[i] -= K * vq[i];
    __syncthreads();
}

__global__ void __launch_bounds__(WG) k_trd_col(LocalArgs A, const int32_t* big, int j, int j0) {
    __shared__ double red[WG / 64];
    __shared__ double rowvw[2 * NB];
    __shared__ double part[WG / 64][2 * NB];
    const Mat m = mat_of(A, big[blockIdx.x]);
    const int n = m.n;
    if (j + 2 >= n) return;
    const int p = j - j0;
    if (p > 0) finish_w(m, j - 1, p - 1, red);
    // column j (rows j..n-1) with the panel's earlier reflectors applied
    if (tid() < p) {
        rowvw[tid()] = m.V[j + (int64_t)tid() * n];
        rowvw[NB + tid()] = m.W[j + (int64_t)tid() * n];
    }
    __syncthreads();
    double* col = m.a + (int64_t)j * n;
    for (int i = j + tid(); i < n; i += WG) {
        double s = col[i];
        for (int q = 0; q < p; ++q) s -= m.V[i + (int64_t)q * n] * rowvw[NB + q] + m.W[i + (int64_t)q * n] * rowvw[q];
        col[i] = s;
    }
    __syncthreads();
    // reflector from x = col[j+1 .. n-1]
    const int mm = n - j - 1;
    double* x = col + j + 1;
    double s2 = 0.0;
    for (int i = 1 + tid(); i < mm; i += WG) s2 += x[i] * x[i];
    s2 = wg_sum(s2, red);
    const double alpha = x[0];
    double t = 0.0, beta = alpha, sc = 0.0;
    if (s2 > 0.0) {
        const double nrm = sqrt(alpha * alpha + s2);
        beta = alpha >= 0.0 ? -nrm : nrm;
        t = (beta - alpha) / beta;
        sc = 1.0 / (alpha - beta);
    }
    if (tid() == 0) {
        m.d[j] = col[j];
        m.e[j] = beta;
        m.tau[j] = t;
    }
    __syncthreads();
    double* vp = m.V + (int64_t)p * n;
    for (int i = tid(); i < mm; i += WG) {
        const double vi = (i == 0) ? 1.0 : (s2 > 0.0 ? x[i] * sc : 0.0);
        x[i] = vi;
        vp[j + 1 + i] = vi;
    }
    for (int i = j0 + tid(); i <= j; i += WG) {
        vp[i] = 0.0;
        m.W[i + (int64_t)p * n] = 0.0;
    }
    __syncthreads();
    // zw_q = W(j+1:, q) . v, zv_q = V(j+1:, q) . v for q < p
    const int w = tid() >> 6, l = tid() & 63;
    for (int q0 = 0; q0 < p; q0 += 8) {
        double aw[8], av[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) aw[u] = av[u] = 0.0;
        for (int i = j + 1 + tid(); i < n; i += WG) {
            const double vi = x[i - j - 1];
            // columns past p re-read column p - 1 (the loads stay unconditional and in
            // flight together) and are not added
            double ww[8], vv[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int64_t qc = min(q0 + u, p - 1);
                ww[u] = m.W[i + qc * n];
                vv[u] = m.V[i + qc * n];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (q0 + u < p) {
                    aw[u] += ww[u] * vi;
                    av[u] += vv[u] * vi;
                }
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            aw[u] = wave_sum(aw[u]);
            av[u] = wave_sum(av[u]);
        }
        if (l == 0)
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                part[w][q0 + u] = aw[u];
                part[w][NB + q0 + u] = av[u];
            }
    }
    __syncthreads();
    if (tid() < p) {
        double sw = 0.0, sv = 0.0;
        for (int r = 0; r < WG / 64; ++r) {
            sw += part[r][tid()];
            sv += part[r][NB + tid()];
        }
        m.zw[tid()] = sw;
        m.zv[tid()] = sv;
    }
}

__global__ void __launch_bounds__(WG) k_trd_symv(LocalArgs A, const int32_t* big, int j, int j0) {
    extern __shared__ double s_v[];    // v (n - j - 1), then zw, zv
    const Mat m = mat_of(A, big[blockIdx.y]);
    const int n = m.n;
    if (j + 2 >= n) return;
    const int mm = n - j - 1;
    const int c0 = (int)blockIdx.x * CPG;
    if (c0 >= mm) return;
    const int p = j - j0;
    const double* v = m.a + (int64_t)j * n + j + 1;
    double* zz = s_v + mm;
    for (int i = tid(); i < mm; i += WG) s_v[i] = v[i];
    if (tid() < p) {
        zz[tid()] = m.zw[tid()];
        zz[NB + tid()] = m.zv[tid()];
    }
    __syncthreads();
    const double t = m.tau[j];
    const int w = tid() >> 6, l = tid() & 63;
    for (int cc = 0; cc < CPW; ++cc) {
        const int c = c0 + w * CPW + cc;
        if (c >= mm) break;
        const double* cp = m.a + (int64_t)(j + 1 + c) * n + j + 1;
        double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
        int i = l;
        for (; i + 192 < mm; i += 256) {
            s0 += cp[i] * s_v[i];
            s1 += cp[i + 64] * s_v[i + 64];
            s2 += cp[i + 128] * s_v[i + 128];
            s3 += cp[i + 192] * s_v[i + 192];
        }
        for (; i < mm; i += 64) s0 += cp[i] * s_v[i];
        // the panel's correction V (W^T v) + W (V^T v) of row gi, one term per lane
        // (p <= NB < 64), folded into the same wave reduction
        const int gi = j + 1 + c;
        double corr = 0.0;
        if (l < p) corr = m.V[gi + (int64_t)l * n] * zz[l] + m.W[gi + (int64_t)l * n] * zz[NB + l];
        const double s = wave_sum(((s0 + s1) + (s2 + s3)) - corr);
        if (l == 0) m.W[gi + (int64_t)p * n] = t * s;
    }
}

__global__ void __launch_bounds__(WG) k_trd_fin(LocalArgs A, const int32_t* big, int j0) {
    __shared__ double red[WG / 64];
    const Mat m = mat_of(A, big[blockIdx.x]);
    const int pc = min(NB, m.n - 2 - j0);
    if (pc <= 0) return;
    finish_w(m, j0 + pc - 1, pc - 1, red);
}

// C[r0:, r0:] -= V W^T + W V^T over lower tile pairs, stored to both triangles
__global__ void __launch_bounds__(WG) k_trd_update(LocalArgs A, const int32_t* big, int j0) {
    __shared__ mg::Smem sm;
    const Mat m = mat_of(A, big[blockIdx.y]);
    const int n = m.n;
    const int pc = min(NB, n - 2 - j0);
    if (pc <= 0) return;
    const int r0 = j0 + pc, M = n - r0;
    const int mt = (M + mg::T - 1) / mg::T;
    int job = (int)blockIdx.x;
    if (job >= mt * (mt + 1) / 2) return;
    int jt = 0;
    while (job >= mt - jt) {
        job -= mt - jt;
        ++jt;
    }
    const int it = jt + job;
    const double* Vr = m.V + r0;                 // (k = reflector, i = row) at Vr[i + k n]
    const double* Wr = m.W + r0;
    mg::d4 acc[2][2];
    mg::zero(acc);
    mg::tile_mma<mg::IMAJ, mg::IMAJ>(sm, Vr, n, it * mg::T, M, Wr, n, jt * mg::T, M, 0, pc, acc);
    mg::tile_mma<mg::IMAJ, mg::IMAJ>(sm, Wr, n, it * mg::T, M, Vr, n, jt * mg::T, M, 0, pc, acc);
    double old[2][2][4];   // loaded before use, addresses clamped (no conditional loads)
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int64_t rr = r0 + min(it * mg::T + mg::acc_row(p, e), M - 1);
                const int64_t cc = r0 + min(jt * mg::T + mg::acc_col(q), M - 1);
                old[p][q][e] = m.a[rr + cc * n];
            }
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = it * mg::T + mg::acc_row(p, e), c = jt * mg::T + mg::acc_col(q);
                if (i < M && c < M && i >= c) {
                    const int64_t rr = r0 + i, cc = r0 + c;
                    const double x = old[p][q][e] - acc[p][q][e];
                    m.a[rr + cc * n] = x;
                    if (i != c) m.a[cc + rr * n] = x;
                }
            }
}

__global__ void k_trd_tail(LocalArgs A, const int32_t* big) {
    const Mat m = mat_of(A, big[blockIdx.x]);
    const int n = m.n;
    if (tid() == 0 && n >= 3) {
        m.d[n - 2] = m.a[(n - 2) + (int64_t)(n - 2) * n];
        m.e[n - 2] = m.a[(n - 1) + (int64_t)(n - 2) * n];
        m.d[n - 1] = m.a[(n - 1) + (int64_t)(n - 1) * n];
    }
}

// All eigenvalues of the large problems' tridiagonal matrices by bisection,
// WG of them per workgroup (before the mode-count phase of k_local_eig).
__global__ void __launch_bounds__(WG) k_trd_bisect(LocalArgs A, const int32_t* big) {
    __shared__ double red[WG / 64];
    const int b = big[blockIdx.y];
    const int ag = A.first + b;
    const int n = (int)(A.agg_ptr[ag + 1] - A.agg_ptr[ag]);
    const int i0 = (int)blockIdx.x * WG;
    if (i0 >= n) return;
    const double* T = A.t_buf + A.t_off[b];
    wg_bisect_range(T, T + n, n, A.mu + A.mu_off[ag], i0, min(n, i0 + WG), red);
}

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

// 1 / x for normal x whose reciprocal is normal: the hardware's estimate and two Newton
// steps (each doubles its bits), about half the chain of a division
__device__ inline double quick_rcp(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    return fma(fma(-x, r, 1.0), r, r);
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

// Members of one cluster (cl[t] equal) are made orthonormal, members of different ones only
// normalised: with D the inverse column norms and the cross-cluster entries of the Gram
// matrix left out, D Y^T Y D = L L^T and Y <- Y D L^{-T}, the Q that Gram-Schmidt in index
// order gives per cluster (Y: n x bn, row-major, ld 64).  The Gram matrix and the product with the 64 x 64 inverse run on the matrix cores
// (row-wise substitution, 2016 dependent loads a row, took about 1 ms a pass at n = 882),
// the Cholesky factor and its inverse in LDS.  False, with Y unchanged, when a pivot falls
// below 1e-12, where one pass would lose orthogonality.  M: 64 x 64 doubles of scratch.
__device__ inline bool batch_cholqr(mg::Smem& sm, double* Y, int n, int bn, const int* cl, double* M) {
    __shared__ double s_d[64], s_col[2][64], s_piv[64];
    __shared__ int s_ok;
    constexpr int LD = 65;
    double* G = reinterpret_cast<double*>(&sm);                // bn x bn, leading dimension 65
    static_assert(sizeof(mg::Smem) >= 64 * LD * sizeof(double), "Gram matrix in the staging buffers");
    mg::d4 acc[2][2];
    mg::zero(acc);
    mg::tile_mma<mg::IMAJ, mg::IMAJ>(sm, Y, 64, 0, bn, Y, 64, 0, bn, 0, n, acc);
    __syncthreads();
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = mg::acc_row(p, v), j = mg::acc_col(q);
                G[i + j * LD] = i < bn && j < bn ? (cl[i] == cl[j] ? acc[p][q][v] : 0.0) : (i == j ? 1.0 : 0.0);
            }
    if (tid() == 0) s_ok = 1;
    __syncthreads();
    if (tid() < 64) {
        const double g = G[tid() * (LD + 1)];
        s_d[tid()] = g > 0.0 ? 1.0 / sqrt(g) : 0.0;
    }
    __syncthreads();
    // thread (row i, columns k = g mod 4) of the scaled matrix; column j is final when its
    // step begins, one barrier a step (two column buffers)
    const int i = tid() & 63, g = tid() >> 6;
    double x[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) x[u] = G[i + (4 * u + g) * LD] * s_d[i] * s_d[4 * u + g];
#pragma unroll
    for (int j = 0; j < 64; ++j) {
        if (j >= bn) break;                                    // the rest is the identity
        if (g == (j & 3)) s_col[j & 1][i] = x[j >> 2];
        __syncthreads();
        const double* c = s_col[j & 1];
        const double pj = c[j];
        if (!(pj > 1e-12) && j < bn && tid() == 0) s_ok = 0;
        const double r = pj > 1e-12 ? quick_rcp(pj) : 0.0, li = c[i] * r;
#pragma unroll
        for (int u = j >> 2; u < 16; ++u)
            if (4 * u + g > j) x[u] -= li * c[4 * u + g];
        if (tid() == j) s_piv[j] = pj;
    }
    __syncthreads();
    const bool ok = s_ok != 0;
    if (!ok) {
        __syncthreads();
        return false;
    }
    if (tid() < 64) s_piv[tid()] = tid() < bn ? 1.0 / sqrt(s_piv[tid()]) : 1.0;   // 1 / L(j, j)
    __syncthreads();
    // M = D L^{-T}: thread c solves L z = e_c (z = column c of L^{-1}), four threads a column,
    // rows r = 4 u + s; M(k, j) = s_d[k] (L^{-1})(j, k)
#pragma unroll
    for (int u = 0; u < 16; ++u) G[i + (4 * u + g) * LD] = x[u] * s_piv[4 * u + g];   // (rows above: unused)
    __syncthreads();
    {
        const int c = tid() >> 2, s = tid() & 3;
        double z[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) z[u] = 4 * u + s == c ? 1.0 : 0.0;
#pragma unroll
        for (int j = 0; j < 64; ++j) {
            if (j >= bn) break;
            double zj = z[j >> 2] * s_piv[j];
            zj = __shfl(zj, (tid() & 60) + (j & 3), 64);
            if (s == (j & 3)) z[j >> 2] = zj;
#pragma unroll
            for (int u = j >> 2; u < 16; ++u)
                if (4 * u + s > j) z[u] -= G[4 * u + s + j * LD] * zj;
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) M[c + (4 * u + s) * 64] = s_d[c] * z[u];
    }
    __syncthreads();
    for (int r0 = 0; r0 < n; r0 += mg::T) {
        mg::zero(acc);
        // the rows of this tile are in LDS before the product ends: updated in place
        mg::tile_mma<mg::KMAJ, mg::KMAJ>(sm, Y, 64, r0, n, M, 64, 0, bn, 0, bn, acc);
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int r = r0 + mg::acc_row(p, v), t = mg::acc_col(q);
                    if (r < n && t < bn) Y[(int64_t)r * 64 + t] = acc[p][q][v];
                }
    }
    __syncthreads();
    return true;
}

// Retained eigenvectors of the large problems' tridiagonal matrices by inverse iteration.
// Eigenvalues closer than 1e-4 ||T|| form a cluster; workgroup x takes the clusters that
// start at the eigenvalue indices [64x, 64x + 64), as many whole ones at a time as 64 lanes
// hold (symmetric aggregates have dozens of pairs and triples; one cluster at a time took 7
// ms), a larger cluster 64 members at a time: solve every member's system on its own lane,
// make the batch orthogonal to the cluster's earlier members, then orthonormal (Cholesky QR;
// Gram-Schmidt member by member where that is refused).  The batch stays row-major in the
// scratch, interleaved by lane for the solves and an operand of the matrix cores as it is;
// its last iteration orthogonalises twice, the others once (they only have to keep the
// members apart).
//
// Convergence: from the second solve on, the iterate entering a solve has unit norm, so the
// norm of the result is the solve's growth 1 / |lambda - shift| along the eigenvector; once it
// exceeds 1 / (1e-10 ||T||) (shift within 1e-10 ||T|| of an eigenvalue, at least 1e-4 ||T||
// from every other cluster) each further solve would shrink the error by at least 1e6, and
// the iteration stops when every member is there (at most 4 solves).
//
// Bound by the serial chains of the solves and of the 64-column factorisations, not by
// bytes.  FIGURES
__global__ void __launch_bounds__(WG) k_trd_invit(LocalArgs A, const int32_t* big, const int64_t* iw_off,
                                                  double* iw) {
    __shared__ double red[WG / 64];
    __shared__ double s_dot[64];
    __shared__ int s_cl[64];
    __shared__ int s_conv;
    __shared__ mg::Smem sm;
    extern __shared__ double s_dyn[];
    unsigned char* first = reinterpret_cast<unsigned char*>(s_dyn);   // kk + 1: a cluster starts here
    const int b = big[blockIdx.y];
    const int ag = A.first + b;
    const int n = (int)(A.agg_ptr[ag + 1] - A.agg_ptr[ag]);
    const int kk = A.k_out[ag];
    const int r0 = (int)blockIdx.x * 64, r1 = min(kk, r0 + 64);
    if (r0 >= kk) return;
    const double* d = A.t_buf + A.t_off[b];
    const double* e = d + n;
    const double* lam = A.mu + A.mu_off[ag];
    double* V = A.w1 + A.ws_off[b];                    // n x kk, column-major
    double tnorm = 0.0;
    for (int i = tid(); i < n; i += WG)
        tnorm = fmax(tnorm, fabs(d[i]) + (i > 0 ? fabs(e[i - 1]) : 0.0) + (i + 1 < n ? fabs(e[i]) : 0.0));
    tnorm = fmax(wg_max(tnorm, red), 1e-300);
    double* ws = iw + iw_off[blockIdx.y] + (int64_t)blockIdx.x * ((int64_t)INVIT_BLK_SLOTS * n + 4096 + 64);
    double* dd = ws + (int64_t)INVIT_BLK_SLOTS * n + 64;   // 64 x 64
    double* Y = ws + (int64_t)3 * 64 * n;              // n x 64, row-major: the lanes' iterates
    for (int i = tid(); i <= kk; i += WG)
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
            s_cl[tid()] = c;
        }
        for (int64_t q = tid(); q < (int64_t)64 * n; q += WG) {
            const int t = (int)(q & 63), k = (int)(q >> 6);
            Y[q] = t < bn ? start_value(b0 + t, k) : 0.0;
        }
        __syncthreads();
        for (int it = 0; it < 4; ++it) {
            if (tid() == 0) s_conv = it >= 1;
            __syncthreads();
            if (tid() < bn) {
                const int i = b0 + tid();
                const TriLane L = tri_lane(ws, n, tid());
                if (it == 0) tri_factor_solve(d, e, n, lam[i] + (i - s_cl[tid()]) * 2.0 * tiny, L, tiny);
                else tri_apply_factor(n, L);
                const double nr = tri_back(n, L);
                if (!(nr >= grow2)) s_conv = 0;
            }
            __syncthreads();
            const bool last = s_conv != 0 || it == 3;
            for (int pass = 0; pass < (last ? 2 : 1); ++pass) {
                // against the earlier members of the cluster, 64 at a time
                for (int q0 = qa; q0 < b0; q0 += 64) {
                    const double* Q = V + (int64_t)q0 * n;
                    const int qn = min(64, b0 - q0);
                    mg::d4 acc[2][2];
                    mg::zero(acc);
                    mg::tile_mma<mg::KMAJ, mg::IMAJ>(sm, Q, n, 0, qn, Y, 64, 0, bn, 0, n, acc);
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
                        mg::tile_mma<mg::IMAJ, mg::KMAJ>(sm, Q + t0, n, 0, n - t0, dd, qn, 0, bn, 0, qn, acc);
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
                if (batch_cholqr(sm, Y, n, bn, s_cl, dd)) continue;
                // member by member, each normalised before its use
                for (int t = 0; t < bn; ++t) {
                    const int w = tid() >> 6, l = tid() & 63, t0 = max(0, s_cl[t] - b0);
                    for (int s0 = t0 + w; s0 < t; s0 += WG / 64) {
                        double s = 0.0;
                        for (int k = l; k < n; k += 64) s += Y[(int64_t)k * 64 + s0] * Y[(int64_t)k * 64 + t];
                        s = wave_sum(s);
                        if (l == 0) s_dot[s0] = s;
                    }
                    __syncthreads();
                    double nr = 0.0;
                    for (int k = tid(); k < n; k += WG) {
                        double s = 0.0;
                        for (int s0 = t0; s0 < t; ++s0) s += Y[(int64_t)k * 64 + s0] * s_dot[s0];
                        const double v = Y[(int64_t)k * 64 + t] - s;
                        Y[(int64_t)k * 64 + t] = v;
                        nr += v * v;
                    }
                    nr = wg_sum(nr, red);
                    const double sc = 1.0 / sqrt(nr);
                    for (int k = tid(); k < n; k += WG) Y[(int64_t)k * 64 + t] *= sc;
                    __syncthreads();
                }
            }
            if (last) break;
        }
        // to V, column-major, through LDS tiles: rows contiguous on both sides
        double* s = reinterpret_cast<double*>(&sm);    // 64 x 65
        for (int k0 = 0; k0 < n; k0 += 64) {
            __syncthreads();
            for (int q = tid(); q < 64 * 64; q += WG)
                s[(q & 63) * 65 + (q >> 6)] = Y[(int64_t)min(k0 + (q >> 6), n - 1) * 64 + (q & 63)];
            __syncthreads();
            for (int q = tid(); q < 64 * 64; q += WG) {
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
        if (end > b0) {
            batch(b0, end - b0, b0);
            b0 = end;
        } else {
            for (int m = b0; m < ce; m += 64) batch(m, min(64, ce - m), b0);
            b0 = ce;
        }
    }
}

// Retained eigenvectors x <- Q x (Q = H_0 ... H_{n-3}) for the large
// problems: one wave per vector (VS = W1, n x k, ld n), reflectors applied
// from the last to the first, four per round: with the dots d_k = v_k^T x and
// the cross products c_kl = v_k^T v_l of reflectors j, j-1, j-2, j-3 (k = 0..3)
// gathered in one pass, s_k = tau_k (d_k - sum_{l<k} s_l c_kl) are the
// multipliers of applying them one after the other, and x -= sum_k s_k v_k.
// Lane l owns the rows r = l (mod 64) of its vector, so no lane reads another
// lane's writes.
__global__ void __launch_bounds__(WG) k_trd_backtransform(LocalArgs A, const int32_t* big) {
    const int b = big[blockIdx.y];
    const int ag = A.first + b;
    const int n = (int)(A.agg_ptr[ag + 1] - A.agg_ptr[ag]);
    const int kk = A.k_out[ag];
    const int c = (int)blockIdx.x * (WG / 64) + (tid() >> 6);
    if (c >= kk) return;
    const int l = tid() & 63;
    const double* a = A.s_buf + A.sq_off[b];
    const double* tau = A.t_buf + A.t_off[b] + 2 * n;
    double* x = A.w1 + A.ws_off[b] + (int64_t)c * n;
    // entry r of reflector jj: 1 at jj + 1, stored below it, 0 above
    auto vr = [&](int jj, int r) { return r == jj + 1 ? 1.0 : (r > jj + 1 ? a[r + (int64_t)jj * n] : 0.0); };
    int j = n - 3;
    for (; j >= 3; j -= 4) {
        const int r0 = j - 2 + ((l - (j - 2)) % 64 + 64) % 64;     // first owned row >= j - 2
        double d[4] = {0.0, 0.0, 0.0, 0.0}, cc[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        for (int r = r0; r < n; r += 64) {
            const double xr = x[r];
            double v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = vr(j - k, r);
#pragma unroll
            for (int k = 0; k < 4; ++k) d[k] += v[k] * xr;
            cc[0] += v[1] * v[0];
            cc[1] += v[2] * v[0];
            cc[2] += v[2] * v[1];
            cc[3] += v[3] * v[0];
            cc[4] += v[3] * v[1];
            cc[5] += v[3] * v[2];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) d[k] = wave_sum(d[k]);
#pragma unroll
        for (int q = 0; q < 6; ++q) cc[q] = wave_sum(cc[q]);
        double sk[4];
        sk[0] = tau[j] * d[0];
        sk[1] = tau[j - 1] * (d[1] - sk[0] * cc[0]);
        sk[2] = tau[j - 2] * (d[2] - sk[0] * cc[1] - sk[1] * cc[2]);
        sk[3] = tau[j - 3] * (d[3] - sk[0] * cc[3] - sk[1] * cc[4] - sk[2] * cc[5]);
        for (int r = r0; r < n; r += 64) {
            double y = x[r];
#pragma unroll
            for (int k = 0; k < 4; ++k) y -= sk[k] * vr(j - k, r);
            x[r] = y;
        }
    }
    for (; j >= 0; --j) {
        const double t = tau[j];
        if (t == 0.0) continue;
        const double* v = a + (int64_t)j * n;
        const int r0 = j + 1 + ((l - (j + 1)) % 64 + 64) % 64;     // first owned row > j
        double s = 0.0;
        for (int r = r0; r < n; r += 64) s += (r == j + 1 ? 1.0 : v[r]) * x[r];
        s = wave_sum(s) * t;
        for (int r = r0; r < n; r += 64) x[r] -= s * (r == j + 1 ? 1.0 : v[r]);
    }
}

}  // namespace

void launch_local_backtransform_blocked(const LocalArgs& a, const int32_t* d_big, const std::vector<int32_t>& sizes,
                                        hipStream_t st) {
    const int nbig = (int)sizes.size();
    if (nbig == 0) return;
    int max_n = 0;
    for (int32_t s : sizes) max_n = std::max(max_n, (int)s);
    hipLaunchKernelGGL(k_trd_backtransform, dim3((max_n + WG / 64 - 1) / (WG / 64), nbig), dim3(WG), 0, st, a, d_big);
}

void launch_local_invit_blocked(const LocalArgs& a, const int32_t* d_big, const std::vector<int32_t>& sizes,
                                const std::vector<int32_t>& ks, const int64_t* d_iw_off, double* iw, hipStream_t st) {
    const int nbig = (int)sizes.size();
    int max_n = 0, max_g = 0;
    for (int i = 0; i < nbig; ++i) {
        max_n = std::max(max_n, (int)sizes[i]);
        max_g = std::max(max_g, (ks[i] + 63) / 64);
    }
    if (max_g == 0) return;
    const size_t lds = (size_t)max_n + 8;                                         // cluster starts
    hipLaunchKernelGGL(k_trd_invit, dim3(max_g, nbig), dim3(WG), lds, st, a, d_big, d_iw_off, iw);
}

void launch_local_tridiag_blocked(const LocalArgs& a, const int32_t* d_big, const std::vector<int32_t>& sizes,
                                  hipStream_t st) {
    const int nbig = (int)sizes.size();
    if (nbig == 0) return;
    int max_n = 0;
    for (int32_t s : sizes) {
        if (s <= 2 * NB + 1) throw std::runtime_error("blocked tridiagonalisation needs n > 2 * TRD_NB + 1");
        max_n = std::max(max_n, (int)s);
    }
    const size_t lds = (size_t)(max_n + 2 * NB) * sizeof(double);
    for (int j0 = 0; j0 < max_n - 2; j0 += NB) {
        const int j1 = std::min(j0 + NB, max_n - 2);
        for (int j = j0; j < j1; ++j) {
            hipLaunchKernelGGL(k_trd_col, dim3(nbig), dim3(WG), 0, st, a, d_big, j, j0);
            const int mm = max_n - j - 1;
            hipLaunchKernelGGL(k_trd_symv, dim3((mm + CPG - 1) / CPG, nbig), dim3(WG), lds, st, a, d_big, j, j0);
        }
        hipLaunchKernelGGL(k_trd_fin, dim3(nbig), dim3(WG), 0, st, a, d_big, j0);
        int64_t jobs = 0;
        for (int32_t n : sizes) {
            const int pc = std::min(NB, (int)n - 2 - j0);
            if (pc <= 0) continue;
            const int64_t mt = (n - j0 - pc + mg::T - 1) / mg::T;
            jobs = std::max(jobs, mt * (mt + 1) / 2);
        }
        if (jobs > 0) hipLaunchKernelGGL(k_trd_update, dim3((unsigned)jobs, nbig), dim3(WG), 0, st, a, d_big, j0);
    }
    hipLaunchKernelGGL(k_trd_tail, dim3(nbig), dim3(64), 0, st, a, d_big);
    hipLaunchKernelGGL(k_trd_bisect, dim3((max_n + WG - 1) / WG, nbig), dim3(WG), 0, st, a, d_big);
}

}  // namespace lsdd
