// Workgroup-cooperative dense linear algebra for the batched local problems.
//
// Every routine is executed by all threads of one workgroup (blockDim.x ==
// LSDD_WG) on one matrix; matrices are column-major with a leading dimension
// and may live in LDS or in global memory (flat addressing).  The routines
// synchronise internally and leave the workgroup synchronised on return.
#pragma once
#include <hip/hip_runtime.h>

#include <cmath>

#include "consts.hpp"
#include "lanes.hpp"
#include "mgemm.hpp"

#define LSDD_WG 256

namespace lsdd {

__device__ inline int tid() { return (int)threadIdx.x; }

// ---------------------------------------------------------------- reductions

template <typename T>
__device__ inline T wave_sum(T v) {
    return sum_lanes<64>(v);
}

template <typename T>
__device__ inline T wave_max(T v) {
    for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
    return v;
}

// Workgroup sum; `red` is LDS scratch of at least LSDD_WG/64 entries.
template <typename T>
__device__ inline T wg_sum(T v, T* red) {
    v = wave_sum(v);
    const int w = tid() >> 6, l = tid() & 63;
    __syncthreads();
    if (l == 0) red[w] = v;
    __syncthreads();
    T s = 0;
    for (int i = 0; i < LSDD_WG / 64; ++i) s += red[i];
    __syncthreads();
    return s;
}

template <typename T>
__device__ inline T wg_max(T v, T* red) {
    v = wave_max(v);
    const int w = tid() >> 6, l = tid() & 63;
    __syncthreads();
    if (l == 0) red[w] = v;
    __syncthreads();
    T s = red[0];
    for (int i = 1; i < LSDD_WG / 64; ++i) s = fmax(s, red[i]);
    __syncthreads();
    return s;
}

// ---------------------------------------------------------------- elementary ops

__device__ inline void wg_zero(double* a, long long count) {
    for (long long i = tid(); i < count; i += LSDD_WG) a[i] = 0.0;
    __syncthreads();
}

__device__ inline void wg_identity(double* a, int ld, int n) {
    for (int j = tid() >> 6; j < n; j += LSDD_WG / 64)
        for (int i = tid() & 63; i < n; i += 64) a[i + (long long)j * ld] = (i == j) ? 1.0 : 0.0;
    __syncthreads();
}

// a <- (a + a^T)/2 on an n x n block.
__device__ inline void wg_symmetrize(double* a, int ld, int n) {
    for (long long idx = tid(); idx < (long long)n * n; idx += LSDD_WG) {
        int i = (int)(idx % n), j = (int)(idx / n);
        if (i < j) {
            double s = 0.5 * (a[i + (long long)j * ld] + a[j + (long long)i * ld]);
            a[i + (long long)j * ld] = s;
            a[j + (long long)i * ld] = s;
        }
    }
    __syncthreads();
}

// In-place transpose of a square n x n block.
__device__ inline void wg_transpose(double* a, int ld, int n) {
    for (long long idx = tid(); idx < (long long)n * n; idx += LSDD_WG) {
        int i = (int)(idx % n), j = (int)(idx / n);
        if (i < j) {
            double t = a[i + (long long)j * ld];
            a[i + (long long)j * ld] = a[j + (long long)i * ld];
            a[j + (long long)i * ld] = t;
        }
    }
    __syncthreads();
}

// ---------------------------------------------------------------- Cholesky

// Right-looking Cholesky A = L L^T of an SPD n x n matrix, lower triangle in
// place.  Returns the smallest pivot d_j = L_jj^2 seen (<= 0 or NaN: failed at
// that column, the factor is incomplete).  `sh` is LDS scratch of 2 doubles.
__device__ inline double wg_potrf(double* a, int ld, int n, double* sh) {
    if (tid() == 0) sh[1] = INFINITY;
    __syncthreads();
    for (int j = 0; j < n; ++j) {
        if (tid() == 0) {
            double d = a[j + (long long)j * ld];
            sh[1] = fmin(sh[1], d);
            if (!(d > 0.0)) sh[1] = (d == d) ? d : -1.0;
            double s = (d > 0.0) ? sqrt(d) : 0.0;
            a[j + (long long)j * ld] = s;
            sh[0] = s;
        }
        __syncthreads();
        const double s = sh[0];
        if (!(s > 0.0)) {
            double r = sh[1];
            __syncthreads();
            return r;
        }
        const double inv = 1.0 / s;
        double* cj = a + (long long)j * ld;
        for (int i = j + 1 + tid(); i < n; i += LSDD_WG) cj[i] *= inv;
        __syncthreads();
        const int m = n - j - 1;
        for (long long idx = tid(); idx < (long long)m * m; idx += LSDD_WG) {
            int ii = (int)(idx % m), kk = (int)(idx / m);
            if (ii >= kk) {
                int i = j + 1 + ii, k = j + 1 + kk;
                a[i + (long long)k * ld] -= cj[i] * cj[k];
            }
        }
        __syncthreads();
    }
    double r = sh[1];
    __syncthreads();
    return r;
}

// Forward solve L X = B in place (L lower n x n, B n x m).
__device__ inline void wg_trsm_lower(const double* L, int ldl, int n, double* B, int ldb, int m) {
    for (int j = 0; j < n; ++j) {
        const double inv = 1.0 / L[j + (long long)j * ldl];
        for (int c = tid(); c < m; c += LSDD_WG) B[j + (long long)c * ldb] *= inv;
        __syncthreads();
        const int r = n - j - 1;
        if (r > 0) {
            const double* lj = L + (long long)j * ldl;
            for (long long idx = tid(); idx < (long long)r * m; idx += LSDD_WG) {
                int ii = (int)(idx % r), c = (int)(idx / r);
                int i = j + 1 + ii;
                B[i + (long long)c * ldb] -= lj[i] * B[j + (long long)c * ldb];
            }
        }
        __syncthreads();
    }
}

// Backward solve L^T X = B in place (L lower n x n, B n x m).
__device__ inline void wg_trsm_lower_t(const double* L, int ldl, int n, double* B, int ldb, int m) {
    for (int j = n - 1; j >= 0; --j) {
        const double inv = 1.0 / L[j + (long long)j * ldl];
        for (int c = tid(); c < m; c += LSDD_WG) B[j + (long long)c * ldb] *= inv;
        __syncthreads();
        if (j > 0) {
            for (long long idx = tid(); idx < (long long)j * m; idx += LSDD_WG) {
                int i = (int)(idx % j), c = (int)(idx / j);
                B[i + (long long)c * ldb] -= L[j + (long long)i * ldl] * B[j + (long long)c * ldb];
            }
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------- Jacobi eigensolver

// Parallel cyclic Jacobi (round-robin ordering) on a symmetric n x n matrix a, n <= JAC_N.
// On return a is diagonal up to the rotation threshold (eigenvalues on the
// diagonal) and v (n x n) holds the eigenvectors as columns (v must be the
// identity, or any orthogonal start, on entry).  A pair is rotated when
// |a_pq| > rel * sqrt(|a_pp a_qq|) and |a_pq| > abs_tol; the sweep loop stops after a sweep
// that rotated no |a_pq| > conv_tol (the unit roundoff of the largest entry: what is left is
// then below the rounding of the rotations themselves).  A singular block has no end of
// rotations among its null vectors, whose entries are that rounding: stopped by the rotations'
// own thresholds, the 24 x 24 grad-div and 8 x 8 elasticity blocks took all 60 sweeps, now 10
// and 6, with the same residual and vectors closer to orthogonal.  LDS scratch: `pairs` (2 * npair ints),
// `cs` (2 * npair doubles), `flag` (1 int) with npair = (n + 1) / 2.
//
// A round is two steps: the rotations (a lane per pair), then A <- J^T A J by 2 x 2 blocks, a
// thread per pair of pairs, rows before columns, together with V <- V J.  Its cost is LDS
// traffic and integer work: which blocks a thread owns does not change between the rounds and
// is worked out once (a 64-bit division an entry took more time than the rotations), and each
// entry is read and written once a round.  1600 blocks of 24 x 24: 2.4 ->
// 1.36 ms, 2304 of 8 x 8: 0.68 -> 0.30 ms.
constexpr int JAC_N = 48;
__device__ inline int wg_jacobi(double* a, int lda, int n, double* v, int ldv, int max_sweeps,
                                double rel, double abs_tol, double conv_tol, int* pairs, double* cs, int* flag) {
    constexpr int U = (JAC_N / 2 * (JAC_N / 2 + JAC_N) + LSDD_WG - 1) / LSDD_WG;
    const int np = n + (n & 1);
    const int npair = np / 2;
    // work item (r, l): r < npair block of pairs (r, l) of A, else row r - npair of V, pair l
    int it_l[U], it_r[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int idx = tid() + u * LSDD_WG;
        it_l[u] = idx / (npair + n);
        it_r[u] = idx - it_l[u] * (npair + n);
    }
    int sweep = 0;
    for (; sweep < max_sweeps; ++sweep) {
        if (tid() == 0) *flag = 0;
        __syncthreads();
        for (int rnd = 0; rnd < np - 1; ++rnd) {
            if (tid() < npair) {
                const int k = tid();
                auto turn = [&](int i) {               // index 0 stays, the others move on by rnd
                    const int x = i - 1 + rnd;
                    return i == 0 ? 0 : 1 + (x >= np - 1 ? x - (np - 1) : x);
                };
                const int x = turn(k), y = turn(np - 1 - k);
                const int p = min(x, y), q = max(x, y);
                double c = 1.0, s = 0.0;
                if (q < n) {
                    double app = a[p + p * lda], aqq = a[q + q * lda];
                    double apq = a[p + q * lda];
                    if (fabs(apq) > abs_tol && fabs(apq) > rel * sqrt(fabs(app * aqq))) {
                        double th = (aqq - app) / (2.0 * apq);
                        double t = (th >= 0.0 ? 1.0 : -1.0) / (fabs(th) + sqrt(th * th + 1.0));
                        c = 1.0 / sqrt(t * t + 1.0);
                        s = t * c;
                        if (fabs(apq) > conv_tol) *flag = 1;
                    }
                }
                pairs[2 * k] = p;
                pairs[2 * k + 1] = (q < n) ? q : -1;
                cs[2 * k] = c;
                cs[2 * k + 1] = s;
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int l = it_l[u], r = it_r[u];
                if (l >= npair) break;
                const int pl = pairs[2 * l], ql = pairs[2 * l + 1];
                const double cl = cs[2 * l], sl = cs[2 * l + 1];
                if (r >= npair) {                      // V <- V J
                    if (sl == 0.0) continue;
                    double* vp = v + (r - npair) + pl * ldv;
                    double* vq = v + (r - npair) + ql * ldv;
                    const double x = *vp, y = *vq;
                    *vp = cl * x - sl * y;
                    *vq = sl * x + cl * y;
                    continue;
                }
                const int pr = pairs[2 * r], qr = pairs[2 * r + 1];
                const double cr = cs[2 * r], sr = cs[2 * r + 1];
                if (sl == 0.0 && sr == 0.0) continue;
                // a pair without a partner (odd n) has s = 0: its entries are read twice and
                // written once
                const int qr_ = qr < 0 ? pr : qr, ql_ = ql < 0 ? pl : ql;
                double x00 = a[pr + pl * lda], x10 = a[qr_ + pl * lda];
                double x01 = a[pr + ql_ * lda], x11 = a[qr_ + ql_ * lda];
                const double y00 = cr * x00 - sr * x10, y10 = sr * x00 + cr * x10;
                const double y01 = cr * x01 - sr * x11, y11 = sr * x01 + cr * x11;
                x00 = cl * y00 - sl * y01;
                x01 = sl * y00 + cl * y01;
                x10 = cl * y10 - sl * y11;
                x11 = sl * y10 + cl * y11;
                a[pr + pl * lda] = x00;
                if (qr >= 0) a[qr + pl * lda] = x10;
                if (ql >= 0) a[pr + ql * lda] = x01;
                if (qr >= 0 && ql >= 0) a[qr + ql * lda] = x11;
            }
            __syncthreads();
        }
        int any = *flag;
        __syncthreads();
        if (!any) break;
    }
    return sweep;
}

// After wg_jacobi: write eigenvalues ascending into w[n] and the matching
// eigenvectors (columns of v) into vs (n x n, ldvs).  Ties keep index order.
__device__ inline void wg_sort_eig(const double* a, int lda, const double* v, int ldv, int n,
                                   double* w, double* vs, int ldvs, int* rank_scratch) {
    for (int i = tid(); i < n; i += LSDD_WG) {
        double di = a[i + (long long)i * lda];
        int r = 0;
        for (int j = 0; j < n; ++j) {
            double dj = a[j + (long long)j * lda];
            r += (dj < di) || (dj == di && j < i);
        }
        rank_scratch[i] = r;
        w[r] = di;
    }
    __syncthreads();
    for (int j = tid() >> 6; j < n; j += LSDD_WG / 64)
        for (int i = tid() & 63; i < n; i += 64) vs[i + (long long)rank_scratch[j] * ldvs] = v[i + (long long)j * ldv];
    __syncthreads();
}

}  // namespace lsdd

namespace lsdd {

// ---------------------------------------------------------------- tridiagonal eigensolver

// Householder reduction of the symmetric n x n matrix a (column-major, both
// triangles, ld n) to tridiagonal form T = Q^T A Q.  Outputs d[n], e[n-1],
// tau[n-2]; the Householder vector of step j is stored in a[j+2.., j] (its
// leading entry 1 implicit).  LDS scratch: v, w (n doubles each), red.
__device__ inline void wg_tridiag(double* a, int n, double* d, double* e, double* tau, double* v, double* w,
                                  double* red) {
    for (int j = 0; j + 2 < n; ++j) {
        const int m = n - j - 1;
        double* x = a + (j + 1) + (long long)j * n;           // a[j+1.., j]
        double s2 = 0.0;
        for (int i = 1 + tid(); i < m; i += LSDD_WG) s2 += x[i] * x[i];
        s2 = wg_sum(s2, red);
        const double alpha = x[0];
        double t = 0.0, beta = alpha;
        if (s2 > 0.0) {
            double nrm = sqrt(alpha * alpha + s2);
            beta = alpha >= 0.0 ? -nrm : nrm;
            t = (beta - alpha) / beta;
            const double sc = 1.0 / (alpha - beta);
            for (int i = tid(); i < m; i += LSDD_WG) v[i] = (i == 0) ? 1.0 : x[i] * sc;
        } else {
            for (int i = tid(); i < m; i += LSDD_WG) v[i] = (i == 0) ? 1.0 : 0.0;
        }
        __syncthreads();
        if (tid() == 0) {
            d[j] = a[j + (long long)j * n];
            e[j] = beta;
            tau[j] = t;
        }
        if (t != 0.0) {
            // p = t * A22 v  (A22 = a[j+1.., j+1..])
            double* A22 = a + (j + 1) + (long long)(j + 1) * n;
            for (int i = tid(); i < m; i += LSDD_WG) {
                double s = 0.0;
                for (int k = 0; k < m; ++k) s += A22[i + (long long)k * n] * v[k];
                w[i] = t * s;
            }
            __syncthreads();
            double pv = 0.0;
            for (int i = tid(); i < m; i += LSDD_WG) pv += w[i] * v[i];
            pv = wg_sum(pv, red);
            const double K = 0.5 * t * pv;
            for (int i = tid(); i < m; i += LSDD_WG) w[i] -= K * v[i];
            __syncthreads();
            for (int k = tid() >> 6; k < m; k += LSDD_WG / 64) {      // a wave per column
                const double wk = w[k], vk = v[k];
                for (int i = tid() & 63; i < m; i += 64) A22[i + (long long)k * n] -= v[i] * wk + w[i] * vk;
            }
        }
        // keep the reflector below the subdiagonal
        for (int i = 1 + tid(); i < m; i += LSDD_WG) x[i] = v[i];
        __syncthreads();
    }
    if (tid() == 0) {
        if (n >= 2) {
            d[n - 2] = a[(n - 2) + (long long)(n - 2) * n];
            e[n - 2] = a[(n - 1) + (long long)(n - 2) * n];
        }
        d[n - 1] = a[(n - 1) + (long long)(n - 1) * n];
    }
    __syncthreads();
}

// Eigenvalues of the tridiagonal (d, e) smaller than x (Sturm count; d, and the squares of e
// from e2[1] on, e2[0] = 0).  One chain of n reciprocals; the estimate with two Newton steps
// is within an ulp or two of the division, which is what the count's backward error is anyway.
__device__ inline int sturm_quick(const double* d, const double* e2, int n, double x, double pivmin) {
    int c = 0;
    double q = 1.0;
    constexpr int U = 8;
    int k = 0;
    for (; k + U <= n; k += U) {
        double dk[U], ek[U];
#pragma unroll
        for (int u = 0; u < U; ++u) dk[u] = d[k + u] - x, ek[u] = e2[k + u];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            q = dk[u] - ek[u] * quick_rcp(q);
            q = fabs(q) < pivmin ? -pivmin : q;
            c += q < 0.0;
        }
    }
    for (; k < n; ++k) {
        q = d[k] - x - e2[k] * quick_rcp(q);
        q = fabs(q) < pivmin ? -pivmin : q;
        c += q < 0.0;
    }
    return c;
}

// The bracket [lo, hi] of all eigenvalues, the smallest pivot (its reciprocal times e^2 stays
// finite) and the absolute tolerance; stages d and e^2 (e2[0] = 0) in LDS for sturm_quick.
struct TriBracket {
    double lo, hi, pivmin, atol;
};
__device__ inline TriBracket wg_bracket(const double* d, const double* e, int n, double* s_d, double* s_e2, double* red) {
    double lo = INFINITY, hi = -INFINITY, emax2 = 0.0;
    for (int i = tid(); i < n; i += LSDD_WG) {
        const double el = i > 0 ? e[i - 1] : 0.0, er = i + 1 < n ? e[i] : 0.0, di = d[i];
        const double r = fabs(el) + fabs(er);
        lo = fmin(lo, di - r);
        hi = fmax(hi, di + r);
        emax2 = fmax(emax2, er * er);
        s_d[i] = di;
        s_e2[i] = el * el;
    }
    lo = -wg_max(-lo, red);
    hi = wg_max(hi, red);
    emax2 = wg_max(emax2, red);
    const double tnorm = fmax(fabs(lo), fabs(hi));
    TriBracket B;
    B.pivmin = fmax(2.2250738585072014e-308 * fmax(emax2, 1.0), 1e-290);
    B.atol = 2.0 * 2.220446049250313e-16 * tnorm + 1e-300;
    B.lo = lo - B.atol;
    B.hi = hi + B.atol;
    return B;
}

// All eigenvalues of the symmetric tridiagonal (d, e), ascending, by bisection, one lane per
// eigenvalue (lds: 2 n doubles).
__device__ inline void wg_bisect_all(const double* d, const double* e, int n, double* lam, double* lds, double* red) {
    const TriBracket B = wg_bracket(d, e, n, lds, lds + n, red);
    for (int i = tid(); i < n; i += LSDD_WG) {
        double a = B.lo, b = B.hi;
        for (int it = 0; it < 200; ++it) {
            const double mid = 0.5 * (a + b);
            if (b - a <= 2.0 * 2.220446049250313e-16 * fmax(fabs(a), fabs(b)) + B.atol || mid == a || mid == b) break;
            if (sturm_quick(lds, lds + n, n, mid, B.pivmin) > i) b = mid;
            else a = mid;
        }
        lam[i] = 0.5 * (a + b);
    }
    __syncthreads();
}

// ---------------------------------------------------------------- back-transformation

// x <- Q x (Q = H_0 ... H_{n-3}: reflector j below the subdiagonal of column j of a, its
// leading 1 implicit) for nv <= NV vectors (columns of ld n) in one wave, reflectors applied from the last to the first, four per
// round: with the dots d_k = v_k^T x and the cross products c_kl = v_k^T v_l of reflectors j,
// j-1, j-2, j-3 (k = 0..3) gathered in one pass, s_k = tau_k (d_k - sum_{l<k} s_l c_kl) are
// the multipliers of applying them one after the other, and x -= sum_k s_k v_k.  Lane l owns
// the rows l + 64 i, i < RPT (n <= 64 RPT), and holds them in registers, so that a round goes
// to memory once, for the reflectors; only the rows of the diagonal and of the last block
// need masks.
template <int RPT, int NV>
__device__ inline void wave_backtransform(const double* __restrict__ a, int n, const double* __restrict__ tau,
                                          double* xp, int nv) {
    const int l = tid() & 63;
    double x[NV][RPT];
#pragma unroll
    for (int u = 0; u < NV; ++u)
#pragma unroll
        for (int i = 0; i < RPT; ++i) x[u][i] = xp[(int64_t)min(u, nv - 1) * n + min(l + 64 * i, n - 1)];
    for (int j = n - 3; j >= 0; j -= 4) {
        double d[NV][4] = {}, cc[6] = {};
        double v[RPT][4];
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            if (64 * i + 63 < j - 2 || 64 * i >= n) continue;          // the same in every lane
            const int rc = min(l + 64 * i, n - 1);
#pragma unroll
            for (int k = 0; k < 4; ++k) v[i][k] = a[rc + (int64_t)max(j - k, 0) * n];
        }
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            if (64 * i + 63 < j - 2 || 64 * i >= n) continue;
            if (64 * i <= j + 1 || 64 * i + 64 > n || j < 3) {
                // entry r of reflector q: 1 at q + 1, stored below it, 0 above, past the end
                // and where there is no reflector (q < 0)
                const int r = l + 64 * i;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int q = j - k;
                    v[i][k] = q < 0 || r <= q || r >= n ? 0.0 : (r == q + 1 ? 1.0 : v[i][k]);
                }
            }
#pragma unroll
            for (int u = 0; u < NV; ++u)
#pragma unroll
                for (int k = 0; k < 4; ++k) d[u][k] += v[i][k] * x[u][i];
            cc[0] += v[i][1] * v[i][0];
            cc[1] += v[i][2] * v[i][0];
            cc[2] += v[i][2] * v[i][1];
            cc[3] += v[i][3] * v[i][0];
            cc[4] += v[i][3] * v[i][1];
            cc[5] += v[i][3] * v[i][2];
        }
#pragma unroll
        for (int q = 0; q < 6; ++q) cc[q] = wave_sum(cc[q]);
        const double t0 = tau[j], t1 = tau[max(j - 1, 0)], t2 = tau[max(j - 2, 0)], t3 = tau[max(j - 3, 0)];
#pragma unroll
        for (int u = 0; u < NV; ++u) {
#pragma unroll
            for (int k = 0; k < 4; ++k) d[u][k] = wave_sum(d[u][k]);
            double sk[4];
            sk[0] = t0 * d[u][0];
            sk[1] = t1 * (d[u][1] - sk[0] * cc[0]);
            sk[2] = t2 * (d[u][2] - sk[0] * cc[1] - sk[1] * cc[2]);
            sk[3] = t3 * (d[u][3] - sk[0] * cc[3] - sk[1] * cc[4] - sk[2] * cc[5]);
#pragma unroll
            for (int i = 0; i < RPT; ++i) {
                if (64 * i + 63 < j - 2 || 64 * i >= n) continue;
#pragma unroll
                for (int k = 0; k < 4; ++k) x[u][i] -= sk[k] * v[i][k];
            }
        }
    }
#pragma unroll
    for (int u = 0; u < NV; ++u)
#pragma unroll
        for (int i = 0; i < RPT; ++i)
            if (u < nv && l + 64 * i < n) xp[(int64_t)u * n + l + 64 * i] = x[u][i];
}

// The same for any n, x in memory (no lane reads another lane's writes).
__device__ inline void wave_backtransform_long(const double* a, int n, const double* tau, double* x) {
    const int l = tid() & 63;
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

// V <- Q V for the kk columns of V (n x kk, ld n), dealt to the waves four or two at a time
// where they fit the registers: they share a round's reads and cross products.
__device__ inline void wg_backtransform(const double* a, int n, const double* tau, double* V, int kk) {
    auto deal = [&](int nv, auto apply) {
        for (int c = (tid() >> 6) * nv; c < kk; c += LSDD_WG / 64 * nv) apply(V + (int64_t)c * n, min(nv, kk - c));
    };
    if (n <= 128) deal(4, [&](double* x, int nv) { wave_backtransform<2, 4>(a, n, tau, x, nv); });
    else if (n <= 256) deal(2, [&](double* x, int nv) { wave_backtransform<4, 2>(a, n, tau, x, nv); });
    else deal(1, [&](double* x, int) { wave_backtransform_long(a, n, tau, x); });
    __syncthreads();
}

}  // namespace lsdd
