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
//   k_trd_col   (one workgroup per matrix): finish the previous W column
//               (w = tau (C22 v - V (W^T v) - W (V^T v)), then w -= (tau/2) (w . v) v),
//               correct column j, form reflector v_j (stored in column j, with
//               an explicit 1 on the subdiagonal);
//   k_trd_symv  (many workgroups per matrix): C22 v, four columns of C22 per wave,
//               and the workgroup's rows' share of the dots W^T v and V^T v.
// Per panel: k_trd_col once more for the last W column, k_trd_update.
//
// The column kernel is one serial chain per column, so what counts is how often it goes to
// memory: it reads each row of V and W once, for the previous column's finish and this
// column's correction together, and takes the dots as partial sums from the launch before.
// 54 matrices of up to 648, then 8 of up to 882 columns: 26.5 -> 15 us a column (column
// kernel 16.0 -> 7.7, product 10.5 -> 7.0; 256 rows left: 5.8 and 5.2).
//
// Storage per matrix: C (n x n, both triangles kept exactly symmetric), the
// tridiagonal d, e, tau and the dots' partial sums in the T scratch, V and W (n x
// TRD_NB each, column-major, so row sweeps over one column are coalesced) in the v_buf
// slot (n^2 doubles, n > 2 TRD_NB).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <stdexcept>
#include <vector>

#include "dense.hpp"
#include "kernels.hpp"
#include "mgemm.hpp"
#include "tile64.hpp"

namespace lsdd {

namespace {

constexpr int WG = LSDD_WG;
constexpr int NB = TRD_NB;
constexpr int CPW = 4;               // columns per wave in k_trd_symv
constexpr int CPG = CPW * WG / 64;   // columns per workgroup

// One matrix of the batch; a table of these, so that a launch finds its matrix with one
// dependent load (k_trd_mats fills it).
struct Mat {
    int n, pad;
    double* a;
    double* d;
    double* e;
    double* tau;
    double* V;
    double* W;
    double* zp;                      // per k_trd_symv workgroup: its share of W^T v, V^T v (2 NB)
};

__global__ void k_trd_mats(LocalArgs A, const int32_t* big, int nbig, Mat* out) {
    const int i = (int)blockIdx.x * 64 + tid();
    if (i >= nbig) return;
    const int b = big[i], ag = A.first + b;
    Mat m;
    m.n = (int)(A.agg_ptr[ag + 1] - A.agg_ptr[ag]);
    m.pad = 0;
    m.a = A.s_buf + A.sq_off[b];
    double* T = A.t_buf + A.t_off[b];
    m.d = T;
    m.e = T + m.n;
    m.tau = T + 2 * m.n;
    m.zp = T + 3 * m.n;              // the inverse iteration's scratch, not in use yet
    m.V = A.v_buf + A.sq_off[b];
    m.W = m.V + (int64_t)NB * m.n;
    out[i] = m;
}
static_assert(INVIT_SLOTS * 16 >= 2 * NB, "partial dots fit the scratch: (n / CPG + 1) 2 NB <= INVIT_SLOTS n");

// sum over the workgroup's TH threads, the same in every thread (red: TH / 64 entries)
template <int TH>
__device__ inline double col_sum(double v, double* red) {
    v = sum_lanes<64>(v);
    __syncthreads();
    if ((tid() & 63) == 0) red[tid() >> 6] = v;
    __syncthreads();
    double s = red[0];
#pragma unroll
    for (int q = 1; q < TH / 64; ++q) s += red[q];
    return s;
}

// Column j of the panel that starts at j0 (fin: only the last W column of that panel).  TH
// threads, RPT rows each: the factors of a V, W entry come from LDS for every wave that uses
// them, so up to 1024 rows run on four waves with up to four rows a thread, not on sixteen
// (10.4 against 7.7 us a column, averaged over n = 648 and 882).
template <int TH, int RPT>
__global__ void __launch_bounds__(TH) k_trd_col(const Mat* mats, int j, int j0, int fin) {
    constexpr int QC = RPT <= 2 ? 8 : 4;               // panel columns in flight
    constexpr int PW = TH / 64;
    __shared__ double red[PW];
    __shared__ double part[PW][2 * NB];
    __shared__ __align__(16) double fac[NB][4];        // W^T v, V^T v, rows j of V and W
    __shared__ double s_row[2];
    const Mat m = mats[blockIdx.x];
    const int n = m.n;
    if (fin) {
        const int pc = min(NB, n - 2 - j0);            // this matrix's columns in the panel
        if (pc <= 0) return;
        j = j0 + pc;
    } else if (j + 2 >= n) {
        return;
    }
    const int p = j - j0, qf = p - 1;                  // the W column to finish: qf
    double* col = m.a + (int64_t)j * n;
    double x[RPT];
    int row[RPT];
#pragma unroll
    for (int u = 0; u < RPT; ++u) {
        row[u] = j + tid() + u * TH;
        x[u] = fin ? 0.0 : col[min(row[u], n - 1)];
    }
    if (p > 0) {
        // W^T v and V^T v of reflector j - 1 from the partial sums, rows j of V and W
        const int nblk = (n - j + CPG - 1) / CPG;
        const int sidx = tid() & 63, g = tid() >> 6;
        double y[RPT], v[RPT], vv[RPT][QC], ww[RPT][QC];
        // entries q0 .. q0 + QC - 1 of the rows (columns past qf - 1 have zero factors); the
        // first ones arrive while the factors are formed
        auto fetch = [&](int q0) {
#pragma unroll
            for (int u = 0; u < RPT; ++u)
#pragma unroll
                for (int q = 0; q < QC; ++q) {
                    const int64_t o = min(row[u], n - 1) + (int64_t)min(q0 + q, max(qf - 1, 0)) * n;
                    vv[u][q] = m.V[o];
                    ww[u][q] = m.W[o];
                }
        };
        double z = 0.0;
        for (int q0 = g; q0 < nblk; q0 += 8 * PW) {
            double zz[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) zz[u] = m.zp[(int64_t)min(q0 + u * PW, nblk - 1) * 2 * NB + sidx];
#pragma unroll
            for (int u = 0; u < 8; ++u) z += q0 + u * PW < nblk ? zz[u] : 0.0;
        }
        double rj = 0.0;                               // V(j, q) in lanes 0 .. 31, W(j, q) behind
        if (g == 0) rj = (sidx < NB ? m.V : m.W)[j + (int64_t)min(sidx & (NB - 1), max(qf - 1, 0)) * n];
#pragma unroll
        for (int u = 0; u < RPT; ++u) {
            const int i = min(row[u], n - 1);
            y[u] = m.W[i + (int64_t)qf * n];
            v[u] = m.V[i + (int64_t)qf * n];
        }
        fetch(0);
        const double t = m.tau[j - 1];
        part[g][sidx] = z;
        __syncthreads();
        if (g == 0) {
            double sum = 0.0;
#pragma unroll
            for (int q = 0; q < PW; ++q) sum += part[q][sidx];
            const int q = sidx & (NB - 1);
            const bool in = q < qf;
            fac[q][sidx < NB ? 0 : 1] = in ? sum : 0.0;
            fac[q][sidx < NB ? 3 : 2] = in && !fin ? rj : 0.0;   // V meets W's row and the other way round
        }
        __syncthreads();
        double sv = 0.0, corr[RPT], upd[RPT];
#pragma unroll
        for (int u = 0; u < RPT; ++u) corr[u] = upd[u] = 0.0;
        for (int q0 = 0; q0 < qf; q0 += QC) {
            double vc[RPT][QC], wc[RPT][QC];
#pragma unroll
            for (int u = 0; u < RPT; ++u)
#pragma unroll
                for (int q = 0; q < QC; ++q) vc[u][q] = vv[u][q], wc[u][q] = ww[u][q];
            if (q0 + QC < qf) fetch(q0 + QC);
#pragma unroll
            for (int q = 0; q < QC; ++q) {
                const double2 z2 = *reinterpret_cast<const double2*>(&fac[q0 + q][0]);
                const double2 r2 = *reinterpret_cast<const double2*>(&fac[q0 + q][2]);
#pragma unroll
                for (int u = 0; u < RPT; ++u) {
                    corr[u] += vc[u][q] * z2.x + wc[u][q] * z2.y;
                    upd[u] += vc[u][q] * r2.x + wc[u][q] * r2.y;
                }
            }
        }
#pragma unroll
        for (int u = 0; u < RPT; ++u) {
            y[u] = t * (y[u] - corr[u]);
            if (row[u] < n) sv += y[u] * v[u];
        }
        const double K = 0.5 * t * col_sum<TH>(sv, red);
#pragma unroll
        for (int u = 0; u < RPT; ++u) {
            y[u] -= K * v[u];
            if (row[u] < n) m.W[row[u] + (int64_t)qf * n] = y[u];
        }
        if (fin) return;
        if (tid() == 0) s_row[0] = y[0], s_row[1] = v[0];      // row j
        __syncthreads();
        const double wj = s_row[0], vj = s_row[1];
#pragma unroll
        for (int u = 0; u < RPT; ++u) x[u] -= upd[u] + (v[u] * wj + y[u] * vj);
        __syncthreads();
    } else if (fin) {
        return;
    }
    // reflector from x(j + 1 .. n - 1)
    double s2 = 0.0;
#pragma unroll
    for (int u = 0; u < RPT; ++u) {
        if (row[u] == j) col[j] = x[u], m.d[j] = x[u];
        if (row[u] == j + 1) s_row[0] = x[u];
        if (row[u] > j + 1 && row[u] < n) s2 += x[u] * x[u];
    }
    s2 = col_sum<TH>(s2, red);                         // its barriers publish s_row
    const double alpha = s_row[0];
    double t = 0.0, beta = alpha, sc = 0.0;
    if (s2 > 0.0) {
        const double nrm = sqrt(alpha * alpha + s2);
        beta = alpha >= 0.0 ? -nrm : nrm;
        t = (beta - alpha) / beta;
        sc = 1.0 / (alpha - beta);
    }
    if (tid() == 0) {
        m.e[j] = beta;
        m.tau[j] = t;
    }
    double* vp = m.V + (int64_t)p * n;
#pragma unroll
    for (int u = 0; u < RPT; ++u)
        if (row[u] > j && row[u] < n) {
            const double vi = row[u] == j + 1 ? 1.0 : (s2 > 0.0 ? x[u] * sc : 0.0);
            col[row[u]] = vi;
            vp[row[u]] = vi;
        }
    for (int i = j0 + tid(); i <= j; i += TH) {
        vp[i] = 0.0;
        m.W[i + (int64_t)p * n] = 0.0;
    }
}

// W(:, p) <- C22 v (raw), the partial dots of the workgroup's rows
__global__ void __launch_bounds__(WG) k_trd_symv(const Mat* mats, int j, int j0) {
    __shared__ double s_z[WG / 64][2 * NB];
    const Mat m = mats[blockIdx.y];
    const int n = m.n;
    if (j + 2 >= n) return;
    const int mm = n - j - 1;
    const int c0 = (int)blockIdx.x * CPG;
    if (c0 >= mm) return;
    const int p = j - j0;
    const double* v = m.a + (int64_t)j * n + j + 1;
    const int w = tid() >> 6, l = tid() & 63;
    // this workgroup's rows against column l & 31 of W (l < 32) or V, four rows per wave
    const int64_t qo = (int64_t)min(l & (NB - 1), max(p - 1, 0)) * n;
    const double* M = (l < NB ? m.W : m.V) + qo + j + 1;
    double zr[CPG / (WG / 64)], zx[CPG / (WG / 64)];
#pragma unroll
    for (int u = 0; u < CPG / (WG / 64); ++u) {
        const int i = min(c0 + w * CPW + u, mm - 1);
        zr[u] = M[i];
        zx[u] = v[i];
    }
    const double* cp[CPW];
#pragma unroll
    for (int c = 0; c < CPW; ++c) cp[c] = m.a + (int64_t)(j + 1 + min(c0 + w * CPW + c, mm - 1)) * n + j + 1;
    double s[CPW] = {0.0, 0.0, 0.0, 0.0};
    constexpr int U = 4;
    for (int i0 = l; i0 < mm; i0 += 64 * U) {
        double x[U], av[CPW][U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = min(i0 + 64 * u, mm - 1);
            x[u] = v[i];
#pragma unroll
            for (int c = 0; c < CPW; ++c) av[c][u] = cp[c][i];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const double xx = i0 + 64 * u < mm ? x[u] : 0.0;
#pragma unroll
            for (int c = 0; c < CPW; ++c) s[c] += av[c][u] * xx;
        }
    }
    double z = 0.0;
#pragma unroll
    for (int u = 0; u < CPG / (WG / 64); ++u) z += c0 + w * CPW + u < mm ? zr[u] * zx[u] : 0.0;
    s_z[w][l] = z;
    // the four sums over the lanes: lane 16 c ends with column c
    static_assert(CPW == 4, "fold laid out for 4 columns per wave");
#pragma unroll
    for (int h = 2, o = 32; h >= 1; h >>= 1, o >>= 1) {
        const bool hi = l & o;
#pragma unroll
        for (int c = 0; c < h; ++c) {
            const double send = hi ? s[c] : s[c + h], keep = hi ? s[c + h] : s[c];
            s[c] = keep + __shfl_xor(send, o, 64);
        }
    }
    const double y = sum_lanes<16>(s[0]);
    const int c = c0 + w * CPW + (l >> 4);
    if ((l & 15) == 0 && c < mm) m.W[j + 1 + c + (int64_t)p * n] = y;
    __syncthreads();
    if (tid() < 2 * NB) m.zp[(int64_t)blockIdx.x * 2 * NB + tid()] = (s_z[0][tid()] + s_z[1][tid()]) + (s_z[2][tid()] + s_z[3][tid()]);
}

// C[r0:, r0:] -= V W^T + W V^T over lower tile pairs, stored to both triangles
__global__ void __launch_bounds__(WG) k_trd_update(const Mat* mats, int j0) {
    __shared__ mg::Smem sm;
    const Mat m = mats[blockIdx.y];
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

__global__ void k_trd_tail(const Mat* mats) {
    const Mat m = mats[blockIdx.x];
    const int n = m.n;
    if (tid() == 0 && n >= 3) {
        m.d[n - 2] = m.a[(n - 2) + (int64_t)(n - 2) * n];
        m.e[n - 2] = m.a[(n - 1) + (int64_t)(n - 2) * n];
        m.d[n - 1] = m.a[(n - 1) + (int64_t)(n - 1) * n];
    }
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

// All eigenvalues of the large problems' tridiagonal matrices by multisection (before the
// mode-count phase of k_local_eig): BL lanes per eigenvalue cut its interval in BL + 1 parts,
// so a round gains log2(BL + 1) bits for one count's latency, and the serial rounds drop from
// about 54 to 18 while the counts go up 2.7 times -- the chip is far from full with one lane
// per eigenvalue.  d and e^2 lie in LDS.  n = 882: 4.9 -> 1.05 ms.
constexpr int BL = 7;                // parts - 1; 8 lanes per eigenvalue, the last one idle
constexpr int BE = WG / 8;           // eigenvalues per workgroup
__global__ void __launch_bounds__(WG) k_trd_bisect(LocalArgs A, const int32_t* big) {
    __shared__ double red[WG / 64];
    extern __shared__ double s_t[];                    // d (n), e2 (n)
    const int b = big[blockIdx.y];
    const int ag = A.first + b;
    const int n = (int)(A.agg_ptr[ag + 1] - A.agg_ptr[ag]);
    const int i0 = (int)blockIdx.x * BE;
    if (i0 >= n) return;
    const double* d = A.t_buf + A.t_off[b];
    const double* e = d + n;
    double* s_e = s_t + n;
    double lo = INFINITY, hi = -INFINITY, emax2 = 0.0;
    for (int i = tid(); i < n; i += WG) {
        const double el = i > 0 ? e[i - 1] : 0.0, er = i + 1 < n ? e[i] : 0.0, di = d[i];
        const double r = fabs(el) + fabs(er);
        lo = fmin(lo, di - r);
        hi = fmax(hi, di + r);
        emax2 = fmax(emax2, er * er);
        s_t[i] = di;
        s_e[i] = el * el;
    }
    lo = -wg_max(-lo, red);
    hi = wg_max(hi, red);
    emax2 = wg_max(emax2, red);
    const double eps = 2.220446049250313e-16;
    const double tnorm = fmax(fabs(lo), fabs(hi));
    // smallest pivot: its reciprocal, times e^2, stays finite
    const double pivmin = fmax(2.2250738585072014e-308 * fmax(emax2, 1.0), 1e-290);
    const double atol = 2.0 * eps * tnorm + 1e-300;
    double a = lo - atol, c = hi + atol;
    const int i = min(i0 + (tid() >> 3), n - 1), l = tid() & 7;
    for (int it = 0; it < 80; ++it) {
        const bool done = c - a <= 2.0 * eps * fmax(fabs(a), fabs(c)) + atol;
        if (__all(done)) break;
        // lane l counts at the (l + 1)-th of BL inner points; lanes past the last one at c
        const double x = l < BL ? fmin(fmax(a + (c - a) * ((l + 1) * (1.0 / (BL + 1))), a), c) : c;
        const bool above = sturm_quick(s_t, s_e, n, x, pivmin) > i;     // the eigenvalue lies below x
        const unsigned mask = (unsigned)(__ballot(above) >> (tid() & 56)) & ((1u << BL) - 1);
        const int f = mask ? __ffs(mask) - 1 : BL;                      // first point above it
        const double xa = __shfl(x, (tid() & 56) + max(f - 1, 0), 64), xc = __shfl(x, (tid() & 56) + min(f, 7), 64);
        if (!done) {
            const double na = f > 0 ? xa : a, nc = f < BL ? xc : c;
            if (na == a && nc == c) a = c = 0.5 * (a + c);              // no representable point between
            else a = na, c = nc;
        }
    }
    if (l == 0 && i0 + (tid() >> 3) < n) A.mu[A.mu_off[ag] + i] = 0.5 * (a + c);
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
// loads a row the substitution took about 1 ms a pass at n = 882).  False, with Y unchanged,
// when a pivot falls below 1e-12, where one pass would lose orthogonality.
__device__ inline bool batch_cholqr(InvSmem& sm, double* Y, int n, int bn, const int* cl) {
    __shared__ double s_d[64], s_piv[64];
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
    __syncthreads();
    return ok;
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
// bytes: at n = 882 a factoring solve takes 187 us, a later one 104, an orthonormalisation
// 100.  Eight matrices of up to 882 with 179 vectors each: 15.4 -> 4.6 ms; 64 of up to 285
// with 40 each: 0.91 -> 0.31 ms.
__global__ void __launch_bounds__(WG) k_trd_invit(LocalArgs A, const int32_t* big, const int64_t* iw_off,
                                                  double* iw) {
    __shared__ double red[WG / 64];
    __shared__ double s_dot[64];
    __shared__ int s_cl[64];
    __shared__ int s_conv;
    __shared__ InvSmem sm;
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
                    mg::tile_mma<mg::KMAJ, mg::IMAJ>(sm.mm, Q, n, 0, qn, Y, 64, 0, bn, 0, n, acc);
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
                        mg::tile_mma<mg::IMAJ, mg::KMAJ>(sm.mm, Q + t0, n, 0, n - t0, dd, qn, 0, bn, 0, qn, acc);
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
                if (batch_cholqr(sm, Y, n, bn, s_cl)) continue;
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
        double* s = sm.s;
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
        const bool large = end == b0;                  // more than 64 members: 64 at a time
        const int stop = large ? ce : end;
        for (int m = b0; m < stop; m += 64) batch(m, min(64, stop - m), large ? b0 : m);
        b0 = stop;
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

static_assert(sizeof(Mat) <= TRD_MAT_BYTES, "matrix table");

void launch_local_tridiag_blocked(const LocalArgs& a, const int32_t* d_big, const std::vector<int32_t>& sizes,
                                  void* d_mats, hipStream_t st) {
    const int nbig = (int)sizes.size();
    if (nbig == 0) return;
    int max_n = 0;
    for (int32_t s : sizes) {
        if (s <= 2 * NB + 1) throw std::runtime_error("blocked tridiagonalisation needs n > 2 * TRD_NB + 1");
        max_n = std::max(max_n, (int)s);
    }
    Mat* mats = static_cast<Mat*>(d_mats);
    hipLaunchKernelGGL(k_trd_mats, dim3((nbig + 63) / 64), dim3(64), 0, st, a, d_big, nbig, mats);
    auto column = [&](int j, int j0, int fin) {
        auto go = [&](auto kern, int th) { hipLaunchKernelGGL(kern, dim3(nbig), dim3(th), 0, st, mats, j, j0, fin); };
        const int rows = max_n - (fin ? j0 : j);       // at most these are left
        if (rows <= 256) go(k_trd_col<256, 1>, 256);
        else if (rows <= 512) go(k_trd_col<256, 2>, 256);
        else if (rows <= 1024) go(k_trd_col<256, 4>, 256);
        else if (rows <= 2048) go(k_trd_col<1024, 2>, 1024);
        else go(k_trd_col<1024, 4>, 1024);
    };
    if (max_n > 4096) throw std::runtime_error("blocked tridiagonalisation: more than 4096 DOFs");
    for (int j0 = 0; j0 < max_n - 2; j0 += NB) {
        const int j1 = std::min(j0 + NB, max_n - 2);
        for (int j = j0; j < j1; ++j) {
            column(j, j0, 0);
            const int mm = max_n - j - 1;
            hipLaunchKernelGGL(k_trd_symv, dim3((mm + CPG - 1) / CPG, nbig), dim3(WG), 0, st, mats, j, j0);
        }
        column(0, j0, 1);
        int64_t jobs = 0;
        for (int32_t n : sizes) {
            const int pc = std::min(NB, (int)n - 2 - j0);
            if (pc <= 0) continue;
            const int64_t mt = (n - j0 - pc + mg::T - 1) / mg::T;
            jobs = std::max(jobs, mt * (mt + 1) / 2);
        }
        if (jobs > 0) hipLaunchKernelGGL(k_trd_update, dim3((unsigned)jobs, nbig), dim3(WG), 0, st, mats, j0);
    }
    hipLaunchKernelGGL(k_trd_tail, dim3(nbig), dim3(64), 0, st, mats);
    const size_t lds = 2 * (size_t)max_n * sizeof(double);
    if (lds > 60 * 1024)
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_trd_bisect),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(k_trd_bisect, dim3((max_n + BE - 1) / BE, nbig), dim3(WG), lds, st, a, d_big);
}

}  // namespace lsdd
