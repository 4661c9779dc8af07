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
#include "invit.hpp"
#include "kernels.hpp"
#include "mgemm.hpp"

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
// (10.4 against 7.7 us a column, averaged over n = 648 and 882).  The order of the sums depends
// on TH, so a matrix takes the TH of its own remaining rows whatever else is in the batch: a
// launch is for matrices with more than `above` rows left and at most TH RPT.
template <int TH, int RPT>
__global__ void __launch_bounds__(TH) k_trd_col(const Mat* mats, int j, int j0, int fin, int above) {
    constexpr int QC = RPT <= 2 ? 8 : 4;               // panel columns in flight
    constexpr int PW = TH / 64;
    __shared__ double red[PW];
    __shared__ double part[PW][2 * NB];
    __shared__ __align__(16) double fac[NB][4];        // W^T v, V^T v, rows j of V and W
    __shared__ double s_row[2];
    const Mat m = mats[blockIdx.x];
    const int n = m.n;
    const int left = n - (fin ? j0 : j);
    if (left <= above || left > TH * RPT) return;
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
    const TriBracket B = wg_bracket(d, e, n, s_t, s_e, red);
    const double eps = 2.220446049250313e-16, atol = B.atol, pivmin = B.pivmin;
    double a = B.lo, c = B.hi;
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

// Retained eigenvectors of the large problems' tridiagonal matrices; workgroup x takes the
// clusters that start at the eigenvalue indices [64x, 64x + 64).
__global__ void __launch_bounds__(WG) k_trd_invit(LocalArgs A, const int32_t* big, const int64_t* iw_off,
                                                  double* iw) {
    __shared__ InvShared S;
    extern __shared__ double s_dyn[];
    const int b = big[blockIdx.y];
    const int ag = A.first + b;
    const int n = (int)(A.agg_ptr[ag + 1] - A.agg_ptr[ag]);
    const int kk = A.k_out[ag];
    const int r0 = (int)blockIdx.x * 64;
    if (r0 >= kk) return;
    const double* d = A.t_buf + A.t_off[b];
    wg_invit(d, d + n, n, A.mu + A.mu_off[ag], kk, r0, min(kk, r0 + 64), A.w1 + A.ws_off[b],
             iw + iw_off[blockIdx.y] + (int64_t)blockIdx.x * invit_ws(n), reinterpret_cast<unsigned char*>(s_dyn), S);
}

// Retained eigenvectors for the large problems, a wave each (VS = W1, n x k, ld n; RPT: rows
// per lane, 0 for more than 1024, which sum in another order and so have a launch of their own); bound by the reads of the reflectors and the ten sums over the wave
// a round takes.  Eight matrices of up to 882 with 179 vectors each: 1.94 -> 1.04
// ms.
template <int RPT>
__global__ void __launch_bounds__(WG) k_trd_backtransform(LocalArgs A, const int32_t* big) {
    const int b = big[blockIdx.y];
    const int ag = A.first + b;
    const int n = (int)(A.agg_ptr[ag + 1] - A.agg_ptr[ag]);
    const int c = (int)blockIdx.x * (WG / 64) + (tid() >> 6);
    if (c >= A.k_out[ag] || (n > 1024) != (RPT == 0)) return;
    const double* a = A.s_buf + A.sq_off[b];
    const double* tau = A.t_buf + A.t_off[b] + 2 * n;
    double* x = A.w1 + A.ws_off[b] + (int64_t)c * n;
    if constexpr (RPT > 0) wave_backtransform<RPT, 1>(a, n, tau, x, 1);
    else wave_backtransform_long(a, n, tau, x);
}

}  // namespace

void launch_local_backtransform_blocked(const LocalArgs& a, const int32_t* d_big, const std::vector<int32_t>& sizes,
                                        hipStream_t st) {
    const int nbig = (int)sizes.size();
    if (nbig == 0) return;
    int max_n = 0, min_n = INT32_MAX;
    for (int32_t s : sizes) {
        max_n = std::max(max_n, (int)s);
        min_n = std::min(min_n, (int)s);
    }
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3((max_n + WG / 64 - 1) / (WG / 64), nbig), dim3(WG), 0, st, a, d_big);
    };
    if (max_n <= 256) go(k_trd_backtransform<4>);
    else if (max_n <= 512) go(k_trd_backtransform<8>);
    else if (min_n <= 1024) go(k_trd_backtransform<16>);
    if (max_n > 1024) go(k_trd_backtransform<0>);
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
        auto go = [&](auto kern, int th, int above) {
            hipLaunchKernelGGL(kern, dim3(nbig), dim3(th), 0, st, mats, j, j0, fin, above);
        };
        const int base = fin ? j0 : j, rows = max_n - base;       // at most these are left
        const bool short_ones = std::any_of(sizes.begin(), sizes.end(),
                                            [&](int32_t n) { return n - base > 2 && n - base <= 1024; });
        if (rows <= 256) go(k_trd_col<256, 1>, 256, 0);
        else if (rows <= 512) go(k_trd_col<256, 2>, 256, 0);
        else if (short_ones) go(k_trd_col<256, 4>, 256, 0);
        if (rows > 2048) go(k_trd_col<1024, 4>, 1024, 1024);
        else if (rows > 1024) go(k_trd_col<1024, 2>, 1024, 1024);
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
