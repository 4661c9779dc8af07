// Kernels of the hierarchies that keep the order of operations (fixed.hpp): the diagonal-tile
// steps of the Cholesky factorisation and triangular solves, and the eigenproblems of aggregates
// above 32 DOFs, in one workgroup below trd_min and blocked from there on.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cfloat>
#include <stdexcept>
#include <vector>

#include "batched.hpp"
#include "dense.hpp"
#include "fixed.hpp"
#include "kernels.hpp"
#include "mgemm.hpp"

namespace lsdd::fixed {

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

// Retained eigenvectors of the large problems' tridiagonal matrices by
// inverse iteration: workgroup x takes the eigenvalue indices [64x, 64x + 64)
// (singletons one per thread, and the clusters that start there).
__global__ void __launch_bounds__(WG) k_trd_invit(LocalArgs A, const int32_t* big, const int64_t* iw_off,
                                                  double* iw) {
    __shared__ double red[WG / 64];
    __shared__ int s_ncl;
    __shared__ mg::Smem sm;
    extern __shared__ double s_dyn[];
    const int b = big[blockIdx.y];
    const int ag = A.first + b;
    const int n = (int)(A.agg_ptr[ag + 1] - A.agg_ptr[ag]);
    const int kk = A.k_out[ag];
    const int r0 = (int)blockIdx.x * 64;
    if (r0 >= kk) return;
    const double* T = A.t_buf + A.t_off[b];
    const double* d = T;
    const double* e = T + n;
    double tnorm = 0.0;
    for (int i = tid(); i < n; i += WG)
        tnorm = fmax(tnorm, fabs(d[i]) + (i > 0 ? fabs(e[i - 1]) : 0.0) + (i + 1 < n ? fabs(e[i]) : 0.0));
    tnorm = wg_max(tnorm, red);
    double* ws = iw + iw_off[blockIdx.y] + (int64_t)blockIdx.x * ((int64_t)FIXED_INVIT_SLOTS * n + 4096);
    wg_inverse_iteration_range(d, e, n, A.mu + A.mu_off[ag], kk, r0, min(kk, r0 + 64), A.w1 + A.ws_off[b], ws,
                               ws + (int64_t)FIXED_INVIT_SLOTS * n, fmax(tnorm, 1e-300), (int*)(s_dyn + 64), s_dyn, red,
                               &s_ncl, &sm);
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

// ---------------------------------------------------------------- diagonal-tile steps

constexpr int TB = 64;
constexpr int NT = 256;
__device__ inline int t_id() { return (int)threadIdx.x; }
__device__ inline double wave_min(double v) {
    for (int off = 32; off > 0; off >>= 1) v = fmin(v, __shfl_xor(v, off, 64));
    return v;
}
__device__ inline int ntiles(int n) { return (n + TB - 1) / TB; }

// 64 x 64 tile (rows r0.., cols c0..) into LDS, zero outside the view; if
// `unit_pad`, padded diagonal entries are 1 (a padded triangular factor).
__device__ inline void ld_tile64(double (*t)[TB + 1], const double* a, const View& v, int r0, int c0,
                                 bool unit_pad = false) {
    for (int idx = t_id(); idx < TB * TB; idx += NT) {
        int i = idx % TB, j = idx / TB;
        int r = r0 + i, c = c0 + j;
        double x = (r < v.rows && c < v.cols) ? a[v.off + r + (int64_t)c * v.ld] : 0.0;
        if (unit_pad && i == j && !(r < v.rows && c < v.cols)) x = 1.0;
        t[i][j] = x;
    }
}

// ---------------------------------------------------------------- substitution in registers
//
// 64 right-hand sides at once: thread t works on vector t / 4 and holds its
// entries sub, sub + 4, ..., sub + 60 (sub = t % 4) in x[16]; the four lanes
// of a vector are adjacent, so pivots are passed by lane shuffles.

// L x = b (L lower, LDS), first nb rows
__device__ inline void fwd_subst(const double (*L)[TB + 1], double (&x)[16], int nb) {
    const int sub = t_id() & 3, base = (t_id() & 63) & ~3;
#pragma unroll
    for (int i = 0; i < TB; ++i) {
        if (i < nb) {
            double xi = x[i >> 2] / L[i][i];
            xi = __shfl(xi, base | (i & 3), 64);
            if (sub == (i & 3)) x[i >> 2] = xi;
#pragma unroll
            for (int q = 0; q < 16; ++q)
                if (4 * q + sub > i) x[q] -= L[4 * q + sub][i] * xi;
        }
    }
}

// L^T x = b (L lower, LDS), first nb rows
__device__ inline void bwd_subst(const double (*L)[TB + 1], double (&x)[16], int nb) {
    const int sub = t_id() & 3, base = (t_id() & 63) & ~3;
#pragma unroll
    for (int i = TB - 1; i >= 0; --i) {
        if (i < nb) {
            double xi = x[i >> 2] / L[i][i];
            xi = __shfl(xi, base | (i & 3), 64);
            if (sub == (i & 3)) x[i >> 2] = xi;
#pragma unroll
            for (int q = 0; q < 16; ++q)
                if (4 * q + sub < i) x[q] -= L[i][4 * q + sub] * xi;
        }
    }
}

// ---------------------------------------------------------------- Cholesky

// unblocked Cholesky of diagonal tile kb by one wave: lane i holds row i of the
// tile in registers; at column j the pivot is broadcast by a lane shuffle and
// the new column L[:, j] through LDS.  minpiv[view] tracks the smallest pivot
// (a non-positive or NaN pivot is replaced by 1 so the factorisation runs to
// the end; the caller reads minpiv)
__global__ void __launch_bounds__(64) k_potrf_diag(double* base, const View* views, int kb, double* minpiv) {
    __shared__ double col[TB];
    const View v = views[blockIdx.y];
    const int n = v.rows;
    if (kb * TB >= n) return;
    const int r0 = kb * TB, nb = min(TB, n - r0);
    const int i = t_id();
    double x[TB];
    // every lane loads a full row of the block first (row and column clamped into
    // the block, so the 64 loads are unconditional and in flight together), then
    // keeps its lower part (identity rows past the block end)
    const int ic = min(i, nb - 1);
#pragma unroll
    for (int k = 0; k < TB; ++k) x[k] = base[v.off + (r0 + ic) + (int64_t)(r0 + min(k, nb - 1)) * v.ld];
#pragma unroll
    for (int k = 0; k < TB; ++k) x[k] = (i < nb && k <= i) ? x[k] : (k == i ? 1.0 : 0.0);
    double dmin = INFINITY;
#pragma unroll
    for (int j = 0; j < TB; ++j) {
        if (j < nb) {
            double dj = 1.0;
            if (i == j) {
                const double d = x[j];
                dmin = (d == d) ? d : -1.0;
                dj = d > 0.0 ? sqrt(d) : 1.0;
                x[j] = dj;
            }
            dj = __shfl(dj, j, 64);
            if (i > j) x[j] /= dj;
            col[i] = i > j ? x[j] : 0.0;
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int k = j + 1; k < TB; ++k)
                if (i >= k) x[k] -= x[j] * col[k];
            __builtin_amdgcn_wave_barrier();
        }
    }
    dmin = wave_min(dmin);
    if (i < nb) {
#pragma unroll
        for (int k = 0; k < TB; ++k)
            if (k <= i) base[v.off + (r0 + i) + (int64_t)(r0 + k) * v.ld] = x[k];
    }
    if (i == 0) minpiv[blockIdx.y] = (kb == 0) ? dmin : fmin(minpiv[blockIdx.y], dmin);
}

// L_ib,kb = A_ib,kb L_kk^{-T}, ib = kb + 1 + blockIdx.x: each row solves
// L_kk x^T = a^T (forward substitution)
__global__ void __launch_bounds__(NT) k_potrf_panel(double* base, const View* views, int kb) {
    __shared__ double L[TB][TB + 1];
    const View v = views[blockIdx.y];
    const int n = v.rows;
    const int nt = ntiles(n);
    const int ib = kb + 1 + (int)blockIdx.x;
    if (ib >= nt) return;
    const int nb = min(TB, n - kb * TB);
    ld_tile64(L, base, v, kb * TB, kb * TB, true);
    __syncthreads();
    const int r = ib * TB + t_id() / 4, sub = t_id() & 3;
    double x[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int c = kb * TB + 4 * q + sub;
        x[q] = (r < n && 4 * q + sub < nb) ? base[v.off + r + (int64_t)c * v.ld] : 0.0;
    }
    fwd_subst(L, x, nb);
    if (r < n) {
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int c = kb * TB + 4 * q + sub;
            if (4 * q + sub < nb) base[v.off + r + (int64_t)c * v.ld] = x[q];
        }
    }
}

// step s of L X = B (forward, kb = s) or L^T X = B (backward, kb = nt-1-s):
// solve the diagonal tile for column tile jc = blockIdx.x of B.  lower_b: B is
// lower triangular (forward only), so column tiles jc > kb are still zero.
__global__ void __launch_bounds__(NT) k_trsm_diag(const double* lbase, const View* lv, double* bbase, const View* bv,
                                                  int s, int trans, int lower_b) {
    __shared__ double L[TB][TB + 1];
    const View l = lv[blockIdx.y], b = bv[blockIdx.y];
    const int n = l.rows;
    const int nt = ntiles(n);
    if (s >= nt) return;
    const int kb = trans ? nt - 1 - s : s;
    const int jc = (int)blockIdx.x;
    if (jc * TB >= b.cols || (lower_b && jc > kb)) return;
    const int nb = min(TB, n - kb * TB);
    ld_tile64(L, lbase, l, kb * TB, kb * TB, true);
    __syncthreads();
    const int c = jc * TB + t_id() / 4, sub = t_id() & 3;
    double x[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int r = kb * TB + 4 * q + sub;
        x[q] = (c < b.cols && 4 * q + sub < nb) ? bbase[b.off + r + (int64_t)c * b.ld] : 0.0;
    }
    if (!trans) fwd_subst(L, x, nb);
    else bwd_subst(L, x, nb);
    if (c < b.cols) {
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int r = kb * TB + 4 * q + sub;
            if (4 * q + sub < nb) bbase[b.off + r + (int64_t)c * b.ld] = x[q];
        }
    }
}

// ---------------------------------------------------------------- one workgroup per aggregate

// Aggregates of 33 to trd_min - 1 DOFs, a workgroup each: reduction and eigenvalues (PHASE 0),
// inverse iteration (1), back-transformation (2).
template <int PHASE>
__global__ void __launch_bounds__(WG) k_local_eig(LocalArgs A) {
    __shared__ double s_red[WG / 64];
    __shared__ int s_ncl;
    extern __shared__ double s_dyn[];
    const int b = blockIdx.x;
    const int ag = A.first + b;
    const int nw = (int)(A.agg_ptr[ag + 1] - A.agg_ptr[ag]);
    double* W1 = A.w1 + A.ws_off[b];
    double* S = A.s_buf + A.sq_off[b];
    double* V = A.v_buf + A.sq_off[b];
    double* T = A.t_buf + A.t_off[b];
    double* mu = A.mu + A.mu_off[ag];
    double* VS = W1;
    if (nw <= 32 || (A.trd_min > 0 && nw >= A.trd_min)) return;     // Jacobi; the multi-workgroup path
    if (PHASE == 0) {
        wg_tridiag(S, nw, T, T + nw, T + 2 * nw, s_dyn, s_dyn + nw, s_red);
        wg_bisect_all(T, T + nw, nw, mu, s_red);
        return;
    }
    const int k = A.k_out[ag];
    if (k == 0) return;
    if (PHASE == 1) {
        const double* d = T;
        const double* e = T + nw;
        double tnorm = 0.0;
        for (int i = tid(); i < nw; i += WG)
            tnorm = fmax(tnorm, fabs(d[i]) + (i > 0 ? fabs(e[i - 1]) : 0.0) + (i + 1 < nw ? fabs(e[i]) : 0.0));
        tnorm = wg_max(tnorm, s_red);
        wg_inverse_iteration(d, e, nw, mu, k, VS, T + 3 * nw, fmax(tnorm, 1e-300), (int*)s_dyn, s_dyn + nw, s_red,
                             &s_ncl);
        return;
    }
    wg_tridiag_backtransform(S, nw, T + 2 * nw, VS, k, s_dyn, s_dyn + nw);
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
    const size_t lds = 64 * sizeof(double) + (size_t)(max_n + 1) * sizeof(int);   // dots, cluster starts
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

void launch_local_tridiag(int32_t nbatch, const LocalArgs& a, int32_t max_nw, hipStream_t st) {
    if (nbatch <= 0 || max_nw <= 32) return;
    hipLaunchKernelGGL(k_local_eig<0>, dim3(nbatch), dim3(WG), 2 * (size_t)max_nw * sizeof(double), st, a);
}

void launch_local_vectors(int32_t nbatch, const LocalArgs& a, int32_t max_nw, hipStream_t st) {
    if (nbatch <= 0 || max_nw <= 32) return;
    const size_t lds = (size_t)std::max(2 * max_nw, max_nw + 64) * sizeof(double);
    hipLaunchKernelGGL(k_local_eig<1>, dim3(nbatch), dim3(WG), lds, st, a);
    hipLaunchKernelGGL(k_local_eig<2>, dim3(nbatch), dim3(WG), lds, st, a);
}

void launch_potrf_diag(unsigned nm, double* base, const View* views, int kb, double* minpiv, hipStream_t st) {
    hipLaunchKernelGGL(k_potrf_diag, dim3(1, nm), dim3(64), 0, st, base, views, kb, minpiv);
}
void launch_potrf_panel(unsigned below, unsigned nm, double* base, const View* views, int kb, hipStream_t st) {
    hipLaunchKernelGGL(k_potrf_panel, dim3(below, nm), dim3(NT), 0, st, base, views, kb);
}
void launch_trsm_diag(unsigned nct, unsigned nm, const double* lbase, const View* lv, double* bbase, const View* bv,
                      int s, int trans, int lower_b, hipStream_t st) {
    hipLaunchKernelGGL(k_trsm_diag, dim3(nct, nm), dim3(NT), 0, st, lbase, lv, bbase, bv, s, trans, lower_b);
}

}  // namespace lsdd::fixed
