// Fused single-vector cycle kernels for CDNA4 (gfx950).
//
// On a level of up to some ten thousand DOFs the V-cycle moves a few megabytes per colour,
// which HBM delivers in a microsecond; what its time goes into are the dependent loads and
// the tails of its launches: residual rows, local product and partial sums took 3 to 10 us
// each, three launches a colour.  Here one workgroup carries a subdomain (an aggregate)
// from its residual rows through LDS to its update, so that a colour, a restriction and a
// prolongation are one launch each.  The colour kernel is for classes whose subdomains share
// no element (a colouring of the overlaps), so that none of them reads an x that another one
// of the launch writes; block Jacobi's one class of aggregates is none.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <stdexcept>

#include "blk.hpp"
#include "fuse.hpp"

namespace lsdd {

namespace {

// Row tables have `pad` entries per subdomain (DOF -1 past its end), so that a workgroup
// knows its entries' addresses from its number: one dependent load less than through an
// offset.
__global__ void k_row_table(const int64_t* off, const int32_t* dofs, const int64_t* rowptr, const int64_t* scoff,
                            int pad, int4* tab) {
    const int s = blockIdx.x;
    const int64_t o = off[s];
    const int m = (int)(off[s + 1] - o);
    for (int i = threadIdx.x; i < pad; i += 256) {
        int4 e = make_int4(-1, 0, 0, 0);
        if (i < m) {
            const int32_t d = dofs[o + i];
            const int64_t q0 = rowptr[d];
            e = make_int4(d, (int)q0, (int)(rowptr[d + 1] - q0), (int)(scoff ? scoff[d] : q0));
        }
        tab[(int64_t)s * pad + i] = e;
    }
}

// sums over the entries of R rows at once, L lanes per row, U entries per lane and row in
// flight (a slot past the end re-reads the last entry and adds zero; an empty row reads
// entry 0); the next step's columns and values are loaded before this step's gathers
// return, so a step costs one dependent load.  Every lane of the row gets the sums
template <typename T, int L, int R, int U = 4>
__device__ inline void row_sums(const int4 (&e)[R], int lane, const int32_t* __restrict__ col,
                                const T* __restrict__ val, const T* __restrict__ x, T (&s)[R]) {
    int len = 0;
#pragma unroll
    for (int i = 0; i < R; ++i) {
        s[i] = 0;
        len = max(len, e[i].z);
    }
    int32_t c[R][U];
    T a[R][U];
    auto load = [&](int q0) {
#pragma unroll
        for (int i = 0; i < R; ++i)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int q = max(min(q0 + u * L, e[i].z - 1), 0);
                c[i][u] = col[(uint32_t)e[i].w + q];
                a[i][u] = val[(uint32_t)e[i].y + q];
            }
    };
    load(lane);
    for (int q0 = lane; q0 < len; q0 += U * L) {
        T xv[R][U], av[R][U];
#pragma unroll
        for (int i = 0; i < R; ++i)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                xv[i][u] = x[c[i][u]];
                av[i][u] = q0 + u * L < e[i].z ? a[i][u] : (T)0;
            }
        if (q0 + U * L < len) load(q0 + U * L);
#pragma unroll
        for (int i = 0; i < R; ++i)
#pragma unroll
            for (int u = 0; u < U; ++u) s[i] += av[i][u] * xv[i][u];
    }
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
        for (int off = L / 2; off > 0; off >>= 1) s[i] += __shfl_xor(s[i], off, L);
}

// One workgroup of NW waves per subdomain.  The inverse does not depend on x, so its first
// entries are loaded before the residual rows and arrive while these are formed.
//
// |Omega| <= 64: the packed triangle goes through LDS, G = NW threads per row.  Larger: the
// tiles (I, J), J <= I, in storage order, 64 / NW rows of a tile per wave, lane = column;
// four tiles are in flight behind the four in use.  A tile gives its rows' sums (kept in
// registers over the tile row, then folded over the lanes) and, below the diagonal, its
// columns' sums (one LDS slot per wave and column, summed over the waves at the end).
// Every sum has a fixed order.
//
// Measured against the launches it replaces (residual rows, local product, partial sums), us
// per colour of a sweep: 30 overlaps of 50 DOFs (FP64) 10.0 -> 4.8; 484 of 50 (FP32) 11.0 ->
// 5.0; 210 of 65 to 123 (FP64) 20 -> 10, there the 20 MB of padded tiles set the time.
template <typename T, int NW, int L, int R, bool TILED>
__global__ void __launch_bounds__(NW * 64) k_colour_step(const SubItem* __restrict__ items,
                                                         const int4* __restrict__ rows,
                                                         const int32_t* __restrict__ col, const T* __restrict__ val,
                                                         const T* __restrict__ pk, const T* __restrict__ tiles,
                                                         const T* __restrict__ r, T* x, int x_zero, int m_pad) {
    constexpr int TH = NW * 64;
    extern __shared__ __align__(16) unsigned char s_mem[];
    T* s_r = reinterpret_cast<T*>(s_mem);              // residual, zero padded to m_pad
    T* s_x = s_r + m_pad;                              // x before the update
    T* s_y = s_x + m_pad;                              // row sums
    T* s_w = s_y + m_pad;                              // packed triangle, or NW x m_pad column sums
    int32_t* s_d = reinterpret_cast<int32_t*>(s_w + max(TILED ? NW * m_pad : 0, SMALL_M * (SMALL_M + 1) / 2));
    const int t = threadIdx.x;
    const SubItem it = items[blockIdx.x];
    const int m = it.m;
    const bool small = !TILED || m <= SMALL_M;
    const T* A = (small ? pk : tiles) + it.off;
    const int lane = t & 63, w = t >> 6;
    // first entries of the inverse
    constexpr int PS = (SMALL_M * (SMALL_M + 1) / 2 + TH - 1) / TH;   // triangle entries per thread
    constexpr int Q = 64 / NW;                                          // tile rows per wave
    constexpr int TG = 4;                                               // tiles in flight
    constexpr int PN = TILED && TG * Q > PS ? TG * Q : PS;
    T pre[PN];
    const int np = m * (m + 1) / 2;
    const int nt = (m + 63) >> 6, ntile = nt * (nt + 1) / 2;
    auto fetch = [&](T(&v)[PN], int k0) {
#pragma unroll
        for (int g = 0; g < TG; ++g) {
            const T* tp = A + (int64_t)min(k0 + g, ntile - 1) * 4096 + w * 64 + lane;
#pragma unroll
            for (int q = 0; q < Q; ++q) v[g * Q + q] = tp[q * NW * 64];
        }
    };
    if (small) {
#pragma unroll
        for (int u = 0; u < PS; ++u) pre[u] = A[min(t + u * TH, np - 1)];
    } else if constexpr (TILED) {
        fetch(pre, 0);
    }
    // residual rows, R at a time per group of L lanes
    const int4* tab = rows + (int64_t)blockIdx.x * m_pad;
    for (int i0 = t / L; i0 < m_pad; i0 += R * (TH / L)) {
        int4 e[R];
        T xo[R], rr[R], s[R];
#pragma unroll
        for (int j = 0; j < R; ++j) e[j] = tab[min(i0 + j * (TH / L), m_pad - 1)];
#pragma unroll
        for (int j = 0; j < R; ++j) {
            xo[j] = x[max(e[j].x, 0)];
            rr[j] = r[max(e[j].x, 0)];
            s[j] = 0;
        }
        if (!x_zero) row_sums<T, L, R>(e, t & (L - 1), col, val, x, s);
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int i = i0 + j * (TH / L);
            if ((t & (L - 1)) == 0 && i < m_pad) {
                s_r[i] = e[j].x >= 0 ? rr[j] - s[j] : (T)0;
                s_x[i] = xo[j];
                s_d[i] = e[j].x;
            }
        }
    }
    if (small) {
#pragma unroll
        for (int u = 0; u < PS; ++u)
            if (t + u * TH < np) s_w[t + u * TH] = pre[u];
    }
    __syncthreads();
    if (small) {
        constexpr int G = NW;                          // threads per row: TH / 64
        const int i = t / G, g = t % G;
        T y = 0;
        if (i < m) {
            const int ri = i * (i + 1) / 2;
#pragma unroll
            for (int u = 0; u < SMALL_M / G; ++u) {
                const int j = g + u * G;
                if (j < m) y += s_w[j <= i ? ri + j : j * (j + 1) / 2 + i] * s_r[j];
            }
        }
#pragma unroll
        for (int off = G / 2; off > 0; off >>= 1) y += __shfl_xor(y, off, G);
        if (i < m && g == 0) x[s_d[i]] = s_x[i] + y;
        return;
    }
    if constexpr (TILED) {
        T nxt[PN];
        T p[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) p[q] = 0;
        int I = 0, J = 0;
        for (int k0 = 0; k0 < ntile; k0 += TG) {
            if (k0 + TG < ntile) fetch(nxt, k0 + TG);
#pragma unroll
            for (int g = 0; g < TG; ++g) {
                if (k0 + g >= ntile) break;
                const T xj = s_r[J * 64 + lane];
                T c = 0;
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    p[q] += pre[g * Q + q] * xj;
                    c += pre[g * Q + q] * s_r[I * 64 + w + q * NW];
                }
                if (J < I) {
                    T* cs = s_w + w * m_pad + J * 64 + lane;
                    *cs = I == J + 1 ? c : *cs + c;
                    ++J;
                } else {
                    // the tile row is complete: its Q sums over the lanes (lane l ends with
                    // row l / (64 / Q)), then the next one
                    static_assert(Q == 4 || Q == 8, "fold laid out for 4 or 8 rows per wave");
                    T a[Q];
#pragma unroll
                    for (int q = 0; q < Q; ++q) a[q] = p[q], p[q] = 0;
#pragma unroll
                    for (int h = Q / 2, o = 32; h >= 1; h >>= 1, o >>= 1) {
                        const bool hi = lane & o;
#pragma unroll
                        for (int q = 0; q < h; ++q) {
                            const T send = hi ? a[q] : a[q + h], keep = hi ? a[q + h] : a[q];
                            a[q] = keep + __shfl_xor(send, o, 64);
                        }
                    }
                    T v = a[0];
#pragma unroll
                    for (int o = 32 / Q; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
                    if ((lane & (64 / Q - 1)) == 0) s_y[I * 64 + w + (lane / (64 / Q)) * NW] = v;
                    ++I;
                    J = 0;
                }
            }
#pragma unroll
            for (int u = 0; u < TG * Q; ++u) pre[u] = nxt[u];
        }
        __syncthreads();
        for (int i = t; i < m; i += TH) {
            T y = s_y[i];
            if (i < (nt - 1) * 64)
#pragma unroll
                for (int q = 0; q < NW; ++q) y += s_w[q * m_pad + i];
            x[s_d[i]] = s_x[i] + y;
        }
    }
}

// Unpacked inverses from the packed ones, a 64 x 64 tile of the lower triangle at a time through
// LDS, so that the rows of the tile and of its mirror image are contiguous on both sides.
template <typename T>
__global__ void __launch_bounds__(256) k_unpack(const int64_t* __restrict__ sub_off, const int64_t* __restrict__ tp_off,
                                                const int64_t* __restrict__ pk_off, const T* __restrict__ tiles,
                                                const T* __restrict__ pk, const int64_t* __restrict__ full_off,
                                                T* __restrict__ full) {
    __shared__ T s[64][65];
    const int sb = blockIdx.x;
    const int m = (int)(sub_off[sb + 1] - sub_off[sb]);
    const int nt = (m + 63) >> 6;
    T* F = full + full_off[sb];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int t = (int)blockIdx.y; t < nt * (nt + 1) / 2; t += (int)gridDim.y) {
        int I = 0, J = t;
        while (J > I) J -= ++I;
        __syncthreads();
        for (int r = w; r < 64; r += 4) {
            const int i = I * 64 + r, j = J * 64 + lane;
            if (m > SMALL_M) s[r][lane] = tiles[tp_off[sb] + (int64_t)t * 4096 + r * 64 + lane];
            else if (i < m && j <= i) s[r][lane] = s[lane][r] = pk[pk_off[sb] + i * (i + 1) / 2 + j];
        }
        __syncthreads();
        for (int r = w; r < 64; r += 4) {
            const int i = I * 64 + r, j = J * 64 + lane;
            if (i < m && j < m) F[(int64_t)i * m + j] = s[r][lane];
            const int i2 = J * 64 + r, j2 = I * 64 + lane;
            if (I != J && i2 < m && j2 < m) F[(int64_t)i2 * m + j2] = s[lane][r];
        }
    }
}

// x[Omega] += A_Omega^{-1} rloc by rows of the unpacked inverse, for subdomains too large
// for one workgroup: a wave per 4 rows (rloc loaded once for the four), 16 rows per
// workgroup, every row complete in its wave -- no partial sums to add in a second launch.
// It reads each entry pair twice, so it pays where the launches and not the bytes set the
// time.  Measured with the residual launch before it, us per colour of a sweep, against the
// tiled product and its partial sums: 25 overlaps of up to 161 DOFs (FP64) 16 -> 7.5; 30 of
// 552 (FP32, 15,600 rows) 15.5 -> 11.5; 4 of 1225 (FP32) 14 -> 11; 4 of 1515 (FP64, 24 MB
// packed) 17.4 -> 16.2.
template <typename T>
__global__ void __launch_bounds__(256) k_sub_rows(const RowItem* __restrict__ items, const T* __restrict__ inv,
                                                  const T* __restrict__ rloc, const int32_t* __restrict__ dofs, T* x) {
    const RowItem it = items[blockIdx.x];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int i0 = it.row0 + 4 * w, m = it.m;
    if (i0 >= m) return;
    const T* A = inv + it.off;
    const T* rl = rloc + it.o;
    const T* a[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] = A + (int64_t)min(i0 + i, m - 1) * m;
    // the updated entries, lane 16 i for row i
    const int mine = min(i0 + (lane >> 4), m - 1);
    const int32_t d = dofs[it.o + mine];
    T s[4] = {0, 0, 0, 0};
    constexpr int U = 4;
    for (int q0 = lane; q0 < m; q0 += 64 * U) {
        T rv[U], av[4][U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = min(q0 + 64 * u, m - 1);
            rv[u] = rl[q];
#pragma unroll
            for (int i = 0; i < 4; ++i) av[i][u] = a[i][q];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const T v = q0 + 64 * u < m ? rv[u] : (T)0;
#pragma unroll
            for (int i = 0; i < 4; ++i) s[i] += av[i][u] * v;
        }
    }
    const T xo = x[d];
    // fold: lane l ends with row l / 16
#pragma unroll
    for (int h = 2, o = 32; h >= 1; h >>= 1, o >>= 1) {
        const bool hi = lane & o;
#pragma unroll
        for (int i = 0; i < h; ++i) {
            const T send = hi ? s[i] : s[i + h], keep = hi ? s[i + h] : s[i];
            s[i] = keep + __shfl_xor(send, o, 64);
        }
    }
    T v = s[0];
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if ((lane & 15) == 0 && i0 + (lane >> 4) < m) x[d] = xo + v;
}

// Residual of an aggregate's rows in LDS, then its restriction: LC lanes per column of Z.
template <typename T, int TH, int L, int LC>
__global__ void __launch_bounds__(TH) k_resid_restrict(const AggItem* __restrict__ items,
                                                       const int4* __restrict__ rows,
                                                       const int32_t* __restrict__ col, const T* __restrict__ val,
                                                       const T* __restrict__ Zc, const T* __restrict__ r,
                                                       const T* __restrict__ x, T* __restrict__ rc,
                                                       T* __restrict__ xc, int pad) {
    extern __shared__ __align__(16) unsigned char s_mem[];
    T* s_t = reinterpret_cast<T*>(s_mem);              // pad
    const int t = threadIdx.x;
    const AggItem it = items[blockIdx.x];
    const int4* tab = rows + (int64_t)blockIdx.x * pad;
    constexpr int R = 2;
    for (int i0 = t / L; i0 < pad; i0 += R * (TH / L)) {
        int4 e[R];
        T rr[R], s[R];
#pragma unroll
        for (int j = 0; j < R; ++j) e[j] = tab[min(i0 + j * (TH / L), pad - 1)];
#pragma unroll
        for (int j = 0; j < R; ++j) rr[j] = r[max(e[j].x, 0)];
        row_sums<T, L, R>(e, t & (L - 1), col, val, x, s);
#pragma unroll
        for (int j = 0; j < R; ++j)
            if ((t & (L - 1)) == 0 && i0 + j * (TH / L) < pad) s_t[i0 + j * (TH / L)] = rr[j] - s[j];
    }
    __syncthreads();
    const T* Z = Zc + it.zoff;
    const int l = t % LC;
    for (int c = t / LC; c < it.k; c += TH / LC) {
        const T* z = Z + (int64_t)c * it.nw;
        T a[4] = {0, 0, 0, 0};
        for (int i = l; i < it.nw; i += 4 * LC) {
            T zv[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) zv[u] = z[min(i + u * LC, it.nw - 1)];
#pragma unroll
            for (int u = 0; u < 4; ++u) a[u] += (i + u * LC < it.nw ? zv[u] : (T)0) * s_t[min(i + u * LC, it.nw - 1)];
        }
        T v = (a[0] + a[1]) + (a[2] + a[3]);
#pragma unroll
        for (int off = LC / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, LC);
        if (l == 0) {
            rc[it.c0 + c] = v;
            xc[it.c0 + c] = 0;
        }
    }
}

// Prolongation of an aggregate: thread = (row, group of modes), the groups summed in LDS.
template <typename T, int TH>
__global__ void __launch_bounds__(TH) k_prolong_agg(const AggItem* __restrict__ items,
                                                    const int4* __restrict__ rows, const T* __restrict__ Zc,
                                                    const T* __restrict__ ec, T* x, int pad) {
    extern __shared__ __align__(16) unsigned char s_mem[];
    T* s_p = reinterpret_cast<T*>(s_mem);              // TH
    T* s_e = s_p + TH;                                 // max_k
    const int t = threadIdx.x;
    const AggItem it = items[blockIdx.x];
    for (int c = t; c < it.k; c += TH) s_e[c] = ec[it.c0 + c];
    const int rp = min(TH, (it.nw + 63) & ~63);       // rows per pass
    const int G = TH / rp;
    const int g = t / rp, i0 = t % rp;
    for (int i = i0; i - i0 < it.nw; i += rp) {
        const bool in = i < it.nw && g < G;
        const int ic = min(i, it.nw - 1);
        const int32_t d = rows[(int64_t)blockIdx.x * pad + min(i, pad - 1)].x;   // -1 past the end
        const T xo = x[max(d, 0)];
        const T* z = Zc + it.zoff + ic;
        __syncthreads();                               // s_e is there; s_p of the last pass is read
        T a0 = 0, a1 = 0;
        if (in) {
            constexpr int PU = 8;
            for (int c = g; c < it.k; c += PU * G) {
                T zv[PU];
#pragma unroll
                for (int u = 0; u < PU; ++u) zv[u] = z[(int64_t)min(c + u * G, it.k - 1) * it.nw];
#pragma unroll
                for (int u = 0; u < PU; ++u)
                    (u & 1 ? a1 : a0) += (c + u * G < it.k ? zv[u] : (T)0) * s_e[min(c + u * G, it.k - 1)];
            }
        }
        s_p[t] = a0 + a1;
        __syncthreads();
        if (in && g == 0) {
            T v = s_p[i0];
            for (int q = 1; q < G; ++q) v += s_p[q * rp + i0];
            x[d] = xo + v;
        }
    }
}

// x = inv r: two rows per wave against the same r, eight entries of each in flight.  Bound by
// the matrix: 1917 DOFs 7.1 us (4.1 TB/s); 2171 DOFs behind an FP32 cycle 10 us, where the
// packed tiles, their partial sums and two conversions took 24 us; 484 DOFs 15.4 -> 3.4 us.
template <typename T>
__global__ void __launch_bounds__(256) k_dense_apply(int n, const double* __restrict__ inv, const T* __restrict__ r,
                                                     T* __restrict__ x) {
    const int lane = threadIdx.x & 63;
    const int i0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * 2, i1 = min(i0 + 1, n - 1);
    if (i0 >= n) return;
    const double *a = inv + (int64_t)i0 * n, *b = inv + (int64_t)i1 * n;
    double s[2][2] = {{0, 0}, {0, 0}};
    constexpr int U = 8;
    for (int q0 = lane; q0 < n; q0 += 64 * U) {
        double av[U], bv[U];
        T rv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = min(q0 + u * 64, n - 1);
            rv[u] = r[q];
            av[u] = a[q];
            bv[u] = b[q];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const double w = q0 + u * 64 < n ? (double)rv[u] : 0.0;
            s[0][u & 1] += av[u] * w;
            s[1][u & 1] += bv[u] * w;
        }
    }
    double u = s[0][0] + s[0][1], v = s[1][0] + s[1][1];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        u += __shfl_xor(u, off, 64);
        v += __shfl_xor(v, off, 64);
    }
    if (lane == 0) {
        x[i0] = (T)u;
        if (i0 + 1 < n) x[i0 + 1] = (T)v;
    }
}

// Aggregates of a launch from which 256 threads each keep every CU busy; fewer get 1024 (841
// aggregates of 81 DOFs ran 14.6 us at 1024 threads, whose workgroups fill the chip twice).
constexpr int64_t WIDE_AGG = 256;

// a launch with more than 64 KB of LDS asks for it each time (a field of the kernel on this device
// is set: no state of our own to keep per device and kernel)
template <class K>
void allow_lds(K kern, size_t bytes) {
    if (bytes > 160 * 1024) throw std::runtime_error("fused cycle kernel: more LDS than a CU has");
    if (bytes > 64 * 1024 &&
        hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)bytes) != hipSuccess)
        throw std::runtime_error("fused cycle kernel: LDS size refused");
}

// f(lanes per row): lanes for an average row in two steps of four entries per lane
template <class F>
void with_lanes(int row_len, F&& f) {
    if (row_len <= 64) f(std::integral_constant<int, 8>{});
    else if (row_len <= 128) f(std::integral_constant<int, 16>{});
    else f(std::integral_constant<int, 32>{});
}

}  // namespace

void launch_row_table(int64_t n_sub, const int64_t* off, const int32_t* dofs, const int64_t* rowptr,
                      const int64_t* scoff, int pad, int4* tab, hipStream_t st) {
    if (n_sub <= 0) return;
    hipLaunchKernelGGL(k_row_table, dim3((unsigned)n_sub), dim3(256), 0, st, off, dofs, rowptr, scoff, pad, tab);
}

template <typename T>
void launch_unpack(int64_t n_sub, int max_sub, const int64_t* sub_off, const int64_t* tp_off, const int64_t* pk_off,
                   const T* tiles, const T* pk, const int64_t* full_off, T* full, hipStream_t st) {
    if (n_sub <= 0) return;
    const int nt = (max_sub + 63) / 64;
    hipLaunchKernelGGL(k_unpack<T>, dim3((unsigned)n_sub, (unsigned)std::min(nt * (nt + 1) / 2, 256)), dim3(256), 0, st,
                       sub_off, tp_off, pk_off, tiles, pk, full_off, full);
}

template <typename T>
void launch_sub_rows(int64_t n_items, const RowItem* items, const T* inv, const T* rloc, const int32_t* dofs, T* x,
                     hipStream_t st) {
    if (n_items <= 0) return;
    hipLaunchKernelGGL(k_sub_rows<T>, dim3((unsigned)n_items), dim3(256), 0, st, items, inv, rloc, dofs, x);
}

template <typename T>
void launch_colour_step(int64_t n_sub, const SubItem* items, const int4* rows, const int32_t* col, const T* val,
                        const T* pk, const T* tiles, const T* r, T* x, bool x_zero, int pad, int row_len,
                        hipStream_t st) {
    if (n_sub <= 0) return;
    if (pad < 64 || pad > FUSE_M || pad % 64) throw std::runtime_error("launch_colour_step: overlaps outside 1 .. FUSE_M");
    const int m_pad = pad;
    auto go = [&](auto nw, auto lanes, auto rows_at_once) {
        constexpr int NW = decltype(nw)::value, L = decltype(lanes)::value, R = decltype(rows_at_once)::value;
        auto kern = &k_colour_step<T, NW, L, R, (NW > 8)>;
        const int w_len = std::max(NW > 8 ? NW * m_pad : 0, SMALL_M * (SMALL_M + 1) / 2);
        const size_t lds = (3 * (size_t)m_pad + w_len) * sizeof(T) + (size_t)m_pad * sizeof(int32_t);
        allow_lds(kern, lds);
        hipLaunchKernelGGL(kern, dim3((unsigned)n_sub), dim3(NW * 64), lds, st, items, rows, col, val, pk, tiles, r, x,
                           x_zero ? 1 : 0, m_pad);
    };
    with_lanes(row_len, [&](auto lanes) {
        // overlaps of one tile: 8 waves hold all their rows at once (8 lanes each); larger
        // ones take two rows per lane group where one does not cover them
        constexpr std::integral_constant<int, 1> one{};
        constexpr std::integral_constant<int, 2> two{};
        if (pad <= SMALL_M) go(std::integral_constant<int, 8>{}, lanes, one);
        else if (pad * decltype(lanes)::value <= 1024) go(std::integral_constant<int, 16>{}, lanes, one);
        else go(std::integral_constant<int, 16>{}, lanes, two);
    });
}

template <typename T>
void launch_resid_restrict(int64_t n_agg, const AggItem* items, const int4* rows, const int32_t* col, const T* val,
                           const T* Zc, const T* r, const T* x, T* rc, T* xc, int pad, int row_len,
                           hipStream_t st) {
    if (n_agg <= 0) return;
    with_lanes(row_len, [&](auto lanes) {
        constexpr int L = decltype(lanes)::value;
        const size_t lds = (size_t)pad * sizeof(T);
        if (pad <= SMALL_M)
            hipLaunchKernelGGL((k_resid_restrict<T, 256, L, 16>), dim3((unsigned)n_agg), dim3(256), lds, st, items, rows,
                               col, val, Zc, r, x, rc, xc, pad);
        else if (n_agg >= WIDE_AGG)
            hipLaunchKernelGGL((k_resid_restrict<T, 256, L, 64>), dim3((unsigned)n_agg), dim3(256), lds, st, items, rows,
                               col, val, Zc, r, x, rc, xc, pad);
        else
            hipLaunchKernelGGL((k_resid_restrict<T, 1024, L, 64>), dim3((unsigned)n_agg), dim3(1024), lds, st, items,
                               rows, col, val, Zc, r, x, rc, xc, pad);
    });
}

template <typename T>
void launch_prolong_agg(int64_t n_agg, const AggItem* items, const int4* rows, const T* Zc, const T* ec, T* x, int pad,
                        int max_k, hipStream_t st) {
    if (n_agg <= 0) return;
    auto go = [&](auto th) {
        constexpr int TH = decltype(th)::value;
        hipLaunchKernelGGL((k_prolong_agg<T, TH>), dim3((unsigned)n_agg), dim3(TH), (TH + (size_t)max_k) * sizeof(T), st,
                           items, rows, Zc, ec, x, pad);
    };
    if (pad <= SMALL_M || n_agg >= WIDE_AGG) go(std::integral_constant<int, 256>{});
    else go(std::integral_constant<int, 1024>{});
}

template <typename T>
void launch_dense_apply(int64_t n, const double* inv, const T* r, T* x, hipStream_t st) {
    if (n <= 0) return;
    hipLaunchKernelGGL(k_dense_apply<T>, dim3((unsigned)((n + 7) / 8)), dim3(256), 0, st, (int)n, inv, r, x);
}

#define LSDD_FUSE_INST(T)                                                                                             \
    template void launch_colour_step<T>(int64_t, const SubItem*, const int4*, const int32_t*, const T*, const T*,    \
                                        const T*, const T*, T*, bool, int, int, hipStream_t);                          \
    template void launch_resid_restrict<T>(int64_t, const AggItem*, const int4*, const int32_t*, const T*, const T*,  \
                                           const T*, const T*, T*, T*, int, int, hipStream_t);                         \
    template void launch_unpack<T>(int64_t, int, const int64_t*, const int64_t*, const int64_t*, const T*, const T*,  \
                                   const int64_t*, T*, hipStream_t);                                                   \
    template void launch_sub_rows<T>(int64_t, const RowItem*, const T*, const T*, const int32_t*, T*, hipStream_t);   \
    template void launch_prolong_agg<T>(int64_t, const AggItem*, const int4*, const T*, const T*, T*, int, int,       \
                                        hipStream_t);                                                                  \
    template void launch_dense_apply<T>(int64_t, const double*, const T*, T*, hipStream_t);
LSDD_FUSE_INST(double)
LSDD_FUSE_INST(float)

}  // namespace lsdd
