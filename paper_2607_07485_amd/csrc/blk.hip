// Block (multi right-hand side) cycle kernels and the segmented PCG of the
// batched solve, for CDNA4 (gfx950).
//
// Block vectors interleave NRB = 8 right-hand sides per DOF, so each matrix,
// inverse or interpolation entry read from HBM is used for all of them: the
// cycle's bytes per right-hand side drop by up to 8x against separate solves.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <cmath>
#include <stdexcept>
#include <type_traits>

#include "blk.hpp"
#include "kernels.hpp"
#include "dense.hpp"
#include "symv.hpp"

namespace lsdd {

namespace {

constexpr int WG = LSDD_WG;
constexpr int NB = NRB;

// compute units of the current device (queried once per device)
int device_cu_count() {
    static int count[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    if (!count[dev]) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1) n = 256;
        count[dev] = n;
    }
    return count[dev];
}

inline unsigned grid_for(int64_t n, int per_block = WG) {
    int64_t g = (n + per_block - 1) / per_block;
    if (g < 1) g = 1;
    if (g > 65535LL * 64) g = 65535LL * 64;
    return (unsigned)g;
}

// ---------------------------------------------------------------- CSR
// L lanes per row; lane = (nonzero slot, right-hand side): L / NB nonzeros per step.
template <typename T, int L>
__global__ void __launch_bounds__(WG) k_csr_resid_rows_b(int64_t nrows, const int32_t* rows, const int64_t* rowptr,
                                                         const int32_t* col, const T* val, const T* x, const T* r,
                                                         T* out, int x_zero, const int64_t* scoff) {
    constexpr int NS = L / NB;
    const int lane = tid() & (L - 1), k = lane & (NB - 1), slot = lane / NB;
    const int64_t stride = (int64_t)gridDim.x * (WG / L);
    for (int64_t t = ((int64_t)blockIdx.x * WG + tid()) / L; t < nrows; t += stride) {
        const int32_t p = rows[t];   // < 0: masked entry, out = 0
        T s = 0;
        if (!x_zero && p >= 0) {
            const int64_t q1 = rowptr[p + 1], cb = scoff ? scoff[p] - rowptr[p] : 0;
#pragma unroll 4
            for (int64_t q = rowptr[p] + slot; q < q1; q += NS) s += val[q] * x[(int64_t)col[cb + q] * NB + k];
        }
        for (int off = L / 2; off >= NB; off >>= 1) s += __shfl_xor(s, off, L);
        if (slot == 0) out[t * NB + k] = p >= 0 ? r[(int64_t)p * NB + k] - s : (T)0;
    }
}

// L lanes per row (4, 8 or 16); lane = nonzero slot holding all NB right-hand
// sides: it reads its entries' values and columns once and each gathered row of
// x with 16-byte loads (two entries in flight; past the row end the index is
// clamped to the last entry and the value zeroed, so the loads need no branch).
// The NB sums are reduced over the L lanes by a transposing butterfly (4 + 2 + 1
// exchanges over 8 lanes leave lane l with right-hand side l; 4 + 2 over 4 lanes
// leave it with 2l and 2l + 1), then by plain exchanges over the remaining lane
// bits; the order is fixed.
template <typename T>
struct Row16 {
    using V = double2;
};
template <>
struct Row16<float> {
    using V = float4;
};

template <typename T>
__device__ inline void load_xrow(const T* p, T (&v)[NB]) {
    using V = typename Row16<T>::V;
    constexpr int W = 16 / sizeof(T);
    const V* pv = reinterpret_cast<const V*>(p);
#pragma unroll
    for (int u = 0; u < NB / W; ++u) {
        const V t = pv[u];
        const T* tt = reinterpret_cast<const T*>(&t);
#pragma unroll
        for (int c = 0; c < W; ++c) v[u * W + c] = tt[c];
    }
}

template <typename T, int L>
__device__ inline void slot_row_sums(int64_t q0, int64_t q1, int lane, const int32_t* col, int64_t cb, const T* val,
                                     const T* x, T (&s)[NB]) {
    const int nit = (int)((q1 - q0 + L - 1) / L);
    for (int it = 0; it < nit; it += 2) {
        const int64_t qa = q0 + lane + (int64_t)it * L, qb = qa + L;
        const int64_t qac = qa < q1 ? qa : q1 - 1, qbc = qb < q1 ? qb : q1 - 1;
        const T va = val[qac], vb = val[qbc];
        const int32_t ca = col[cb + qac], cc = col[cb + qbc];
        T xa[NB], xb[NB];
        load_xrow(x + (int64_t)ca * NB, xa);
        load_xrow(x + (int64_t)cc * NB, xb);
        const T wa = qa < q1 ? va : (T)0, wb = qb < q1 ? vb : (T)0;
#pragma unroll
        for (int k = 0; k < NB; ++k) s[k] += wa * xa[k];
#pragma unroll
        for (int k = 0; k < NB; ++k) s[k] += wb * xb[k];
    }
}

// one butterfly step: lanes paired across lane bit `o` swap halves of their
// first 2 C values and keep the half selected by that bit
template <typename T, int L, int C>
__device__ inline void slot_fold(T (&s)[NB], int lane, int o) {
    const bool hi = (lane & o) != 0;
#pragma unroll
    for (int i = 0; i < C; ++i) {
        const T send = hi ? s[i] : s[i + C], keep = hi ? s[i + C] : s[i];
        s[i] = keep + __shfl_xor(send, o, L);
    }
}

// B = min(L, NB) lanes split the NB sums: afterwards lane l < B holds right-hand
// sides (NB / B) l + i in s[i], i < NB / B, summed over all L lanes of the row
template <typename T, int L>
__device__ inline void slot_reduce(T (&s)[NB], int lane) {
    static_assert(NB == 8 && L >= 4 && L <= 64, "butterfly laid out for 8 right-hand sides");
    constexpr int B = L < NB ? L : NB;
    slot_fold<T, L, 4>(s, lane, B / 2);
    slot_fold<T, L, 2>(s, lane, B / 4);
    if constexpr (B == 8) slot_fold<T, L, 1>(s, lane, 1);
#pragma unroll
    for (int off = 8; off < L; off <<= 1) s[0] += __shfl_xor(s[0], off, L);
}

template <typename T, int L>
__global__ void __launch_bounds__(WG) k_csr_resid_rows_s(int64_t nrows, const int32_t* rows, const int64_t* rowptr,
                                                         const int32_t* col, const T* val, const T* x, const T* r,
                                                         T* out, int x_zero, const int64_t* scoff) {
    const int lane = tid() & (L - 1);
    const int64_t stride = (int64_t)gridDim.x * (WG / L);
    for (int64_t t = ((int64_t)blockIdx.x * WG + tid()) / L; t < nrows; t += stride) {
        const int32_t p = rows[t];   // < 0: masked entry, out = 0
        T s[NB];
#pragma unroll
        for (int k = 0; k < NB; ++k) s[k] = 0;
        if (!x_zero && p >= 0)
            slot_row_sums<T, L>(rowptr[p], rowptr[p + 1], lane, col, scoff ? scoff[p] - rowptr[p] : 0, val, x, s);
        slot_reduce<T, L>(s, lane);
        constexpr int PL = L < NB ? NB / L : 1;   // right-hand sides per writing lane
        if (lane * PL < NB)
#pragma unroll
            for (int i = 0; i < PL; ++i) {
                const int k = lane * PL + i;
                out[t * NB + k] = p >= 0 ? r[(int64_t)p * NB + k] - s[i] : (T)0;
            }
    }
}

template <typename T, int L>
__global__ void __launch_bounds__(WG) k_csr_spmv_s(int64_t n, const int64_t* rowptr, const int32_t* col,
                                                   const T* val, const T* x, T* y, const T* r_minus,
                                                   const int64_t* scoff) {
    const int lane = tid() & (L - 1);
    const int64_t stride = (int64_t)gridDim.x * (WG / L);
    for (int64_t p = ((int64_t)blockIdx.x * WG + tid()) / L; p < n; p += stride) {
        T s[NB];
#pragma unroll
        for (int k = 0; k < NB; ++k) s[k] = 0;
        slot_row_sums<T, L>(rowptr[p], rowptr[p + 1], lane, col, scoff ? scoff[p] - rowptr[p] : 0, val, x, s);
        slot_reduce<T, L>(s, lane);
        constexpr int PL = L < NB ? NB / L : 1;
        if (lane * PL < NB)
#pragma unroll
            for (int i = 0; i < PL; ++i) {
                const int k = lane * PL + i;
                y[p * NB + k] = r_minus ? r_minus[p * NB + k] - s[i] : s[i];
            }
    }
}

template <typename T, int L>
__global__ void __launch_bounds__(WG) k_csr_spmv_b(int64_t n, const int64_t* rowptr, const int32_t* col,
                                                   const T* val, const T* x, T* y, const T* r_minus,
                                                   const int64_t* scoff) {
    constexpr int NS = L / NB;
    const int lane = tid() & (L - 1), k = lane & (NB - 1), slot = lane / NB;
    const int64_t stride = (int64_t)gridDim.x * (WG / L);
    for (int64_t p = ((int64_t)blockIdx.x * WG + tid()) / L; p < n; p += stride) {
        const int64_t q1 = rowptr[p + 1], cb = scoff ? scoff[p] - rowptr[p] : 0;
        T s = 0;
#pragma unroll 4
        for (int64_t q = rowptr[p] + slot; q < q1; q += NS) s += val[q] * x[(int64_t)col[cb + q] * NB + k];
        for (int off = L / 2; off >= NB; off >>= 1) s += __shfl_xor(s, off, L);
        if (slot == 0) y[p * NB + k] = r_minus ? r_minus[p * NB + k] - s : s;
    }
}

// ---------------------------------------------------------------- subdomain product
// Same work items and partial layout as the single-vector kernel, with NB-wide
// entries.  Each tile is staged once in LDS (rows padded to 65 entries, so both
// row-wise and column-wise reads are free of bank conflicts); the right-hand-side
// entries are wave-uniform and come through the scalar cache.  Every lane works on
// all NB right-hand sides, so one LDS read of a tile entry feeds NB products: for
// the row part wave w takes the tile's columns 16w .. 16w + 15 with lane = row
// (accumulated over the item's tiles in registers), for the column part its rows
// 16w .. 16w + 15 with lane = column; the four waves' partial sums are added in
// wave order through LDS (per tile for the column part, once per item for the
// row part).  The next tile is prefetched into registers (non-temporal loads: the
// tiles stream once per application) while the current one is used.
template <typename T>
__global__ void __launch_bounds__(WG) k_sub_symv_b(const int32_t* items, const int64_t* sub_off,
                                                   const int64_t* tp_off, const T* __restrict__ tiles,
                                                   const T* __restrict__ rloc, const int64_t* scr_off,
                                                   T* __restrict__ scr, int chl) {
    __shared__ T s_t[64 * 65];
    const int s = items[3 * blockIdx.x];
    const int I = items[3 * blockIdx.x + 1];
    const int ch = items[3 * blockIdx.x + 2];
    const int64_t o = sub_off[s];
    const int m = (int)(sub_off[s + 1] - o);
    const int nt = (m + 63) >> 6;
    const int J0 = ch * chl;
    const int nJ = min(chl, I + 1 - J0);
    const int lane = tid() & 63, w = tid() >> 6;
    // wave-uniform quarter of the tile; the right-hand-side entries it multiplies are
    // read at wave-uniform addresses (scalar loads), clamped to the subdomain's last
    // row: the tiles are zero past |Omega|, so a clamped entry adds nothing
    const int wu = __builtin_amdgcn_readfirstlane(w);
    T* part = scr + scr_off[s] * NB;
    T* colpart = part + symv_rowpart_off(nt, chl) * 64 * NB;
    const T* row0 = tiles + tp_off[s] + (int64_t)I * (I + 1) / 2 * 4096;
    T v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = __builtin_nontemporal_load(row0 + (int64_t)J0 * 4096 + i * WG + tid());
    static_assert(WG == 256, "four waves split a tile's columns (row part) and rows (column part)");
    const int q0 = 16 * wu;
    const T* xI = rloc + o * NB;
    T ar[NB];
#pragma unroll
    for (int k = 0; k < NB; ++k) ar[k] = 0;
    for (int jj = 0; jj < nJ; ++jj) {
        const int J = J0 + jj;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int e = i * WG + tid();
            s_t[(e >> 6) * 65 + (e & 63)] = v[i];
        }
        __syncthreads();
        if (jj + 1 < nJ) {
#pragma unroll
            for (int i = 0; i < 16; ++i) v[i] = __builtin_nontemporal_load(row0 + (int64_t)(J + 1) * 4096 + i * WG + tid());
        }
        // row part: lane = row, this wave's 16 columns, all NB right-hand sides
        {
            const T* tr = s_t + lane * 65 + q0;
#pragma unroll 4
            for (int cc = 0; cc < 16; ++cc) {
                const T a = tr[cc];
                const T* xc = xI + (int64_t)min(J * 64 + q0 + cc, m - 1) * NB;
#pragma unroll
                for (int k = 0; k < NB; ++k) ar[k] += a * xc[k];
            }
        }
        if (J < I) {
            // column part: lane = column, this wave's 16 rows; the four row quarters
            // are summed in order through the (then free) tile buffer
            T ac[NB];
#pragma unroll
            for (int k = 0; k < NB; ++k) ac[k] = 0;
#pragma unroll 4
            for (int rr = 0; rr < 16; ++rr) {
                const T a = s_t[(q0 + rr) * 65 + lane];
                const T* xr = xI + (int64_t)min(I * 64 + q0 + rr, m - 1) * NB;
#pragma unroll
                for (int k = 0; k < NB; ++k) ac[k] += a * xr[k];
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < NB; ++k) s_t[(w * 64 + lane) * NB + k] = ac[k];
            __syncthreads();
            const int c = tid() >> 2, k0 = 2 * (tid() & 3);
            T s0 = 0, s1 = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                s0 += s_t[(q * 64 + c) * NB + k0];
                s1 += s_t[(q * 64 + c) * NB + k0 + 1];
            }
            T* cp = colpart + (((int64_t)I * (I - 1) / 2 + J) * 64 + c) * NB + k0;
            cp[0] = s0;
            cp[1] = s1;
        }
    }
    // row part: the four column quarters summed in order
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NB; ++k) s_t[(w * 64 + lane) * NB + k] = ar[k];
    __syncthreads();
    const int r = tid() >> 2, k0 = 2 * (tid() & 3);
    T s0 = 0, s1 = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        s0 += s_t[(q * 64 + r) * NB + k0];
        s1 += s_t[(q * 64 + r) * NB + k0 + 1];
    }
    T* rp = part + ((symv_rowpart_off(I, chl) + ch) * 64 + r) * NB + k0;
    rp[0] = s0;
    rp[1] = s1;
}

// FL threads per DOF sum fixed strided subsets of its partials (all NB
// right-hand sides at once); the FL sums are added in ascending order.
template <typename T, int FL>
__global__ void __launch_bounds__(WG) k_sub_finalize_b(int64_t r0, int64_t r1, const int32_t* pos_sub,
                                                       const int64_t* sub_off, const int64_t* scr_off, const T* scr,
                                                       const int32_t* sub_dofs, T* x, int accumulate, int chl) {
    constexpr int ND = WG / FL;
    __shared__ T s_y[FL][ND][NB];
    const int dl = tid() % ND, j = tid() / ND;
    const int64_t t = r0 + (int64_t)blockIdx.x * ND + dl;
    T y[NB];
#pragma unroll
    for (int q = 0; q < NB; ++q) y[q] = 0;
    if (t < r1) {
        const int s = pos_sub[t];
        const int64_t o = sub_off[s];
        const int c = (int)(t - o);
        const int nt = (int)((sub_off[s + 1] - o + 63) >> 6);
        const int J = c >> 6, l = c & 63;
        const T* part = scr + (scr_off[s] + symv_rowpart_off(J, chl) * 64 + l) * NB;
        const T* colpart = scr + (scr_off[s] + symv_rowpart_off(nt, chl) * 64 + l) * NB;
        const int nch = (J + chl) / chl;
        const int K = nch + (nt - 1 - J);
        for (int k = j; k < K; k += FL) {
            const T* src;
            if (k < nch) {
                src = part + (int64_t)k * 64 * NB;
            } else {
                const int64_t I = J + 1 + (k - nch);
                src = colpart + (I * (I - 1) / 2 + J) * 64 * NB;
            }
#pragma unroll
            for (int q = 0; q < NB; ++q) y[q] += src[q];
        }
    }
#pragma unroll
    for (int q = 0; q < NB; ++q) s_y[j][dl][q] = y[q];
    __syncthreads();
    if (j < NB && t < r1) {
        T v = s_y[0][dl][j];
        for (int q = 1; q < FL; ++q) v += s_y[q][dl][j];
        const int64_t d = sub_dofs ? (int64_t)sub_dofs[t] : t;   // < 0: masked entry
        if (d >= 0) x[d * NB + j] = accumulate ? x[d * NB + j] + v : v;
    }
}

// ---------------------------------------------------------------- transfers
// Restriction rc[coff_i + s] = sum_a Z_i[a, s] t[omega_i[a]] for all right-hand
// sides: work item = (aggregate, 16 columns); t on omega_i is staged in LDS in
// chunks of 256 rows, each wave takes 4 columns, lanes stride the rows.
template <typename T>
__global__ void __launch_bounds__(WG) k_restrict_b(const int32_t* items, const int64_t* agg_ptr,
                                                   const int32_t* agg_dofs, const int64_t* zoff, const int32_t* k,
                                                   const int64_t* coff, const T* Zc, const T* t, T* rc) {
    __shared__ T s_t[256 * NB];
    const int ag = items[2 * blockIdx.x], s0 = items[2 * blockIdx.x + 1];
    const int kk = k[ag];
    const int64_t a0 = agg_ptr[ag];
    const int nw = (int)(agg_ptr[ag + 1] - a0);
    const int lane = tid() & 63, w = tid() >> 6;
    const T* z = Zc + zoff[ag];
    T acc[4][NB];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int q = 0; q < NB; ++q) acc[i][q] = 0;
    for (int c0 = 0; c0 < nw; c0 += 256) {
        const int cn = min(256, nw - c0);
        __syncthreads();
        if (tid() < cn) {
            const T* src = t + (int64_t)agg_dofs[a0 + c0 + tid()] * NB;
#pragma unroll
            for (int q = 0; q < NB; ++q) s_t[tid() * NB + q] = src[q];
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int s = s0 + w + 4 * i;
            if (s < kk) {
                const T* col = z + (int64_t)s * nw + c0;
                for (int a = lane; a < cn; a += 64) {
                    const T zz = col[a];
#pragma unroll
                    for (int q = 0; q < NB; ++q) acc[i][q] += zz * s_t[a * NB + q];
                }
            }
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int s = s0 + w + 4 * i;
        T mine = 0;
#pragma unroll
        for (int q = 0; q < NB; ++q) {
            T v = acc[i][q];
            for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
            if (lane == q) mine = v;
        }
        if (s < kk && lane < NB) rc[(coff[ag] + s) * NB + lane] = mine;
    }
}

// Prolongation x[omega_i[a]] += sum_s Z_i[a, s] ec[coff_i + s]: work item =
// (aggregate, 256 rows); thread per row, ec staged in LDS in chunks of 256 modes.
template <typename T>
__global__ void __launch_bounds__(WG) k_prolong_b(const int32_t* items, const int64_t* agg_ptr,
                                                  const int32_t* agg_dofs, const int64_t* zoff, const int32_t* k,
                                                  const int64_t* coff, const T* Zc, const T* ec, T* x) {
    __shared__ T s_e[256 * NB];
    const int ag = items[2 * blockIdx.x], r0 = items[2 * blockIdx.x + 1];
    const int kk = k[ag];
    const int64_t a0 = agg_ptr[ag];
    const int nw = (int)(agg_ptr[ag + 1] - a0);
    const int a = r0 + tid();
    const T* z = Zc + zoff[ag] + a;
    T acc[NB];
#pragma unroll
    for (int q = 0; q < NB; ++q) acc[q] = 0;
    for (int sc = 0; sc < kk; sc += 256) {
        const int sn = min(256, kk - sc);
        __syncthreads();
        for (int e = tid(); e < sn * NB; e += WG) s_e[e] = ec[(coff[ag] + sc) * NB + e];
        __syncthreads();
        if (a < nw) {
            for (int s = 0; s < sn; ++s) {
                const T zz = z[(int64_t)(sc + s) * nw];
#pragma unroll
                for (int q = 0; q < NB; ++q) acc[q] += zz * s_e[s * NB + q];
            }
        }
    }
    if (a < nw) {
        T* dst = x + (int64_t)agg_dofs[a0 + a] * NB;
#pragma unroll
        for (int q = 0; q < NB; ++q) dst[q] += acc[q];
    }
}

// ---------------------------------------------------------------- small overlaps
// Overlaps with |Omega| <= SMALL_M: the inverse is stored as its packed lower
// triangle (entry (i, j), j <= i, at i (i + 1) / 2 + j), staged in LDS by one
// wave per subdomain; lane i forms y_i = sum_j (A_Omega^{-1})_{ij} r_j over all j in
// ascending order (fixed order) and adds it to x (entries with a negative DOF are
// skipped): subdomains of one colour are disjoint, so the update needs no partial
// sums.  The LDS is sized by the launch's largest overlap (max_m), so small
// overlaps leave room for more waves per CU.  FACT: the packed triangle is a
// lower-triangular factor X and the local solve is X^T (X r): lane i first forms
// w_i = sum_{j <= i} X_ij r_j into LDS, then y_i = sum_{j >= i} X_ji w_j.
//
// Persistent waves: wave b takes subdomains b, b + gridDim.x, ...; the triangle and
// right-hand sides of the next subdomain are loaded into registers while the
// current one is computed from LDS, so the loads of one subdomain overlap the
// arithmetic of the previous one.  Loads go in groups of 8 per lane, a group only
// where the subdomain reaches it; inside a group a slot past the end re-reads the
// last entry (same cache line) and is never stored.
template <typename T, int NR, bool FACT>
__global__ void __launch_bounds__(64) k_small_sub(int32_t s0, int32_t n_sub, const int64_t* sub_off,
                                                  const int32_t* sub_dofs, const int64_t* pk_off, const T* pk,
                                                  const T* rloc, T* x, int max_m) {
    constexpr int PG = 8;
    constexpr int PMAX = ((SMALL_M * (SMALL_M + 1) / 2 + 63) / 64 + PG - 1) / PG * PG;   // triangle loads per lane
    constexpr int XMAX = ((SMALL_M * NR + 63) / 64 + PG - 1) / PG * PG;                   // rhs loads per lane
    extern __shared__ __align__(16) unsigned char s_small[];
    T* s_a = reinterpret_cast<T*>(s_small);
    T* s_x = s_a + max_m * (max_m + 1) / 2;
    T* s_w = s_x + max_m * NR;
    const int lane = tid();
    T ra[PMAX], rx[XMAX];
    int64_t o_n = 0;
    int m_n = 0;
    auto fetch = [&](int sb) {
        o_n = sub_off[s0 + sb];
        m_n = (int)(sub_off[s0 + sb + 1] - o_n);
        const T* A = pk + pk_off[s0 + sb];
        const int np = m_n * (m_n + 1) / 2, nx = m_n * NR;
        const T* r = rloc + o_n * NR;
#pragma unroll
        for (int g = 0; g < PMAX; g += PG)
            if (g * 64 < np) {
#pragma unroll
                for (int u = g; u < g + PG; ++u) ra[u] = A[min(lane + 64 * u, np - 1)];
            }
#pragma unroll
        for (int g = 0; g < XMAX; g += PG)
            if (g * 64 < nx) {
#pragma unroll
                for (int u = g; u < g + PG; ++u) rx[u] = r[min(lane + 64 * u, nx - 1)];
            }
    };
    // the factor form keeps its sums in FP64 (FP32 storage): its two products
    // would otherwise each add FP32 rounding to an ill-conditioned local solve
    using Acc = typename std::conditional<FACT, double, T>::type;
    int sb = blockIdx.x;
    if (sb < n_sub) fetch(sb);
    for (; sb < n_sub; sb += gridDim.x) {
        const int64_t o = o_n;
        const int m = m_n;
        const int np = m * (m + 1) / 2;
        __syncthreads();                                   // the previous subdomain's reads of LDS are done
#pragma unroll
        for (int u = 0; u < PMAX; ++u)
            if (lane + 64 * u < np) s_a[lane + 64 * u] = ra[u];
#pragma unroll
        for (int u = 0; u < XMAX; ++u)
            if (lane + 64 * u < m * NR) s_x[lane + 64 * u] = rx[u];
        __syncthreads();
        // this subdomain's DOFs and their current x, loaded ahead of the prefetch so
        // that waiting for them does not wait for it (lanes >= m read a valid entry and
        // store nothing; a masked entry reads x[0]); the colour's subdomains are
        // disjoint, so no other wave writes these x during the launch
        const int32_t d = m > 0 ? sub_dofs[o + min(lane, m - 1)] : -1;
        T xo[NR];
#pragma unroll
        for (int k = 0; k < NR; ++k) xo[k] = x[(int64_t)max(d, 0) * NR + k];
        if (sb + (int)gridDim.x < n_sub) fetch(sb + gridDim.x);   // in flight during the arithmetic below
        if (FACT) {
            if (lane < m) {
                const int i = lane;
                const int ri = i * (i + 1) / 2;
                Acc wv[NR];
#pragma unroll
                for (int k = 0; k < NR; ++k) wv[k] = 0;
                for (int j = 0; j <= i; ++j) {
                    const Acc a = s_a[ri + j];
#pragma unroll
                    for (int k = 0; k < NR; ++k) wv[k] += a * (Acc)s_x[j * NR + k];
                }
#pragma unroll
                for (int k = 0; k < NR; ++k) s_w[i * NR + k] = (T)wv[k];
            }
            __syncthreads();
        }
        if (lane < m) {
            const int i = lane;
            const int ri = i * (i + 1) / 2;
            Acc y[NR];
#pragma unroll
            for (int k = 0; k < NR; ++k) y[k] = 0;
            if (FACT) {
                for (int j = i; j < m; ++j) {
                    const Acc a = s_a[j * (j + 1) / 2 + i];
#pragma unroll
                    for (int k = 0; k < NR; ++k) y[k] += a * (Acc)s_w[j * NR + k];
                }
            } else {
                for (int j = 0; j < m; ++j) {
                    const T a = s_a[j <= i ? ri + j : j * (j + 1) / 2 + i];
#pragma unroll
                    for (int k = 0; k < NR; ++k) y[k] += a * s_x[j * NR + k];
                }
            }
            if (d >= 0) {                        // < 0: masked entry
                T* dst = x + (int64_t)d * NR;
#pragma unroll
                for (int k = 0; k < NR; ++k) dst[k] = xo[k] + y[k];
            }
        }
    }
}

// The same for NB right-hand sides in FP32 on the matrix cores, y^T = x^T A with A from the packed
// triangle: 16 rows of A, four columns at a time, against four rows of x (8 of the 16 rows of x^T
// carry right-hand sides).  With a lane per row a step took an entry of A and two 16-byte rows of
// x from LDS, whose one pipe the CU's waves share, for 8 products a lane; here it takes an entry
// of each for 16 x 16 x 4.  The transposed product leaves a row's right-hand sides in a lane, four
// at a time, as they lie in x.  The data go to LDS without registers in between, so that a CU
// holds the wave of every subdomain at once (with the next one's loads waiting in registers 12
// waves, 3530 subdomains on 3072 of them: nearly two full rounds).  3500 overlaps of up to 50
// DOFs: 12.9 -> 9.7 us.
// cnt consecutive values from memory to LDS without passing through registers
__device__ inline void wave_to_lds(const float* src, float* dst, int cnt) {
    for (int g = 0; g < cnt; g += 64)
        if (g + tid() < cnt)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + g + tid()),
                                             (__attribute__((address_space(3))) void*)(dst + g), 4, 0, 0);
}

__global__ void __launch_bounds__(64) k_small_sub_mm(int32_t s0, const int64_t* sub_off, const int32_t* sub_dofs,
                                                     const int64_t* pk_off, const float* pk, const float* rloc, float* x,
                                                     int max_m) {
    using Acc = float __attribute__((ext_vector_type(4)));
    static_assert(NB == 8, "a lane of the first two groups of 16 holds four right-hand sides of a row");
    constexpr int RT = (SMALL_M + 15) / 16;
    extern __shared__ __align__(16) unsigned char s_small[];
    float* s_a = reinterpret_cast<float*>(s_small);
    float* s_x = s_a + max_m * (max_m + 1) / 2;        // rows up to a multiple of four, zero past m
    const int lane = tid(), c = lane & 15, q = lane >> 4;
    const int64_t sb = s0 + (int64_t)blockIdx.x;
    const int64_t o = sub_off[sb];
    const int m = (int)(sub_off[sb + 1] - o);
    if (m < 1) return;
    const int m4 = (m + 3) & ~3;
    if (lane < (m4 - m) * NB) s_x[m * NB + lane] = 0;  // before the copies, which a later store would wait for
    // DOFs of the rows this lane writes; rows >= m read a valid entry and store nothing
    int32_t d[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) d[t] = sub_dofs[o + min(16 * t + c, m - 1)];
    wave_to_lds(rloc + o * NB, s_x, m * NB);
    wave_to_lds(pk + pk_off[sb], s_a, m * (m + 1) / 2);
    // and their current x (a masked entry reads x[0])
    float4 xo[RT];
    const bool writes = q < 2;
    if (writes)
#pragma unroll
        for (int t = 0; t < RT; ++t) xo[t] = *reinterpret_cast<const float4*>(x + (int64_t)max(d[t], 0) * NB + 4 * q);
    Acc y[RT];
    int ri[RT], ti[RT];                                // this lane's row of A in every row tile
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        y[t] = Acc{0, 0, 0, 0};
        ri[t] = min(16 * t + c, m - 1);
        ti[t] = ri[t] * (ri[t] + 1) / 2;
    }
    __builtin_amdgcn_s_waitcnt(0);                     // the copies to LDS are done
    __syncthreads();
    for (int k = 0; k < m4; k += 4) {
        const int j = min(k + q, m - 1), tj = j * (j + 1) / 2;
        const float b = s_x[(k + q) * NB + (c & (NB - 1))];
        float a[RT];
#pragma unroll
        for (int t = 0; t < RT; ++t) a[t] = s_a[j <= ri[t] ? ti[t] + j : tj + ri[t]];
#pragma unroll
        for (int t = 0; t < RT; ++t) y[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(b, a[t], y[t], 0, 0, 0);
    }
    if (writes)
#pragma unroll
        for (int t = 0; t < RT; ++t)
            if (16 * t + c < m && d[t] >= 0)
                *reinterpret_cast<float4*>(x + (int64_t)d[t] * NB + 4 * q) =
                    make_float4(xo[t].x + y[t][0], xo[t].y + y[t][1], xo[t].z + y[t][2], xo[t].w + y[t][3]);
}

// Transfers for aggregates with |omega| <= SMALL_M, one thread per coarse DOF for
// the restriction and per aggregate entry for the prolongation, each for all NR
// right-hand sides (the index and the Z entry are loaded once for the NR products;
// AL: the NR interleaved values of a DOF are 16-byte aligned and load as 16-byte
// vectors); four independent entries (modes) per step, summed in four partial sums
// added in a fixed order.
template <typename T, int NR, bool AL>
__device__ inline void load_nr(const T* p, T (&v)[NR]) {
    const T* q = AL ? static_cast<const T*>(__builtin_assume_aligned(p, 16)) : p;
#pragma unroll
    for (int k = 0; k < NR; ++k) v[k] = q[k];
}

template <typename T, int NR, bool AL>
__global__ void __launch_bounds__(WG) k_restrict_small(int64_t nc, const int32_t* agg_of_c, const int64_t* agg_ptr,
                                                       const int32_t* agg_dofs, const int64_t* zoff,
                                                       const int64_t* coff, const T* Zc, const T* t, T* rc) {
    for (int64_t c = blockIdx.x * (int64_t)WG + tid(); c < nc; c += (int64_t)gridDim.x * WG) {
        const int ag = agg_of_c[c];
        if (ag < 0) continue;
        const int64_t a0 = agg_ptr[ag];
        const int nw = (int)(agg_ptr[ag + 1] - a0);
        const T* z = Zc + zoff[ag] + (c - coff[ag]) * nw;
        const int32_t* dd = agg_dofs + a0;
        // four independent entries per step: their indices, then their gathers
        T acc[4][NR];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int k = 0; k < NR; ++k) acc[u][k] = 0;
        int a = 0;
        for (; a + 4 <= nw; a += 4) {
            int32_t d[4];
            T zz[4], tv[4][NR];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                d[u] = dd[a + u];
                zz[u] = z[a + u];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) load_nr<T, NR, AL>(t + (int64_t)d[u] * NR, tv[u]);
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int k = 0; k < NR; ++k) acc[u][k] += zz[u] * tv[u][k];
        }
        for (; a < nw; ++a) {
            T tv[NR];
            const T zz = z[a];
            load_nr<T, NR, AL>(t + (int64_t)dd[a] * NR, tv);
#pragma unroll
            for (int k = 0; k < NR; ++k) acc[0][k] += zz * tv[k];
        }
        T* out = AL ? static_cast<T*>(__builtin_assume_aligned(rc + c * NR, 16)) : rc + c * NR;
#pragma unroll
        for (int k = 0; k < NR; ++k) out[k] = (acc[0][k] + acc[1][k]) + (acc[2][k] + acc[3][k]);
    }
}

template <typename T, int NR, bool AL>
__global__ void __launch_bounds__(WG) k_prolong_small(int64_t na, const int32_t* agg_of_p, const int64_t* agg_ptr,
                                                      const int32_t* agg_dofs, const int64_t* zoff,
                                                      const int32_t* k, const int64_t* coff, const T* Zc,
                                                      const T* ec, T* x) {
    for (int64_t p = blockIdx.x * (int64_t)WG + tid(); p < na; p += (int64_t)gridDim.x * WG) {
        const int ag = agg_of_p[p];
        if (ag < 0) continue;
        const int64_t a0 = agg_ptr[ag];
        const int nw = (int)(agg_ptr[ag + 1] - a0);
        const int kk = k[ag];
        const T* z = Zc + zoff[ag] + (p - a0);
        const T* ev = ec + coff[ag] * NR;
        T acc[4][NR];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int q = 0; q < NR; ++q) acc[u][q] = 0;
        int s = 0;
        for (; s + 4 <= kk; s += 4) {
            T zz[4], e[4][NR];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                zz[u] = z[(int64_t)(s + u) * nw];
                load_nr<T, NR, AL>(ev + (int64_t)(s + u) * NR, e[u]);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int q = 0; q < NR; ++q) acc[u][q] += zz[u] * e[u][q];
        }
        for (; s < kk; ++s) {
            T e[NR];
            const T zz = z[(int64_t)s * nw];
            load_nr<T, NR, AL>(ev + (int64_t)s * NR, e);
#pragma unroll
            for (int q = 0; q < NR; ++q) acc[0][q] += zz * e[q];
        }
        T* dst = x + (int64_t)agg_dofs[p] * NR;
        if (AL) dst = static_cast<T*>(__builtin_assume_aligned(dst, 16));
        T old[NR];
#pragma unroll
        for (int q = 0; q < NR; ++q) old[q] = dst[q];
#pragma unroll
        for (int q = 0; q < NR; ++q) dst[q] = old[q] + ((acc[0][q] + acc[1][q]) + (acc[2][q] + acc[3][q]));
    }
}

__global__ void k_scatter_sol(int64_t n, int nr, const double* X, double* x, int64_t ldx) {
    for (int64_t e = blockIdx.x * (int64_t)WG + tid(); e < n * NB; e += (int64_t)gridDim.x * WG) {
        const int64_t d = e / NB;
        const int k = (int)(e % NB);
        if (k < nr) x[k * ldx + d] = X[e];
    }
}

// ---------------------------------------------------------------- segmented PCG
// Block b of the table covers DOFs [lo, hi) of one segment; thread = (DOF lane,
// right-hand side).  An iteration is bound by the latency of its chain of small
// launches and, for blocks of right-hand sides, by the vector traffic, so the
// scalars have no launches of their own: a kernel that needs a dot product adds the
// block partials of its segment itself (every block the same sum in the same order),
// and the vectors the cycle starts from (its FP32 residual, its zero iterate) are
// written by the kernel that has the residual in registers.  Six launches per
// iteration around the cycle instead of eleven (FP64) or fifteen (FP32 cycle): 162 DOFs
// 1.17 -> 0.92 ms per solve, 33,800 DOFs with an FP32 cycle 5.95 -> 5.48 ms.
constexpr int PCG_WG = 256;
constexpr int PCG_U = 4;                               // vector entries per thread in flight

// Sum of u over the block for every right-hand side k = tid % NR, in a fixed order; all
// threads of right-hand side k get the result.  s_w: WG / 64 * NR entries.
template <int NR>
__device__ inline double block_sum(double u, double* s_w) {
    const int lane = tid() & 63, w = tid() >> 6;
#pragma unroll
    for (int off = NR; off < 64; off <<= 1) u += __shfl_xor(u, off, 64);
    __syncthreads();                                   // s_w may hold an earlier sum
    if (lane < NR) s_w[w * NR + lane] = u;
    __syncthreads();
    const int k = tid() % NR;
    double v = s_w[k];
#pragma unroll
    for (int q = 1; q < PCG_WG / 64; ++q) v += s_w[q * NR + k];
    return v;
}

// The dot product of segment s from its block partials (part[b * NR + k]).
template <int NR>
__device__ inline double seg_total(const double* part, int b0, int b1, double* s_w) {
    constexpr int DL = PCG_WG / NR;
    const int k = tid() % NR;
    double u = 0.0;
#pragma unroll 4
    for (int b = b0 + tid() / NR; b < b1; b += DL) u += part[(int64_t)b * NR + k];
    return block_sum<NR>(u, s_w);
}

// partials of <a0, b0> and, with a1, <a1, b1> (b0, b1 of type Z, products in FP64)
template <int NR, typename Z>
__global__ void __launch_bounds__(PCG_WG) k_seg_dot(const int64_t* blk_lo, const int64_t* blk_hi, const double* a0,
                                                    const Z* b0, const double* a1, const Z* b1, double* part0,
                                                    double* part1) {
    __shared__ double s_w[PCG_WG / 64 * NR];
    const int b = blockIdx.x;
    constexpr int DL = PCG_WG / NR;
    const int64_t e0 = blk_lo[b] * NR, e1 = blk_hi[b] * NR;
    double u = 0.0, v = 0.0;
#pragma unroll 4
    for (int64_t e = e0 + tid(); e < e1; e += DL * NR) {
        u += a0[e] * (double)b0[e];
        if (a1) v += a1[e] * (double)b1[e];
    }
    u = block_sum<NR>(u, s_w);
    if (tid() < NR) part0[(int64_t)b * NR + tid()] = u;
    if (a1) {
        v = block_sum<NR>(v, s_w);
        if (tid() < NR) part1[(int64_t)b * NR + tid()] = v;
    }
}

// out[s * NR + k] = sum over the blocks of segment s (one workgroup per segment); host:
// optional pinned copy of the first NR sums
template <int NR>
__global__ void __launch_bounds__(PCG_WG) k_seg_sum(const int32_t* seg_blk, const double* part, double* out,
                                                    double* host) {
    __shared__ double s_w[PCG_WG / 64 * NR];
    const int s = blockIdx.x;
    const double v = seg_total<NR>(part, seg_blk[s], seg_blk[s + 1], s_w);
    if (tid() < NR) {
        out[s * NR + tid()] = v;
        if (host && s == 0) host[tid()] = v;
    }
}

// Start of a solve: r = b, x = 0 (b: nr right-hand sides at stride ldb, the others zero),
// the cycle's start vectors, partials of <b, b> and of the count of non-finite entries.
template <int NR, typename Z>
__global__ void __launch_bounds__(PCG_WG) k_pcg_begin(const int64_t* blk_lo, const int64_t* blk_hi, int nr,
                                                      const double* b, int64_t ldb, double* r, double* x, float* r32,
                                                      Z* z, double* part_bb, double* part_bad) {
    __shared__ double s_w[PCG_WG / 64 * NR];
    const int blk = blockIdx.x, k = tid() % NR;
    constexpr int DL = PCG_WG / NR;
    double u = 0.0, bad = 0.0;
#pragma unroll 2
    for (int64_t d = blk_lo[blk] + tid() / NR; d < blk_hi[blk]; d += DL) {
        const double v = k < nr ? b[k * ldb + d] : 0.0;
        const int64_t e = d * NR + k;
        r[e] = v;
        x[e] = 0.0;
        if (r32) r32[e] = (float)v;
        z[e] = (Z)0;
        u += v * v;
        if (!isfinite(v)) bad += 1.0;
    }
    u = block_sum<NR>(u, s_w);
    if (tid() < NR) part_bb[(int64_t)blk * NR + tid()] = u;
    bad = block_sum<NR>(bad, s_w);
    if (tid() < NR) part_bad[(int64_t)blk * NR + tid()] = bad;
}

// A wave adds the partials of a segment's NR pairs: lanes = (block lane, right-hand side).
template <int NR>
__device__ inline double wave_seg_total(const double* part, int b0, int b1) {
    const int lane = tid() & 63, k = lane % NR;
    double u = 0.0;
#pragma unroll 4
    for (int b = b0 + lane / NR; b < b1; b += 64 / NR) u += part[(int64_t)b * NR + k];
#pragma unroll
    for (int off = NR; off < 64; off <<= 1) u += __shfl_xor(u, off, 64);
    return u;
}

constexpr int PCG_CHECK_WG = 1024;

// Sums of two sets of partials (p1 NULL: one) for every pair, a wave per segment: for tables of so
// many segments that one workgroup, a wave per segment, takes longer than a launch.
template <int NR>
__global__ void __launch_bounds__(PCG_WG) k_seg_totals(int n_seg, const int32_t* seg_blk, const double* p0,
                                                       const double* p1, double* tot0, double* tot1) {
    const int s = (int)blockIdx.x * (PCG_WG / 64) + (tid() >> 6), lane = tid() & 63;
    if (s >= n_seg) return;
    const double u = wave_seg_total<NR>(p0, seg_blk[s], seg_blk[s + 1]);
    const double v = p1 ? wave_seg_total<NR>(p1, seg_blk[s], seg_blk[s + 1]) : 0.0;
    if (lane < NR) {
        tot0[s * NR + lane] = u;
        if (p1) tot1[s * NR + lane] = v;
    }
}

// f(pair, first sum, second sum) for every pair, from one workgroup: the sums as given (tot), else a
// wave per segment adds the partials
template <int NR, class F>
__device__ inline void each_pair(int n_seg, const int32_t* seg_blk, const double* p0, const double* p1,
                                 const double* tot0, const double* tot1, F&& f) {
    if (tot0) {
        for (int i = tid(); i < n_seg * NR; i += PCG_CHECK_WG) f(i, tot0[i], p1 ? tot1[i] : 0.0);
        return;
    }
    const int lane = tid() & 63;
    for (int s = tid() >> 6; s < n_seg; s += PCG_CHECK_WG / 64) {
        const double u = wave_seg_total<NR>(p0, seg_blk[s], seg_blk[s + 1]);
        const double v = p1 ? wave_seg_total<NR>(p1, seg_blk[s], seg_blk[s + 1]) : 0.0;
        if (lane < NR) f(s * NR + lane, u, v);
    }
}

template <int NR>
__global__ void __launch_bounds__(PCG_CHECK_WG) k_pcg_init(int n_seg, const int32_t* seg_blk, const double* part_bb,
                                                           const double* part_bad, const double* tot_bb,
                                                           const double* tot_bad, double* bb, int32_t* act,
                                                           int32_t* iters, double* relres, int32_t* st) {
    __shared__ int s_bad;
    if (tid() == 0) s_bad = 0;
    __syncthreads();
    each_pair<NR>(n_seg, seg_blk, part_bb, part_bad, tot_bb, tot_bad, [&](int i, double v, double bad) {
        bb[i] = v;
        act[i] = v > 0.0 ? 1 : 0;
        iters[i] = 0;
        relres[i] = v > 0.0 ? 1.0 : 0.0;
        if (bad > 0.0) s_bad = 1;
    });
    __syncthreads();
    if (tid() == 0) {
        st[PCG_ST_COUNT] = 0;
        st[PCG_ST_IT] = 0;
        st[PCG_ST_FLAG] = 0;
        st[PCG_ST_BAD] = s_bad;
    }
}

// alpha = <r, z> / <p, q> of the block's segment from the partials of <p, q> (0 for
// pairs that have left the iteration and at a breakdown), then x += alpha p,
// r -= alpha q, the partials of <r, r> and the cycle's start vectors; rold: the residual
// before the step (flexible beta).  rz has two slots, used in turn: the iteration it
// reads the one the previous iteration wrote.  Bound by the vector traffic (four vectors
// in, up to five out).  The block table decides how much of the chip that traffic uses: at
// 2048 DOFs a block, the 8-vector blocks of a 243,420-DOF batch ran 126 workgroups of 64
// serial steps, 59.6 us; at 256 DOFs (batch solve 17.7 -> 15.3 ms) there are 957 of 8.
template <int NR, typename Z>
__global__ void __launch_bounds__(PCG_WG) k_pcg_update_xr(int n_seg, const int32_t* blk_seg,
                                                          const int64_t* blk_lo, const int64_t* blk_hi,
                                                          const int32_t* seg_blk,
                                                          const int32_t* act, const double* rz2, int nsm,
                                                          const double* part_pq, const double* p, const double* q,
                                                          double* x, double* r, double* rold, float* r32, Z* z,
                                                          double* part_rr, int32_t* st) {
    __shared__ double s_w[PCG_WG / 64 * NR];
    const int b = blockIdx.x;
    // the first chunk of the vectors arrives while the scalars are formed
    const int64_t e0 = blk_lo[b] * NR, e1 = blk_hi[b] * NR;
    double pv[PCG_U], qv[PCG_U], xv[PCG_U], rv[PCG_U];
    auto load = [&](int64_t e) {
#pragma unroll
        for (int j = 0; j < PCG_U; ++j) {
            const int64_t ec = min(e + tid() + j * PCG_WG, e1 - 1);
            pv[j] = p[ec];
            qv[j] = q[ec];
            xv[j] = x[ec];
            rv[j] = r[ec];
        }
    };
    load(e0);
    const int s = n_seg == 1 ? 0 : blk_seg[b];
    const int k = tid() % NR, i = s * NR + k;
    const int b0 = n_seg == 1 ? 0 : seg_blk[s], b1 = n_seg == 1 ? (int)gridDim.x : seg_blk[s + 1];
    const bool on = act[i] != 0;
    const double rzv = rz2[(int64_t)(st[PCG_ST_IT] & 1) * nsm + i];
    const double d = seg_total<NR>(part_pq, b0, b1, s_w);
    double a = 0.0;
    if (on) {
        // breakdown cause bits: 1 p^T A p <= 0, 2 p^T A p or r^T z not finite
        int bits = 0;
        if (!isfinite(d) || !isfinite(rzv)) bits = 2;
        else if (!(d > 0.0)) bits = 1;
        else a = rzv / d;
        if (bits && b == b0 && tid() < NR) atomicOr(st + PCG_ST_FLAG, bits);
    }
    double u = 0.0;
    for (int64_t ec = e0; ec < e1; ec += PCG_U * PCG_WG) {
        if (ec > e0) load(ec);
#pragma unroll
        for (int j = 0; j < PCG_U; ++j) {
            const int64_t e = ec + tid() + j * PCG_WG;
            if (e >= e1) break;
            double re = rv[j];
            if (rold) rold[e] = re;
            if (on) {
                x[e] = xv[j] + a * pv[j];
                re -= a * qv[j];
                r[e] = re;
            }
            if (r32) r32[e] = (float)re;
            z[e] = (Z)0;
            u += re * re;
        }
    }
    u = block_sum<NR>(u, s_w);
    if (tid() < NR) part_rr[(int64_t)b * NR + tid()] = u;
}

// State transitions and the active count, one workgroup; the status goes to the device and to
// the host's pinned mirror, which the host reads after the launch has ended (no copy launch);
// behind them the largest |r|^2 / (tol^2 |b|^2) of the pairs still active.
template <int NR>
__global__ void __launch_bounds__(PCG_CHECK_WG) k_pcg_check(int n_seg, const int32_t* seg_blk, const double* part_rr,
                                                            const double* tot_rr, double tol2, const double* bb,
                                                            int32_t* act, int32_t* iters, double* relres, int32_t* st,
                                                            int32_t* host_st) {
    __shared__ int s_count, s_flag;
    __shared__ unsigned long long s_excess;             // non-negative doubles order like their bits
    if (tid() == 0) s_count = s_flag = 0, s_excess = 0;
    __syncthreads();
    const int it = st[PCG_ST_IT] + 1;
    int count = 0, flag = 0;
    unsigned long long excess = 0;
    each_pair<NR>(n_seg, seg_blk, part_rr, nullptr, tot_rr, nullptr, [&](int i, double v, double) {
        if (!act[i]) return;
        if (!isfinite(v)) {
            flag = 4;                                   // residual norm not finite
            return;
        }
        relres[i] = sqrt(v / bb[i]);
        iters[i] = it;
        if (v <= tol2 * bb[i]) {
            act[i] = 0;
        } else {
            ++count;
            excess = max(excess, (unsigned long long)__double_as_longlong(v / (tol2 * bb[i])));
        }
    });
    if (count) {
        atomicAdd(&s_count, count);
        atomicMax(&s_excess, excess);
    }
    if (flag) atomicOr(&s_flag, flag);
    __syncthreads();
    if (tid() == 0) {
        const int flag = st[PCG_ST_FLAG] | s_flag;
        st[PCG_ST_COUNT] = s_count;
        st[PCG_ST_IT] = it;
        st[PCG_ST_FLAG] = flag;
        host_st[PCG_ST_COUNT] = s_count;
        host_st[PCG_ST_IT] = it;
        host_st[PCG_ST_FLAG] = flag;
        host_st[PCG_ST_BAD] = st[PCG_ST_BAD];
        *reinterpret_cast<double*>(host_st + PCG_ST_WORDS) = __longlong_as_double((long long)s_excess);
        __threadfence_system();
    }
}

// beta = (<r, z> - <rold, z>) / <r, z>_old of the block's segment (part_rzo NULL: the
// standard beta) and p = z + beta p; before the first iteration (counter 0) p = z.  The
// segment's first block writes <r, z> to the slot the next step reads.
template <int NR, typename Z>
__global__ void __launch_bounds__(PCG_WG) k_pcg_update_p(int n_seg, const int32_t* blk_seg,
                                                         const int64_t* blk_lo, const int64_t* blk_hi,
                                                         const int32_t* seg_blk,
                                                         const int32_t* act, double* rz2, int nsm,
                                                         const double* part_rz, const double* part_rzo, const Z* z,
                                                         double* p, int32_t* st) {
    __shared__ double s_w[PCG_WG / 64 * NR];
    const int b = blockIdx.x;
    const int64_t e0 = blk_lo[b] * NR, e1 = blk_hi[b] * NR;
    const int it = st[PCG_ST_IT];
    // the first chunk of the vectors arrives while the scalars are formed
    Z zv[PCG_U];
    double pv[PCG_U];
    auto load = [&](int64_t e) {
#pragma unroll
        for (int j = 0; j < PCG_U; ++j) {
            const int64_t ec = min(e + tid() + j * PCG_WG, e1 - 1);
            zv[j] = z[ec];
            pv[j] = p[ec];
        }
    };
    load(e0);
    const int s = n_seg == 1 ? 0 : blk_seg[b];
    const int k = tid() % NR, i = s * NR + k;
    const int b0 = n_seg == 1 ? 0 : seg_blk[s], b1 = n_seg == 1 ? (int)gridDim.x : seg_blk[s + 1];
    const bool on = act[i] != 0;
    const double rz_old = rz2[(int64_t)((it + 1) & 1) * nsm + i];
    const double rz_new = seg_total<NR>(part_rz, b0, b1, s_w);
    double num = rz_new;
    if (part_rzo && it > 0) num -= seg_total<NR>(part_rzo, b0, b1, s_w);
    double bt = 0.0;
    if (on && it > 0) {
        bt = num / rz_old;
        if (!isfinite(bt) && b == b0 && tid() < NR) atomicOr(st + PCG_ST_FLAG, 8);   // beta not finite
    }
    if (b == b0 && tid() < NR) rz2[(int64_t)(it & 1) * nsm + i] = on || it == 0 ? rz_new : rz_old;
    if (!on && it > 0) return;
    for (int64_t ec = e0; ec < e1; ec += PCG_U * PCG_WG) {
        if (ec > e0) load(ec);
#pragma unroll
        for (int j = 0; j < PCG_U; ++j) {
            const int64_t e = ec + tid() + j * PCG_WG;
            if (e < e1) p[e] = it == 0 ? (double)zv[j] : (double)zv[j] + bt * pv[j];   // p holds anything before
        }
    }
}

}  // namespace

// ====================================================================== launchers

// The residual rows of a supernode-blocked level by supernode row blocks, for blocks
// of NB right-hand sides: L lanes per block (blk as in k_sup_resid_blocks) take its
// shared column list; per entry a lane gathers the NB interleaved x values once and
// uses them for up to 4 rows of the block at a time (slots past the block's end
// repeat its last row and are never stored).  Per row the products, the per-lane
// sums and the cross-lane sums are those of k_csr_resid_rows_s for the same L: the
// results are bit-identical to it.
template <typename T, int L>
__global__ void __launch_bounds__(WG) k_sup_resid_blocks_s(int64_t nblk, const int32_t* blk, const int32_t* rows,
                                                           const int64_t* rowptr, const int32_t* scol,
                                                           const int64_t* scoff, const T* val, const T* x,
                                                           const T* r, T* out, int x_zero) {
    constexpr int RB = 4;
    const int lane = tid() & (L - 1);
    const int64_t stride = (int64_t)gridDim.x * (WG / L);
    for (int64_t b = ((int64_t)blockIdx.x * WG + tid()) / L; b < nblk; b += stride) {
        const int32_t t0 = blk[2 * b], nb = blk[2 * b + 1];
        const int32_t p0 = rows[t0];
        const int64_t q0 = rowptr[p0], q1 = rowptr[p0 + 1];
        const int64_t cb = scoff[p0] - q0;   // the list entry of position q is scol[cb + q]
        for (int j0 = 0; j0 < nb; j0 += RB) {
            int32_t p[RB];
            int64_t vo[RB];   // value offset of row j relative to the first row's
#pragma unroll
            for (int j = 0; j < RB; ++j) {
                p[j] = rows[t0 + min(j0 + j, nb - 1)];
                vo[j] = rowptr[p[j]] - q0;
            }
            T s[RB][NB];
#pragma unroll
            for (int j = 0; j < RB; ++j)
#pragma unroll
                for (int k = 0; k < NB; ++k) s[j][k] = 0;
            if (!x_zero) {
                const int nit = (int)((q1 - q0 + L - 1) / L);
                for (int it = 0; it < nit; it += 2) {
                    const int64_t qa = q0 + lane + (int64_t)it * L, qb = qa + L;
                    const int64_t qac = qa < q1 ? qa : q1 - 1, qbc = qb < q1 ? qb : q1 - 1;
                    const int32_t ca = scol[cb + qac], cc = scol[cb + qbc];
                    T va[RB], vb[RB];
#pragma unroll
                    for (int j = 0; j < RB; ++j) {
                        va[j] = val[vo[j] + qac];
                        vb[j] = val[vo[j] + qbc];
                    }
                    T xa[NB], xb[NB];
                    load_xrow(x + (int64_t)ca * NB, xa);
                    load_xrow(x + (int64_t)cc * NB, xb);
#pragma unroll
                    for (int j = 0; j < RB; ++j) {
                        const T wa = qa < q1 ? va[j] : (T)0, wb = qb < q1 ? vb[j] : (T)0;
#pragma unroll
                        for (int k = 0; k < NB; ++k) s[j][k] += wa * xa[k];
#pragma unroll
                        for (int k = 0; k < NB; ++k) s[j][k] += wb * xb[k];
                    }
                }
            }
            constexpr int PL = L < NB ? NB / L : 1;   // right-hand sides per writing lane
#pragma unroll
            for (int j = 0; j < RB; ++j) {
                slot_reduce<T, L>(s[j], lane);
                if (j0 + j < nb && lane * PL < NB)
#pragma unroll
                    for (int i = 0; i < PL; ++i) {
                        const int k = lane * PL + i;
                        out[(int64_t)(t0 + j0 + j) * NB + k] = r[(int64_t)p[j] * NB + k] - s[j][i];
                    }
            }
        }
    }
}

template <typename T>
void launch_sup_resid_blocks_b(int64_t nblk, const int32_t* blk, const int32_t* rows, const int64_t* rowptr,
                               const int32_t* scol, const int64_t* scoff, const T* val, const T* x, const T* r, T* out,
                               bool x_zero, int lanes, hipStream_t st) {
    if (nblk <= 0) return;
    const int xz = x_zero ? 1 : 0;
    if (lanes <= 4)
        hipLaunchKernelGGL((k_sup_resid_blocks_s<T, 4>), dim3(grid_for(nblk * 4)), dim3(WG), 0, st, nblk, blk, rows,
                           rowptr, scol, scoff, val, x, r, out, xz);
    else if (lanes <= 8)
        hipLaunchKernelGGL((k_sup_resid_blocks_s<T, 8>), dim3(grid_for(nblk * 8)), dim3(WG), 0, st, nblk, blk, rows,
                           rowptr, scol, scoff, val, x, r, out, xz);
    else
        hipLaunchKernelGGL((k_sup_resid_blocks_s<T, 16>), dim3(grid_for(nblk * 16)), dim3(WG), 0, st, nblk, blk,
                           rows, rowptr, scol, scoff, val, x, r, out, xz);
}

template <typename T>
void launch_csr_resid_rows_b(int64_t nrows, const int32_t* rows, const int64_t* rowptr, const int32_t* col,
                             const T* val, const T* x, const T* r, T* out, bool x_zero, int lanes, hipStream_t st,
                             const int64_t* scoff) {
    if (nrows <= 0) return;
    if (lanes <= 4)
        hipLaunchKernelGGL((k_csr_resid_rows_s<T, 4>), dim3(grid_for(nrows * 4)), dim3(WG), 0, st, nrows, rows,
                           rowptr, col, val, x, r, out, x_zero ? 1 : 0, scoff);
    else if (lanes <= 8)
        hipLaunchKernelGGL((k_csr_resid_rows_s<T, 8>), dim3(grid_for(nrows * 8)), dim3(WG), 0, st, nrows, rows,
                           rowptr, col, val, x, r, out, x_zero ? 1 : 0, scoff);
    else if (lanes <= 16)
        hipLaunchKernelGGL((k_csr_resid_rows_s<T, 16>), dim3(grid_for(nrows * 16)), dim3(WG), 0, st, nrows, rows,
                           rowptr, col, val, x, r, out, x_zero ? 1 : 0, scoff);
    else if (lanes >= 64)
        hipLaunchKernelGGL((k_csr_resid_rows_b<T, 64>), dim3(grid_for(nrows * 64)), dim3(WG), 0, st, nrows, rows,
                           rowptr, col, val, x, r, out, x_zero ? 1 : 0, scoff);
    else
        hipLaunchKernelGGL((k_csr_resid_rows_b<T, 32>), dim3(grid_for(nrows * 32)), dim3(WG), 0, st, nrows, rows,
                           rowptr, col, val, x, r, out, x_zero ? 1 : 0, scoff);
}

template <typename T>
void launch_csr_spmv_b(int64_t n, const int64_t* rowptr, const int32_t* col, const T* val, const T* x, T* y,
                       const T* r_minus, int lanes, hipStream_t st, const int64_t* scoff) {
    if (n <= 0) return;
    if (lanes <= 4)
        hipLaunchKernelGGL((k_csr_spmv_s<T, 4>), dim3(grid_for(n * 4)), dim3(WG), 0, st, n, rowptr, col, val, x, y,
                           r_minus, scoff);
    else if (lanes <= 8)
        hipLaunchKernelGGL((k_csr_spmv_s<T, 8>), dim3(grid_for(n * 8)), dim3(WG), 0, st, n, rowptr, col, val, x, y,
                           r_minus, scoff);
    else if (lanes <= 16)
        hipLaunchKernelGGL((k_csr_spmv_s<T, 16>), dim3(grid_for(n * 16)), dim3(WG), 0, st, n, rowptr, col, val, x, y,
                           r_minus, scoff);
    else if (lanes >= 64)
        hipLaunchKernelGGL((k_csr_spmv_b<T, 64>), dim3(grid_for(n * 64)), dim3(WG), 0, st, n, rowptr, col, val, x, y,
                           r_minus, scoff);
    else
        hipLaunchKernelGGL((k_csr_spmv_b<T, 32>), dim3(grid_for(n * 32)), dim3(WG), 0, st, n, rowptr, col, val, x, y,
                           r_minus, scoff);
}

template <typename T>
void launch_sub_symv_b(int64_t n_items, const int32_t* items, const int64_t* sub_off, const int64_t* tp_off,
                       const T* tiles, const T* rloc, const int64_t* scr_off, T* scr, int chl, hipStream_t st) {
    if (n_items <= 0) return;
    hipEvent_t e0, e1;
    if (take_launch_events(&e0, &e1))
        hipExtLaunchKernelGGL(k_sub_symv_b<T>, dim3((unsigned)n_items), dim3(WG), 0, st, e0, e1, 0, items, sub_off,
                              tp_off, tiles, rloc, scr_off, scr, chl);
    else
        hipLaunchKernelGGL(k_sub_symv_b<T>, dim3((unsigned)n_items), dim3(WG), 0, st, items, sub_off, tp_off, tiles,
                           rloc, scr_off, scr, chl);
}

template <typename T>
void launch_sub_finalize_b(int64_t r0, int64_t r1, const int32_t* pos_sub, const int64_t* sub_off,
                           const int64_t* scr_off, const T* scr, const int32_t* sub_dofs, T* x, bool accumulate,
                           int chl, int fl, hipStream_t st) {
    if (r1 <= r0) return;
    if (fl >= 32)
        hipLaunchKernelGGL((k_sub_finalize_b<T, 32>), dim3(grid_for(r1 - r0, WG / 32)), dim3(WG), 0, st, r0, r1,
                           pos_sub, sub_off, scr_off, scr, sub_dofs, x, accumulate ? 1 : 0, chl);
    else
        hipLaunchKernelGGL((k_sub_finalize_b<T, 8>), dim3(grid_for(r1 - r0, WG / 8)), dim3(WG), 0, st, r0, r1,
                           pos_sub, sub_off, scr_off, scr, sub_dofs, x, accumulate ? 1 : 0, chl);
}

// The same sums from the per-entry address table of the single-vector finalize
// (int4 per overlap entry: row-part address, column-part address + J * 64 + l, J,
// row-part chunks | tile rows << 16, in single-vector units; the block layout holds
// NB consecutive values at NB times that address): one table load replaces the
// entry's subdomain and offset lookups.  Same per-thread subsets, same order, same
// results as k_sub_finalize_b with accumulate.
template <typename T, int FL>
__global__ void __launch_bounds__(WG) k_sub_finalize_tab_b(int64_t r0, int64_t r1, const int4* tab, const T* scr,
                                                           const int32_t* sub_dofs, T* x) {
    constexpr int ND = WG / FL;
    __shared__ T s_y[FL][ND][NB];
    const int dl = tid() % ND, j = tid() / ND;
    const int64_t t = r0 + (int64_t)blockIdx.x * ND + dl;
    T y[NB];
#pragma unroll
    for (int q = 0; q < NB; ++q) y[q] = 0;
    if (t < r1) {
        const int4 e = tab[t];
        const T* part = scr + (int64_t)(uint32_t)e.x * NB;
        const T* colpart = scr + (int64_t)(uint32_t)e.y * NB;
        const int J = e.z, nch = e.w & 0xffff, nt = e.w >> 16;
        const int K = nch + (nt - 1 - J);
        for (int k = j; k < K; k += FL) {
            const int64_t I = J + 1 + (k - nch);
            const T* src = k < nch ? part + (int64_t)k * 64 * NB : colpart + I * (I - 1) / 2 * 64 * NB;
#pragma unroll
            for (int q = 0; q < NB; ++q) y[q] += src[q];
        }
    }
#pragma unroll
    for (int q = 0; q < NB; ++q) s_y[j][dl][q] = y[q];
    __syncthreads();
    if (j < NB && t < r1) {
        T v = s_y[0][dl][j];
        for (int q = 1; q < FL; ++q) v += s_y[q][dl][j];
        const int64_t d = sub_dofs[t];   // < 0: masked entry
        if (d >= 0) x[d * NB + j] = x[d * NB + j] + v;
    }
}

template <typename T>
void launch_sub_finalize_tab_b(int64_t r0, int64_t r1, const int32_t* tab, const T* scr, const int32_t* sub_dofs,
                               T* x, int fl, hipStream_t st) {
    if (r1 <= r0) return;
    const int4* tb = reinterpret_cast<const int4*>(tab);
    if (fl >= 32)
        hipLaunchKernelGGL((k_sub_finalize_tab_b<T, 32>), dim3(grid_for(r1 - r0, WG / 32)), dim3(WG), 0, st, r0, r1,
                           tb, scr, sub_dofs, x);
    else
        hipLaunchKernelGGL((k_sub_finalize_tab_b<T, 8>), dim3(grid_for(r1 - r0, WG / 8)), dim3(WG), 0, st, r0, r1,
                           tb, scr, sub_dofs, x);
}

template <typename T>
void launch_restrict_b(int64_t n_items, const int32_t* items, const int64_t* agg_ptr, const int32_t* agg_dofs,
                       const int64_t* zoff, const int32_t* k, const int64_t* coff, const T* Zc, const T* t, T* rc,
                       hipStream_t st) {
    if (n_items <= 0) return;
    hipLaunchKernelGGL(k_restrict_b<T>, dim3((unsigned)n_items), dim3(WG), 0, st, items, agg_ptr, agg_dofs, zoff, k,
                       coff, Zc, t, rc);
}

template <typename T>
void launch_prolong_b(int64_t n_items, const int32_t* items, const int64_t* agg_ptr, const int32_t* agg_dofs,
                      const int64_t* zoff, const int32_t* k, const int64_t* coff, const T* Zc, const T* ec, T* x,
                      hipStream_t st) {
    if (n_items <= 0) return;
    hipLaunchKernelGGL(k_prolong_b<T>, dim3((unsigned)n_items), dim3(WG), 0, st, items, agg_ptr, agg_dofs, zoff, k,
                       coff, Zc, ec, x);
}

void launch_scatter_sol(int64_t n, int32_t nr, const double* X, double* x, int64_t ldx, hipStream_t st) {
    hipLaunchKernelGGL(k_scatter_sol, dim3(grid_for(n * NB)), dim3(WG), 0, st, n, (int)nr, X, x, ldx);
}

static_assert(PCG_WG % NB == 0 && 64 % NB == 0, "a thread keeps its right-hand side from step to step");

namespace {

// f(std::integral_constant<int, NR>) for NR = 1 or NB
template <class F>
void with_nr(int nr, F&& f) {
    if (nr == NB) f(std::integral_constant<int, NB>{});
    else f(std::integral_constant<int, 1>{});
}

template <int NR, typename Z>
void seg_dot_parts(const SegTable& t, const double* a0, const Z* b0, const double* a1, const Z* b1, double* part0,
                   double* part1, hipStream_t st) {
    hipLaunchKernelGGL((k_seg_dot<NR, Z>), dim3((unsigned)t.n_blk), dim3(PCG_WG), 0, st, t.blk_lo, t.blk_hi, a0, b0, a1,
                       b1, part0, part1);
}

}  // namespace

namespace {

// Segments up to which k_pcg_init and k_pcg_check add the partials themselves.
constexpr int SEG_DIRECT = 64;

template <int NR>
void seg_totals(const SegTable& t, const double* p0, const double* p1, double* tot0, double* tot1, hipStream_t st) {
    hipLaunchKernelGGL(k_seg_totals<NR>, dim3((unsigned)((t.n_seg + PCG_WG / 64 - 1) / (PCG_WG / 64))), dim3(PCG_WG), 0,
                       st, t.n_seg, t.seg_blk, p0, p1, tot0, tot1);
}

}  // namespace

void launch_seg_dot(const SegTable& t, int nr, const double* a, const double* b, double* part, double* out,
                    double* host, hipStream_t st) {
    with_nr(nr, [&](auto c) {
        constexpr int NR = decltype(c)::value;
        seg_dot_parts<NR, double>(t, a, b, nullptr, nullptr, part, nullptr, st);
        hipLaunchKernelGGL(k_seg_sum<NR>, dim3((unsigned)t.n_seg), dim3(PCG_WG), 0, st, t.seg_blk, part, out, host);
    });
}

template <typename Z>
void launch_pcg_begin(const PcgArgs<Z>& a, int nrhs, const double* b, int64_t ldb, hipStream_t st) {
    with_nr(a.nr, [&](auto c) {
        constexpr int NR = decltype(c)::value;
        const SegTable& t = a.seg;
        hipLaunchKernelGGL((k_pcg_begin<NR, Z>), dim3((unsigned)t.n_blk), dim3(PCG_WG), 0, st, t.blk_lo, t.blk_hi, nrhs,
                           b, ldb, a.r, a.x, a.r32, a.z, a.part_rr, a.part_pq);
        double *tot = nullptr, *tot2 = nullptr;
        if (t.n_seg > SEG_DIRECT) {
            tot = a.tot;
            tot2 = tot + (size_t)t.n_seg * NR;
            seg_totals<NR>(t, a.part_rr, a.part_pq, tot, tot2, st);
        }
        hipLaunchKernelGGL(k_pcg_init<NR>, dim3(1), dim3(PCG_CHECK_WG), 0, st, t.n_seg, t.seg_blk, a.part_rr, a.part_pq,
                           tot, tot2, a.bb, a.act, a.iters, a.relres, a.st);
    });
}

template <typename Z>
void launch_pcg_step(const PcgArgs<Z>& a, double tol2, int32_t* host_st, hipStream_t st) {
    with_nr(a.nr, [&](auto c) {
        constexpr int NR = decltype(c)::value;
        const SegTable& t = a.seg;
        seg_dot_parts<NR, double>(t, a.p, a.q, nullptr, nullptr, a.part_pq, nullptr, st);
        hipLaunchKernelGGL((k_pcg_update_xr<NR, Z>), dim3((unsigned)t.n_blk), dim3(PCG_WG), 0, st, t.n_seg, t.blk_seg, t.blk_lo,
                           t.blk_hi, t.seg_blk, a.act, a.rz2, a.nsm, a.part_pq, a.p, a.q, a.x, a.r, a.rold, a.r32, a.z,
                           a.part_rr, a.st);
        double* tot = t.n_seg > SEG_DIRECT ? a.tot : nullptr;
        if (tot) seg_totals<NR>(t, a.part_rr, nullptr, tot, nullptr, st);
        hipLaunchKernelGGL(k_pcg_check<NR>, dim3(1), dim3(PCG_CHECK_WG), 0, st, t.n_seg, t.seg_blk, a.part_rr, tot, tol2,
                           a.bb, a.act, a.iters, a.relres, a.st, host_st);
    });
}

template <typename Z>
void launch_pcg_direction(const PcgArgs<Z>& a, bool first, hipStream_t st) {
    with_nr(a.nr, [&](auto c) {
        constexpr int NR = decltype(c)::value;
        const SegTable& t = a.seg;
        const bool flex = a.rold && !first;
        seg_dot_parts<NR, Z>(t, a.r, a.z, flex ? a.rold : nullptr, flex ? a.z : nullptr, a.part_pq, a.part_rr, st);
        hipLaunchKernelGGL((k_pcg_update_p<NR, Z>), dim3((unsigned)t.n_blk), dim3(PCG_WG), 0, st, t.n_seg, t.blk_seg, t.blk_lo,
                           t.blk_hi, t.seg_blk, a.act, a.rz2, a.nsm, a.part_pq, flex ? a.part_rr : nullptr, a.z, a.p,
                           a.st);
    });
}

#define LSDD_PCG_INST(Z)                                                                                     \
    template void launch_pcg_begin<Z>(const PcgArgs<Z>&, int, const double*, int64_t, hipStream_t);         \
    template void launch_pcg_step<Z>(const PcgArgs<Z>&, double, int32_t*, hipStream_t);                     \
    template void launch_pcg_direction<Z>(const PcgArgs<Z>&, bool, hipStream_t);
LSDD_PCG_INST(double)
LSDD_PCG_INST(float)

template <typename T, int NR>
void launch_small_sub(int64_t s0, int64_t n_sub, const int64_t* sub_off, const int32_t* sub_dofs,
                      const int64_t* pk_off, const T* pk, const T* rloc, T* x, int max_m, hipStream_t st,
                      bool fact) {
    if (n_sub <= 0) return;
    if (max_m < 1 || max_m > SMALL_M) throw std::runtime_error("launch_small_sub: max_m outside 1 .. SMALL_M");
    if (n_sub > INT32_MAX) throw std::runtime_error("launch_small_sub: more than 2^31 - 1 subdomains");
    const int max_x = NR == NB ? (max_m + 3) & ~3 : max_m;
    const size_t lds = ((size_t)max_m * (max_m + 1) / 2 + (fact ? 2 : 1) * (size_t)max_x * NR) * sizeof(T);
    // persistent waves: as many as fit on the device at once (LDS or registers bound)
    // FP32 blocks on the matrix cores; in FP64, where a step of theirs takes twice the time for
    // half the data, the row form is faster (3500 overlaps 24.3 against 26.4 us, 24 of them 8.6
    // against 9.7)
    if constexpr (NR == NB && sizeof(T) == 4)
        if (!fact && (uintptr_t)x % 16 == 0) {         // a caller's allocator may align to less
            hipLaunchKernelGGL(k_small_sub_mm, dim3((unsigned)n_sub), dim3(64), lds, st, (int32_t)s0, sub_off,
                               sub_dofs, pk_off, pk, rloc, x, max_m);
            return;
        }
    auto kern = fact ? &k_small_sub<T, NR, true> : &k_small_sub<T, NR, false>;
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(kern), 64, lds) !=
            hipSuccess ||
        per_cu < 1)
        per_cu = (int)std::max<size_t>(1, std::min<size_t>(8, (size_t)(160 * 1024) / lds));
    const unsigned grid = (unsigned)std::min<int64_t>(n_sub, (int64_t)per_cu * device_cu_count());
    hipLaunchKernelGGL(kern, dim3(grid), dim3(64), lds, st, (int32_t)s0, (int32_t)n_sub, sub_off, sub_dofs, pk_off,
                       pk, rloc, x, max_m);
}

template <typename T, int NR>
void launch_restrict_small(int64_t nc, const int32_t* agg_of_c, const int64_t* agg_ptr, const int32_t* agg_dofs,
                           const int64_t* zoff, const int64_t* coff, const T* Zc, const T* t, T* rc, hipStream_t st) {
    if (nc <= 0) return;
    if ((NR * sizeof(T)) % 16 == 0 && (((uintptr_t)t | (uintptr_t)rc) & 15) == 0)
        hipLaunchKernelGGL((k_restrict_small<T, NR, true>), dim3(grid_for(nc)), dim3(WG), 0, st, nc, agg_of_c,
                           agg_ptr, agg_dofs, zoff, coff, Zc, t, rc);
    else
        hipLaunchKernelGGL((k_restrict_small<T, NR, false>), dim3(grid_for(nc)), dim3(WG), 0, st, nc, agg_of_c,
                           agg_ptr, agg_dofs, zoff, coff, Zc, t, rc);
}

template <typename T, int NR>
void launch_prolong_small(int64_t na, const int32_t* agg_of_p, const int64_t* agg_ptr, const int32_t* agg_dofs,
                          const int64_t* zoff, const int32_t* k, const int64_t* coff, const T* Zc, const T* ec, T* x,
                          hipStream_t st) {
    if (na <= 0) return;
    if ((NR * sizeof(T)) % 16 == 0 && (((uintptr_t)ec | (uintptr_t)x) & 15) == 0)
        hipLaunchKernelGGL((k_prolong_small<T, NR, true>), dim3(grid_for(na)), dim3(WG), 0, st, na, agg_of_p,
                           agg_ptr, agg_dofs, zoff, k, coff, Zc, ec, x);
    else
        hipLaunchKernelGGL((k_prolong_small<T, NR, false>), dim3(grid_for(na)), dim3(WG), 0, st, na, agg_of_p,
                           agg_ptr, agg_dofs, zoff, k, coff, Zc, ec, x);
}

#define LSDD_SMALL_INST(T, NR)                                                                                     \
    template void launch_small_sub<T, NR>(int64_t, int64_t, const int64_t*, const int32_t*, const int64_t*,        \
                                          const T*, const T*, T*, int, hipStream_t, bool);                          \
    template void launch_restrict_small<T, NR>(int64_t, const int32_t*, const int64_t*, const int32_t*,            \
                                               const int64_t*, const int64_t*, const T*, const T*, T*, hipStream_t); \
    template void launch_prolong_small<T, NR>(int64_t, const int32_t*, const int64_t*, const int32_t*,             \
                                              const int64_t*, const int32_t*, const int64_t*, const T*, const T*,   \
                                              T*, hipStream_t);
LSDD_SMALL_INST(double, 1)
LSDD_SMALL_INST(double, NRB)
LSDD_SMALL_INST(float, 1)
LSDD_SMALL_INST(float, NRB)

#define LSDD_BLK_INST(T)                                                                                            \
    template void launch_sup_resid_blocks_b<T>(int64_t, const int32_t*, const int32_t*, const int64_t*,            \
                                               const int32_t*, const int64_t*, const T*, const T*, const T*, T*,     \
                                               bool, int, hipStream_t);                                              \
    template void launch_csr_resid_rows_b<T>(int64_t, const int32_t*, const int64_t*, const int32_t*, const T*,      \
                                             const T*, const T*, T*, bool, int, hipStream_t, const int64_t*);         \
    template void launch_csr_spmv_b<T>(int64_t, const int64_t*, const int32_t*, const T*, const T*, T*, const T*,    \
                                       int, hipStream_t, const int64_t*);                                             \
    template void launch_sub_symv_b<T>(int64_t, const int32_t*, const int64_t*, const int64_t*, const T*, const T*,  \
                                       const int64_t*, T*, int, hipStream_t);                                         \
    template void launch_sub_finalize_tab_b<T>(int64_t, int64_t, const int32_t*, const T*, const int32_t*, T*, int, \
                                               hipStream_t);                                                          \
    template void launch_sub_finalize_b<T>(int64_t, int64_t, const int32_t*, const int64_t*, const int64_t*,         \
                                           const T*, const int32_t*, T*, bool, int, int, hipStream_t);                \
    template void launch_restrict_b<T>(int64_t, const int32_t*, const int64_t*, const int32_t*, const int64_t*,      \
                                       const int32_t*, const int64_t*, const T*, const T*, T*, hipStream_t);          \
    template void launch_prolong_b<T>(int64_t, const int32_t*, const int64_t*, const int32_t*, const int64_t*,       \
                                      const int32_t*, const int64_t*, const T*, const T*, T*, hipStream_t);
LSDD_BLK_INST(double)
LSDD_BLK_INST(float)

}  // namespace lsdd
