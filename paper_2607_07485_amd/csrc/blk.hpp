// Launchers of the block (multi right-hand side) cycle kernels and of the
// segmented PCG kernels (implemented in blk.hip).  Block vectors hold NRB
// right-hand sides interleaved per DOF: entry (d, k) at d * NRB + k.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace lsdd {

constexpr int NRB = 8;   // right-hand sides per block

// ---------------------------------------------------------------- cycle, block vectors
// lanes per row of the CSR kernels: 4, 8 or 16 (lane = nonzero slot, all NRB
// right-hand sides per lane) or 32 or 64 (lane = (nonzero slot, right-hand side));
// residual rows of a supernode-blocked level by supernode row blocks (blk, rows, out
// as in launch_sup_resid_blocks; scol/scoff: the shared column lists), blocks of NRB
// right-hand sides, 4 / 8 / 16 lanes per row block
template <typename T>
void launch_sup_resid_blocks_b(int64_t nblk, const int32_t* blk, const int32_t* rows, const int64_t* rowptr,
                               const int32_t* scol, const int64_t* scoff, const T* val, const T* x, const T* r, T* out,
                               bool x_zero, int lanes, hipStream_t st);
// scoff != NULL: shared per-supernode column lists, as in launch_csr_resid_rows
template <typename T>
void launch_csr_resid_rows_b(int64_t nrows, const int32_t* rows, const int64_t* rowptr, const int32_t* col,
                             const T* val, const T* x, const T* r, T* out, bool x_zero, int lanes, hipStream_t st,
                             const int64_t* scoff = nullptr);
template <typename T>
void launch_csr_spmv_b(int64_t n, const int64_t* rowptr, const int32_t* col, const T* val, const T* x, T* y,
                       const T* r_minus, int lanes, hipStream_t st, const int64_t* scoff = nullptr);
template <typename T>
void launch_sub_symv_b(int64_t n_items, const int32_t* items, const int64_t* sub_off, const int64_t* tp_off,
                       const T* tiles, const T* rloc, const int64_t* scr_off, T* scr, int chl, hipStream_t st);
// the block finalize from the single-vector finalize's address table (int4 per entry);
// accumulates into x
template <typename T>
void launch_sub_finalize_tab_b(int64_t r0, int64_t r1, const int32_t* tab, const T* scr, const int32_t* sub_dofs,
                               T* x, int fl, hipStream_t st);
template <typename T>
void launch_sub_finalize_b(int64_t r0, int64_t r1, const int32_t* pos_sub, const int64_t* sub_off,
                           const int64_t* scr_off, const T* scr, const int32_t* sub_dofs, T* x, bool accumulate,
                           int chl, int fl, hipStream_t st);
template <typename T>
void launch_restrict_b(int64_t n_items, const int32_t* items, const int64_t* agg_ptr, const int32_t* agg_dofs,
                       const int64_t* zoff, const int32_t* k, const int64_t* coff, const T* Zc, const T* t, T* rc,
                       hipStream_t st);
template <typename T>
void launch_prolong_b(int64_t n_items, const int32_t* items, const int64_t* agg_ptr, const int32_t* agg_dofs,
                      const int64_t* zoff, const int32_t* k, const int64_t* coff, const T* Zc, const T* ec, T* x,
                      hipStream_t st);

// ---------------------------------------------------------------- small overlaps (NR = 1 or NRB)
constexpr int SMALL_M = 64;   // overlaps and aggregates up to this size use the kernels below

// x[Omega_s] += A_Omega_s^{-1} rloc[Omega_s] for the sweep-order subdomains s0 .. s0+n_sub-1
// (packed lower inverses at pk + pk_off[s]; rloc and x hold NR interleaved vectors);
// max_m (1 .. SMALL_M) bounds |Omega_s| over the launch and sizes its LDS.  fact: the
// packed triangles are lower-triangular factors X with A_Omega^{-1} = X^T X
template <typename T, int NR>
void launch_small_sub(int64_t s0, int64_t n_sub, const int64_t* sub_off, const int32_t* sub_dofs,
                      const int64_t* pk_off, const T* pk, const T* rloc, T* x, int max_m, hipStream_t st,
                      bool fact = false);
// rc[c] = Z_i[:, c - coff_i]^T t[omega_i] for every coarse DOF c of an aggregate i
// with agg_of_c[c] = i (agg_of_c[c] < 0: skipped)
template <typename T, int NR>
void launch_restrict_small(int64_t nc, const int32_t* agg_of_c, const int64_t* agg_ptr, const int32_t* agg_dofs,
                           const int64_t* zoff, const int64_t* coff, const T* Zc, const T* t, T* rc, hipStream_t st);
// x[agg_dofs[p]] += Z_i[p - agg_ptr_i, :] ec[coff_i ..] for aggregate entries p with agg_of_p[p] = i
template <typename T, int NR>
void launch_prolong_small(int64_t na, const int32_t* agg_of_p, const int64_t* agg_ptr, const int32_t* agg_dofs,
                          const int64_t* zoff, const int32_t* k, const int64_t* coff, const T* Zc, const T* ec, T* x,
                          hipStream_t st);

// x[k * ldx + d] = X[d * NRB + k] (d < n, k < nr)
void launch_scatter_sol(int64_t n, int32_t nr, const double* X, double* x, int64_t ldx, hipStream_t st);

// ---------------------------------------------------------------- segmented PCG
// A "segment" is a contiguous DOF range of the level-0 vector (one problem
// instance); every (segment, right-hand side) pair i = seg * NR + k runs its own
// CG recurrence.  Reductions use a fixed block table (segment, DOF range) and
// add the block partials in block order, so every scalar is reproducible.
struct SegTable {
    int32_t n_seg = 0;
    int32_t n_blk = 0;
    const int32_t* blk_seg = nullptr;   // [n_blk]
    const int64_t* blk_lo = nullptr;    // [n_blk] first DOF
    const int64_t* blk_hi = nullptr;    // [n_blk] one past the last DOF
    const int32_t* seg_blk = nullptr;   // [n_seg + 1] blocks of segment s
};

// Status words of a solve: active pairs, iterations, breakdown cause bits (1 p^T A p <= 0,
// 2 p^T A p or r^T z not finite, 4 residual not finite, 8 beta not finite), 1 when the
// right-hand side holds a NaN or an infinity.
enum { PCG_ST_COUNT = 0, PCG_ST_IT = 1, PCG_ST_FLAG = 2, PCG_ST_BAD = 3, PCG_ST_WORDS = 4 };

// Vectors and scalars of a solve (blocks of nr = 1 or NRB vectors).  Z: type of the
// cycle's output (float: an FP32 cycle, whose input r32 the kernels fill from r).
template <typename Z>
struct PcgArgs {
    SegTable seg;
    int nr;
    double *x, *r, *p, *q;
    double* rold;                 // residual before the step (flexible beta), or NULL
    float* r32;                   // FP32 residual for the cycle, or NULL
    Z* z;                         // cycle output; zeroed where the residual is formed
    int nsm;                      // stride of the per-pair arrays
    double *bb, *rz2, *relres;    // rz2: two slots of nsm
    int32_t *act, *iters, *st;
    double *part_pq, *part_rr;    // n_blk * nr partials each
    double* tot;                  // 2 * n_seg * nr sums (tables of many segments)
};

// out[i] = <a, b>_i (and, for the first segment, host[k]); part holds n_blk * nr doubles
void launch_seg_dot(const SegTable& t, int nr, const double* a, const double* b, double* part, double* out,
                    double* host, hipStream_t st);
// r = b, x = 0, z = 0 and the state of the recurrences (nrhs <= nr right-hand sides at
// stride ldb, the others zero)
template <typename Z>
void launch_pcg_begin(const PcgArgs<Z>& a, int nrhs, const double* b, int64_t ldb, hipStream_t st);
// with q = A p: the step along p on the active pairs; pairs with <r, r> <= tol2 <b, b>
// leave the iteration; z = 0; the status words go to a.st and host_st
template <typename Z>
void launch_pcg_step(const PcgArgs<Z>& a, double tol2, int32_t* host_st, hipStream_t st);
// with z = cycle(r): the next direction (first: p = z)
template <typename Z>
void launch_pcg_direction(const PcgArgs<Z>& a, bool first, hipStream_t st);

}  // namespace lsdd
