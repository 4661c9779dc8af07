// Launchers of the fused single-vector cycle kernels (fuse.hip): one launch per colour,
// per restriction, per prolongation and per coarsest solve, for levels whose cycle is a
// chain of short launches rather than a stream of matrix entries.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace lsdd {

// Largest overlap of the fused colour kernel: its workgroup keeps the column sums of its
// 16 waves in LDS (16 x 640 doubles = 80 KB of the 160 KB of a CU).
constexpr int FUSE_M = 640;

// a subdomain of a sweep: its size and where its inverse starts (packed triangles for
// |Omega| <= SMALL_M, else 64 x 64 tiles)
struct SubItem {
    int32_t m, pad;
    int64_t off;
};

// 16 rows of a subdomain's unpacked inverse: its first entry in the sweep list, its size,
// the first of the rows, where its inverse starts
struct RowItem {
    int32_t o, m, row0, pad;
    int64_t off;
};

// an aggregate: its size, its coarse DOFs, its block of Z (column-major)
struct AggItem {
    int32_t nw, c0, k, pad;
    int64_t zoff;
};

// Row tables of n_sub DOF lists (list s at dofs[off[s]] .. dofs[off[s + 1]]), pad entries
// each: {DOF, first value, entries, first column index}, {-1, 0, 0, 0} past the list's end;
// scoff != NULL: shared column lists (the column index counts into the lists)
void launch_row_table(int64_t n_sub, const int64_t* off, const int32_t* dofs, const int64_t* rowptr,
                      const int64_t* scoff, int pad, int4* tab, hipStream_t st);

// x[Omega] += A_Omega^{-1} (r - A x)[Omega] for n_sub subdomains no two of which share an
// element (x is read and written in one launch); rows: their row tables (pad a multiple of 64,
// <= FUSE_M), row_len: average entries per row of A; x_zero: x is zero
template <typename T>
void launch_colour_step(int64_t n_sub, const SubItem* items, const int4* rows, const int32_t* col, const T* val,
                        const T* pk, const T* tiles, const T* r, T* x, bool x_zero, int pad, int row_len,
                        hipStream_t st);
// Row-major inverses full[full_off[s] ..) of n_sub subdomains of up to max_sub DOFs from the
// packed ones: triangles at pk_off[s] for |Omega| <= SMALL_M, else 64 x 64 tiles at tp_off[s]
template <typename T>
void launch_unpack(int64_t n_sub, int max_sub, const int64_t* sub_off, const int64_t* tp_off, const int64_t* pk_off,
                   const T* tiles, const T* pk, const int64_t* full_off, T* full, hipStream_t st);
// x[Omega] += A_Omega^{-1} rloc[Omega] (inverses unpacked, row-major)
template <typename T>
void launch_sub_rows(int64_t n_items, const RowItem* items, const T* inv, const T* rloc, const int32_t* dofs, T* x,
                     hipStream_t st);
// rc = Z^T (r - A x) and xc = 0 on the coarse DOFs of n_agg aggregates; rows: their row tables
template <typename T>
void launch_resid_restrict(int64_t n_agg, const AggItem* items, const int4* rows, const int32_t* col, const T* val,
                           const T* Zc, const T* r, const T* x, T* rc, T* xc, int pad, int row_len, hipStream_t st);
// x[omega] += Z ec; max_k: the most modes of an aggregate
template <typename T>
void launch_prolong_agg(int64_t n_agg, const AggItem* items, const int4* rows, const T* Zc, const T* ec, T* x, int pad,
                        int max_k, hipStream_t st);
// x = inv r for a dense symmetric n x n inverse in FP64 (products and sums in FP64)
template <typename T>
void launch_dense_apply(int64_t n, const double* inv, const T* r, T* x, hipStream_t st);

}  // namespace lsdd
