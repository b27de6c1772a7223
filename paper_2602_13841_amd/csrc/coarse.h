// Coarsest-level direct solver (internal).
#pragma once

#include <hip/hip_runtime.h>

namespace stmg {

// in-place inverse of the m x m FP64 matrix A (row stride ld, a multiple of
// 32) with partial pivoting
struct DenseInverse {
    double *A;      // m x ld
    int m, ld;
    double *W;      // [m rounded up to 32][32]
    double *B;      // [32][ld] (before the interchanges: the panel's multipliers)
    double *Pt;     // [32][ld] the next panel, transposed
    double *dinv;   // [32][32] inverse of the pivot block
    int *rowsrc;    // [m]
    int *perm;      // [m] row of the right-hand side behind each column of the inverse
};
// largest system the inverse takes (its panels keep the candidate rows in
// the registers of one workgroup); larger ones are LU factored
constexpr int DINV_MAX_M = 6144;
constexpr int dinv_ld(int m) { return (m + 31) & ~31; }
// coarse matrix (with nb border rows and columns) from the columns J e_i
// (to w.A, its first panel to w.Pt), then its inverse in place
hipError_t launch_inv_matrix(const double *Y, int n, int nb, long long pbase, long long Np1, int npm,
                             const DenseInverse &w, hipStream_t s);
hipError_t launch_dense_inverse(const DenseInverse &w, hipStream_t s);
// d = first n entries of the solution for the right-hand side (r, 0)
template <typename T>
hipError_t launch_inverse_apply(const DenseInverse &w, const T *r, T *d, int n, hipStream_t s);

} // namespace stmg
