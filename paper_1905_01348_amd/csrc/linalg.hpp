// FP64 complex dense linear algebra used by the ACE build and apply.
#pragma once

#include "common.hpp"

namespace fx {

// What a product may leave out: output tiles strictly above the diagonal of a
// Hermitian C (the strict upper part is then undefined), and the zeros of a
// triangular operand (A or B lower).  With
// mlim > 0, product b of the batch has min(M, mlim - b * mstep) rows (and, with
// A lower, as many k).
constexpr int kZgHermitian = 1, kZgALower = 2, kZgBLower = 4;
struct ZgShape {
  int flags = 0, mlim = 0, mstep = 0;
};

// With psi set, C = psi - half + i hdt (h - op(A) op(B)) instead (alpha and beta
// unused, nsplit 1): the residual of the PT-CN step formed where its last
// product ends.  Columns at psi + c*ldp, and so on.
struct ZgResidual {
  const cpx<double>*psi = nullptr, *half = nullptr, *h = nullptr;
  int64_t ldp = 0, ldf = 0, ldh = 0;
  double hdt = 0.0;
};

// C = alpha op(A) op(B) + beta C (complex double, column-major), op 0 = N,
// 1 = conjugate transpose; `batch` independent products with element strides
// sA, sB, sC.  nsplit_hint > 0 fixes the number of K splits (1 = none);
// 0 chooses one.  Split partial sums are reduced in FP64 in a fixed order.
fx_status zgemm(fx_ctx* ctx, Workspace* ws, hipStream_t st, int opa, int opb, int M, int N, int K, cpx<double> alpha,
                const void* A, int64_t lda, const void* B, int64_t ldb, cpx<double> beta, void* C, int64_t ldc,
                int batch, int64_t sA, int64_t sB, int64_t sC, int nsplit_hint, ZgShape shape = {},
                ZgResidual res = {});

// In-place blocked Cholesky A = L L^H (lower; reads the lower part only, the
// strict upper part is zeroed).  dinv (kCholBlock values per column, n rounded
// up to a whole block) receives the inverses of L's diagonal blocks for
// ztrinv.  *info_dev (device int, must start at 0) receives 1 + the first
// column whose pivot was not positive, or stays 0.
constexpr int kCholBlock = 64;
// Workspaces of zpotrf (*dinv) and ztrinv; got before a split product, whose
// partial sums take what memory is left.
fx_status chol_workspace(fx_ctx* ctx, Workspace* ws, int n, void** dinv);
fx_status zpotrf(fx_ctx* ctx, Workspace* ws, hipStream_t st, int n, void* A, int64_t lda, void* dinv, int* info_dev);

// In-place inverse of the lower triangular n x n factor of zpotrf.
fx_status ztrinv(fx_ctx* ctx, Workspace* ws, hipStream_t st, int n, void* A, int64_t lda, const void* dinv);

// H = (M + M^H)/2 (n x n, ld n), Aneg = -H, *ex_dev = 1/2 Re tr H (nullable).
fx_status zherm(hipStream_t st, int n, const void* M, int64_t ldm, void* H, void* Aneg, double* ex_dev);

// X <- X Linv^H in place: X is M x n (ldx), Linv lower triangular n x n.
fx_status zmul_upper_inplace(fx_ctx* ctx, hipStream_t st, int M, int n, void* X, int64_t ldx, const void* Linv,
                             int64_t ldl);

}  // namespace fx
