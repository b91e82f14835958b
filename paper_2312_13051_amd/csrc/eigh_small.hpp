// Small-order eigensolver (eigh_small.hip): the whole solve in FP64 or, up to
// order 16, on the mixed paths, or their tridiagonal part, in one launch.
#pragma once

#include "common.hpp"

namespace be {

// Largest order of these kernels: a matrix's arrays take ~45 KB of LDS (three
// matrices resident per compute unit) and its rows half a wave.
constexpr int kSmallOrder = 32;

// As eigh_fp64, without workspace.
int eigh_small_fp64(be_ctx *ctx, double2 *H, int N, int ld, int64_t ms, int64_t n_mat, int lo, int hi, double *evals,
                    double2 *U, int ldu, int64_t us, uint32_t *status, hipStream_t stream, double clu_rel);

// The mixed path for orders up to kSmallMixed, from H to U in one launch, with
// the general path's bits. The line lies where a row per lane still leaves four
// matrices to a wave; general path -> this one, half the bands, order 4, 52,500
// matrices: 460 -> 123 us; 8, 4,096: 161 -> 97; 12: 233 -> 130; 16: 334 -> 334
// (56 KB of LDS per wave), 16, 64: 227 -> 166.
constexpr int kSmallMixed = 16;
int eigh_small_c64(be_ctx *ctx, float2 *H, int N, int ld, int64_t ms, int64_t n_mat, int lo, int hi, double *evals,
                   double2 *U, int ldu, int64_t us, uint32_t *status, hipStream_t stream, double clu_rel);

// Eigenvalues and eigenvectors Z (written as c64, N x m) of n_mat real
// symmetric tridiagonal matrices d, e (N values per matrix each).
int tri_small_c64(be_ctx *ctx, const double *d, const double *e, int N, int64_t n_mat, int lo, int hi, double *evals,
                  float2 *Z, int ldz, int64_t sz, uint32_t *status, hipStream_t stream, double clu_rel, double tol_orth);

}  // namespace be
