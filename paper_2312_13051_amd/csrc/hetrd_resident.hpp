// On-chip Householder reduction (hetrd_resident.hip).
#pragma once

#include "common.hpp"

namespace be {

// Largest order the kernel reduces: 192 rows and columns in registers and up
// to 24 further columns in LDS (131 KB with the vectors and partial sums).
constexpr int kResidentOrder = 216;

// Reduces the trailing matrices H(p0:N, p0:N) of order N - p0 <= kResidentOrder
// (FP64, lower triangle read) to tridiagonal form: d, e from index p0 on, the
// reflectors in H's columns (zeros above) and tau (N per matrix).
int hetrd_resident(be_ctx *ctx, double2 *H, int64_t ms, int ld, int N, int p0, int64_t n_mat, double *d, double *e,
                   int64_t sDE, double2 *tau, hipStream_t stream);

// Compact-WY factors (nb x nb, nb = 32) of the panels p_first .. of reflectors held in
// H's columns: T of panel p at Tm + q*sT + p*nb*nb.
int larft(be_ctx *ctx, const double2 *H, int64_t ms, int ld, int N, int p_first, int64_t n_mat, const double2 *tau,
          double2 *Tm, int64_t sT, hipStream_t stream);

// Matrices of order n resident on the device at once.
int64_t resident_slots(be_ctx *ctx, int n);

}  // namespace be
