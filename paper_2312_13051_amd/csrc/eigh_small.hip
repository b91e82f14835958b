// Batched Hermitian eigensolver for small orders: one launch, several
// matrices per wave, everything in LDS.
//
// A group of TPM lanes (8, 16 or 64) takes a matrix through the steps of the
// general solver (Householder reduction, bisection, inverse iteration,
// orthonormalization inside clusters, Newton-Schulz orthonormalization of
// all vectors, back-transformation) without leaving LDS. Only lanes of one
// wave cooperate, so there are no workgroup barriers. The general path gives
// such a matrix four workgroups of 256 threads one after another, a padded
// 16 x 16 tile in each of five MFMA products and ~12 launches with a
// read-back. Bound by the latency of the serial recurrences (Sturm counts, one
// lane per eigenvalue, and the columns of the reduction), hence as many matrices
// per wave as have rows for its lanes. FP64, half the bands, general path ->
// this one: order 4, 10,000 matrices 945 -> 50 us; 16, 4,096: 1,416 -> 126; 32,
// 12, all bands: 613 -> 255; 8,192: 6,547 -> 1,566. The Sturm counts read T from
// registers (from LDS: 62, 158, 287 and 1,833 us).
// Mixed path up to order 16, likewise: order 4, 52,500 matrices (a quarter of
// the nested loops of 21 planes) 460 -> 123 us, of which the panel kernel took
// 252 (a wave per matrix), three 16 x 16 products 87 and the copy to FP64 24;
// 210,000: 360 -> 298 with the counts from registers.
// Tridiagonal part alone, for orders 17 to 32 on the mixed path (reduction by
// the panel kernel, FP32 products for the back-transformation): 32, 4,096:
// 810 -> 260 us.
#include <algorithm>

#include "common.hpp"
#include "eigh_small.hpp"
#include "lanes.hpp"
#include "tridiag.hpp"

namespace {

__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Sum and maximum over the TPM lanes of a matrix
template <int TPM>
__device__ __forceinline__ double grp_sum(double v) {
  if constexpr (TPM > 16) {
    v = fold<32>(v, v);
    v = fold<16>(v, v);
  }
  if constexpr (TPM > 8) v += lane_xor<8>(v);
  v += lane_xor<4>(v);
  v += lane_xor<2>(v);
  v += lane_xor<1>(v);
  return v;
}
template <int TPM>
__device__ __forceinline__ double grp_max(double v) {
  if constexpr (TPM > 16) v = fold_max<16>(fold_max<32>(v));
  if constexpr (TPM > 8) v = fmax(v, lane_xor<8>(v));
  v = fmax(v, lane_xor<4>(v));
  v = fmax(v, lane_xor<2>(v));
  v = fmax(v, lane_xor<1>(v));
  return v;
}

// What a launch takes in and gives out
enum SmallMode {
  kFull,     // FP64: H -> U
  kFullC64,  // FP32 reduction and back-transformation: c64 H -> U (c128)
  kTri       // d, e -> Z (c64)
};

// LDS of one matrix, in doubles: d, e, e^2 (N each), eigenvalues (m + 4),
// block starts, group ids and marks (N + 1 + 2 m ints), X (N m), scratch for the
// elimination's diagonals and the Gram matrix or, later, U (2 (N + 1) m), and
// with kFull the matrix, v, w and tau (N N + 3 N complex), with kFullC64 the
// matrix, W and T (N N each) and four vectors in c64.
__host__ __device__ inline int small_doubles(int N, int m, SmallMode mode) {
  const int d = 3 * N + (m + 4) + (2 * m + N + 2) / 2 + N * m + 2 * (N + 1) * m;
  const int c = mode == kFull ? 2 * (N * N + 3 * N) : mode == kFullC64 ? 3 * N * N + 4 * N : 0;
  return (d + 1 + c) & ~1;  // even: the complex part is 16-byte aligned
}

// Sum over the TPM lanes of a matrix, in the order in which wave_sum adds the
// lanes of a wave whose others hold zeros
template <int TPM>
__device__ __forceinline__ float grp_sum_f(float v) {
  if constexpr (TPM > 8) v += lane_xor<8>(v);
  v += lane_xor<4>(v);
  v += lane_xor<2>(v);
  v += lane_xor<1>(v);
  return v;
}

// Householder reduction of a c64 matrix A (N x N, in LDS, lower triangle; its
// columns become the reflectors) of order N <= TPM with the panel kernel's
// arithmetic: that kernel's steps with its lanes' rows, products and sums in
// the same order, so that a matrix's T and reflectors have the same bits. W:
// N x N, T: N x N with zeros on entry, the compact-WY factor on return; sv,
// sy, st2: N each.
template <int TPM>
__device__ __forceinline__ void reduce_c64(float2 *A, float2 *W, float2 *T, float2 *sv, float2 *sy, float2 *st2,
                                           double *sd, double *se, int N, int t) {
  for (int j = 0; j < N; ++j) {
    {  // the last reflector's share of column j
      const int r = j + t;
      if (r < N) {
        const float2 a = A[r + j * N];
        float ar = a.x, ai = a.y;
        if (j > 0) {
          const float2 vr = sv[r], wr = sy[r], wj = sy[j], vj = sv[j];
          ar -= vr.x * wj.x + vr.y * wj.y + wr.x * vj.x + wr.y * vj.y;
          ai -= vr.y * wj.x - vr.x * wj.y + wr.y * vj.x - wr.x * vj.y;
        }
        if (r == j) {
          ai = 0;
          sd[j] = double(ar);
        }
        A[r + j * N] = make_float2(ar, ai);
      }
    }
    wave_lds_sync();
    if (j == N - 1) {
      if (t < N) A[t + j * N] = make_float2(0.f, 0.f);
      if (t == 0) se[j] = 0.0;
      wave_lds_sync();
      break;
    }
    float xn = 0;
    if (j + 2 + t < N) {
      const float2 a = A[j + 2 + t + j * N];
      xn += a.x * a.x + a.y * a.y;
    }
    xn = grp_sum_f<TPM>(xn);
    const float2 alpha = A[j + 1 + j * N];
    float2 tau = make_float2(0.f, 0.f), scal = tau;
    float beta = alpha.x;
    if (!(xn == 0.f && alpha.y == 0.f)) {
      const float nrm = sqrt(alpha.x * alpha.x + alpha.y * alpha.y + xn);
      beta = alpha.x >= 0.f ? -nrm : nrm;
      tau = make_float2((beta - alpha.x) / beta, -alpha.y / beta);
      const float dr = alpha.x - beta, di = alpha.y;
      const float den = dr * dr + di * di;
      scal = make_float2(dr / den, -di / den);
    }
    if (t == 0) se[j] = double(beta);
    float2 v = make_float2(0.f, 0.f);
    if (t == j + 1) {
      v = make_float2(1.f, 0.f);
    } else if (t > j && t < N) {
      const float2 a = A[t + j * N];
      v = make_float2(a.x * scal.x - a.y * scal.y, a.x * scal.y + a.y * scal.x);
    }
    wave_lds_sync();
    if (t < N) {
      sv[t] = v;
      A[t + j * N] = v;
    }
    wave_lds_sync();
    // y = A v: a lane's row, plus its column of the rows below
    const int r0 = j + 1, r = r0 + t;
    const bool rok = r < N;
    const float2 vr = rok ? sv[r] : make_float2(0.f, 0.f);
    float yr = 0, yi = 0;
    float2 col = make_float2(0.f, 0.f);
    for (int c = r0; c < N; ++c) {
      const float2 a = (rok && r >= c) ? A[r + c * N] : make_float2(0.f, 0.f);
      const float2 vc = sv[c];
      const bool dg = r == c;
      const float ax = a.x, ay = dg ? 0.f : a.y;
      yr += ax * vc.x - ay * vc.y;
      yi += ax * vc.y + ay * vc.x;
      float2 p = dg ? make_float2(0.f, 0.f) : make_float2(ax * vr.x + ay * vr.y, ax * vr.y - ay * vr.x);
      p.x = grp_sum_f<TPM>(p.x);
      p.y = grp_sum_f<TPM>(p.y);
      if (dg) col = p;
    }
    yr += col.x;
    yi += col.y;
    // y -= V W^H v + W V^H v; the earlier reflectors' share of column j + 1
    float pr = 0, pi = 0;
    for (int c = 0; c < j; ++c) {
      const float2 w = rok ? W[r + c * N] : make_float2(0.f, 0.f), vv = rok ? A[r + c * N] : make_float2(0.f, 0.f);
      float2 a, b;
      a.x = fmaf(w.x, vr.x, w.y * vr.y);
      a.y = fmaf(w.x, vr.y, -(w.y * vr.x));
      b.x = fmaf(vv.x, vr.x, vv.y * vr.y);
      b.y = fmaf(vv.x, vr.y, -(vv.y * vr.x));
      a.x = grp_sum_f<TPM>(a.x);
      a.y = grp_sum_f<TPM>(a.y);
      b.x = grp_sum_f<TPM>(b.x);
      b.y = grp_sum_f<TPM>(b.y);
      if (t == 0) st2[c] = b;
      yr -= vv.x * a.x - vv.y * a.y + w.x * b.x - w.y * b.y;
      yi -= vv.x * a.y + vv.y * a.x + w.x * b.y + w.y * b.x;
      const float2 wj = W[j + 1 + c * N], vj = A[j + 1 + c * N];
      pr += vv.x * wj.x + vv.y * wj.y + w.x * vj.x + w.y * vj.y;
      pi += vv.y * wj.x - vv.x * wj.y + w.y * vj.x - w.x * vj.y;
    }
    const float2 y = make_float2(tau.x * yr - tau.y * yi, tau.x * yi + tau.y * yr);
    wave_lds_sync();
    if (rok && j > 0) {
      const float2 a0 = A[r + (j + 1) * N];
      A[r + (j + 1) * N] = make_float2(a0.x - pr, a0.y - pi);
    }
    if (t < j) {
      float xr = 0, xi = 0;
      for (int c = t; c < j; ++c) {
        const float2 tt = T[t + c * N], b = st2[c];
        xr += tt.x * b.x - tt.y * b.y;
        xi += tt.x * b.y + tt.y * b.x;
      }
      T[t + j * N] = make_float2(-(tau.x * xr - tau.y * xi), -(tau.x * xi + tau.y * xr));
    }
    if (t == 0) T[j + j * N] = tau;
    float dr = 0, di = 0;
    if (rok) {
      dr += y.x * vr.x + y.y * vr.y;
      di += y.x * vr.y - y.y * vr.x;
    }
    dr = grp_sum_f<TPM>(dr);
    di = grp_sum_f<TPM>(di);
    const float alr = -0.5f * (tau.x * dr - tau.y * di), ali = -0.5f * (tau.x * di + tau.y * dr);
    if (t < r0 && t < N) W[t + j * N] = make_float2(0.f, 0.f);
    if (rok) {
      const float2 w = make_float2(y.x + alr * vr.x - ali * vr.y, y.y + alr * vr.y + ali * vr.x);
      W[r + j * N] = w;
      sy[r] = w;
    }
    wave_lds_sync();
  }
}

// Entry (i, c) of a c64 product A B (A conjugated with CONJ) over k = 0 .. K-1,
// A(i, k) = a[k sa], B(k, c) = b[k]: three real products per complex one, each a
// chain of fused multiply-adds in the order of k, as the matrix cores of the
// general path's products add them.
template <bool CONJ>
__device__ __forceinline__ float2 product_c64(const float2 *a, int sa, const float2 *b, int K) {
  float rr = 0.f, ii = 0.f, x = 0.f;
  for (int k = 0; k < K; ++k) {
    const float2 u = a[k * sa], w = b[k];
    const float ai = CONJ ? -u.y : u.y;
    rr = fmaf(u.x, w.x, rr);
    ii = fmaf(ai, w.y, ii);
    x = fmaf(u.x + ai, w.x + w.y, x);
  }
  return make_float2(rr - ii, x - rr - ii);
}

// TPM lanes per matrix of order N <= NM
template <int TPM, int NM, SmallMode MODE, typename IN, typename OUT>
__global__ __launch_bounds__(64) void eigh_small_kernel(IN *H, int64_t sH, int ld, const double *dg,
                                                        const double *eg, int64_t sDE, int N, int lo, int m,
                                                        int64_t n_mat, double clu_rel, double tol_orth, int max_it,
                                                        double *evals, OUT *U, int ldu, int64_t sU, uint32_t *status) {
  extern __shared__ double2 sm2[];
  constexpr int MPB = 64 / TPM;
  constexpr bool FULL = MODE == kFull;
  const int lane = threadIdx.x, t = lane % TPM;
  const int64_t q = int64_t(blockIdx.x) * MPB + lane / TPM;
  const bool live = q < n_mat;
  const int per = small_doubles(N, m, MODE);
  double *base = reinterpret_cast<double *>(sm2) + (lane / TPM) * per;
  double2 *A = reinterpret_cast<double2 *>(base);  // kFull: N x N, then v, w, tau (N each)
  double2 *sv = A + (FULL ? N * N : 0), *sw = sv + (FULL ? N : 0), *stau = sw + (FULL ? N : 0);
  float2 *Af = reinterpret_cast<float2 *>(base), *Wf = Af + N * N, *Tf = Wf + N * N;  // kFullC64
  double *sd = FULL ? reinterpret_cast<double *>(stau + N)
                    : reinterpret_cast<double *>(MODE == kFullC64 ? Tf + N * N + 4 * N : Af), *se = sd + N, *se2 = se + N, *slam = se2 + N;
  double *X0 = slam + m + 4, *ZG = X0 + N * m;
  int *sblk = reinterpret_cast<int *>(ZG + 2 * (N + 1) * m), *smark = sblk + N + 1, *sbad = smark + m;
  const double eps = DBL_EPSILON;
  uint32_t st = 0;

  // ---- Householder reduction (the panel kernel's reflectors), unblocked
  if constexpr (FULL) {
    constexpr int RW = TPM < 32 ? TPM : 32, KS = TPM / RW;  // rows at once, column strides per row
    const int i0 = t % RW, k0 = t / RW;
    double2 *Hq = H + (live ? q : 0) * sH;
    for (int e = t; e < N * N; e += TPM) {
      const int r = e % N, c = e / N;
      double2 v = r >= c ? Hq[r + int64_t(c) * ld] : be::cconj(Hq[c + int64_t(r) * ld]);
      if (r == c) v.y = 0.0;
      A[e] = v;
    }
    wave_lds_sync();
    for (int j = 0; j + 1 < N; ++j) {
      double xn = 0.0;
      for (int r = j + 2 + t; r < N; r += TPM) {
        const double2 a = A[r + j * N];
        xn += a.x * a.x + a.y * a.y;
      }
      xn = grp_sum<TPM>(xn);
      const double2 alpha = A[j + 1 + j * N];
      double2 tau = make_double2(0.0, 0.0), scal = tau;
      double beta = alpha.x;
      if (xn != 0.0 || alpha.y != 0.0) {
        const double nrm = sqrt(alpha.x * alpha.x + alpha.y * alpha.y + xn);
        beta = alpha.x >= 0.0 ? -nrm : nrm;
        tau = make_double2((beta - alpha.x) / beta, -alpha.y / beta);
        const double dr = alpha.x - beta, di = alpha.y, den = dr * dr + di * di;
        scal = make_double2(dr / den, -di / den);
      }
      for (int r = j + 1 + t; r < N; r += TPM) sv[r] = r == j + 1 ? make_double2(1.0, 0.0) : be::cmul(A[r + j * N], scal);
      if (t == 0) {
        sd[j] = A[j + j * N].x;
        se[j] = beta;
        stau[j] = tau;
      }
      wave_lds_sync();
      // w = tau A v, then w -= tau (w^H v) / 2 v
      double dr = 0.0, di = 0.0;
      double2 w = make_double2(0.0, 0.0);
      const int i = i0;  // N <= RW: one row per lane
      if (i > j && i < N)
        for (int k = j + 1 + k0; k < N; k += KS) w = be::cadd(w, be::cmul(A[i + k * N], sv[k]));
      if (KS == 2) {
        w.x += __shfl_xor(w.x, 32, 64);
        w.y += __shfl_xor(w.y, 32, 64);
      }
      w = be::cmul(tau, w);
      const double2 vi = (i > j && i < N) ? sv[i] : make_double2(0.0, 0.0);
      if (k0 == 0) {
        dr = w.x * vi.x + w.y * vi.y;
        di = w.x * vi.y - w.y * vi.x;
      }
      dr = grp_sum<TPM>(dr);
      di = grp_sum<TPM>(di);
      const double2 al = make_double2(-0.5 * (tau.x * dr - tau.y * di), -0.5 * (tau.x * di + tau.y * dr));
      w = be::cadd(w, be::cmul(al, vi));
      if (k0 == 0 && i > j && i < N) sw[i] = w;
      wave_lds_sync();
      // A -= v w^H + w v^H; column j keeps v
      if (i > j && i < N) {
        for (int k = j + 1 + k0; k < N; k += KS) {
          const double2 u = be::cadd(be::cmulc(sw[k], vi), be::cmulc(sv[k], w));
          A[i + k * N] = be::csub(A[i + k * N], u);
        }
        if (k0 == 0) A[i + j * N] = vi;
      }
      wave_lds_sync();
    }
    if (t == 0) {
      sd[N - 1] = A[N * N - 1].x;
      se[N - 1] = 0.0;
    }
    if (live)  // H's columns hold the reflectors, as the panel kernel leaves them
      for (int e = t; e < N * N; e += TPM) {
        const int r = e % N, c = e / N;
        Hq[r + int64_t(c) * ld] = r > c ? A[e] : make_double2(0.0, 0.0);
      }
  } else if constexpr (MODE == kFullC64) {
    float2 *Hq = H + (live ? q : 0) * sH, *vec = Tf + N * N;
    for (int e = t; e < N * N; e += TPM) {
      const int r = e % N, c = e / N;
      Af[e] = r >= c ? Hq[r + int64_t(c) * ld] : make_float2(0.f, 0.f);
      Tf[e] = make_float2(0.f, 0.f);
    }
    wave_lds_sync();
    reduce_c64<TPM>(Af, Wf, Tf, vec, vec + N, vec + 2 * N, sd, se, N, t);
    if (live)
      for (int e = t; e < N * N; e += TPM) Hq[e % N + int64_t(e / N) * ld] = Af[e];
  } else {
    for (int i = t; i < N; i += TPM) {
      sd[i] = live ? dg[q * sDE + i] : 0.0;
      se[i] = live && i < N - 1 ? eg[q * sDE + i] : 0.0;
    }
  }
  wave_lds_sync();
  // ---- non-finite input: NaN outputs; the steps below then run on zeros
  double nonfin = 0.0;
  for (int i = t; i < N; i += TPM)
    if (!isfinite(sd[i]) || !isfinite(se[i])) nonfin = 1.0;
  const bool bad = grp_max<TPM>(nonfin) != 0.0;
  for (int i = t; i < N; i += TPM) {
    if (bad) sd[i] = se[i] = 0.0;
    se2[i] = se[i] * se[i];
  }
  wave_lds_sync();
  // ---- bisection, a lane per eigenvalue (as tri_bisect, from the Gershgorin interval)
  double gl = INFINITY, gu = -INFINITY;
  for (int i = t; i < N; i += TPM) {
    const double rad = fabs(se[i]) + (i > 0 ? fabs(se[i - 1]) : 0.0);
    gl = fmin(gl, sd[i] - rad);
    gu = fmax(gu, sd[i] + rad);
  }
  gl = -grp_max<TPM>(-gl);
  gu = grp_max<TPM>(gu);
  const double tnorm = fmax(fabs(gl), fabs(gu));
  const double sc = sturm_scale(tnorm), isc = 1.0 / sc, tn = tnorm * sc;
  double2 de[NM];  // the scaled pairs, every lane of the matrix all of them
#pragma unroll
  for (int i = 0; i < NM; ++i)
    de[i] = i < N ? make_double2(sd[i] * sc, fmax(i > 0 ? se2[i - 1] * sc * sc : 0.0, kSturmE2)) : sturm_pad();
  gl = gl * sc - 2.0 * eps * tn - DBL_MIN;
  gu = gu * sc + 2.0 * eps * tn + DBL_MIN;
  const double tol_abs = eps * eps * tn;
  const int hi = lo + m;
  auto index = [&](int k0) {  // [lambda_0, lambda_{N-1}, lambda_{lo-1}, lambda_hi, lambda_lo ..]
    return k0 == 0 ? 0 : k0 == 1 ? N - 1 : k0 == 2 ? lo - 1 : k0 == 3 ? (hi < N ? hi : -1) : lo + k0 - 4;
  };
  for (int k0 = t; k0 < m + 4; k0 += TPM) {
    const int k = index(k0);
    double val = NAN;
    if (k >= 0) {
      double a = gl, b = gu;
      bool conv = false;
      for (int it = 0; it <= max_it; ++it) {
        const double mid = 0.5 * (a + b);
        conv = b - a <= fmax(2.0 * eps * fmax(fabs(a), fabs(b)) + DBL_MIN, tol_abs) || mid <= a || mid >= b;
        if (conv || it == max_it) break;
        if ((FULL || b - a > kQuotientWidth ? sturm_count_p(de, mid) : sturm_count_i(de, mid)) > k) b = mid;
        else a = mid;
      }
      if (!conv) st |= BE_ST_NONCONVERGED;
      val = 0.5 * (a + b) * isc;
    }
    slam[k0] = val;
  }
  // ---- near zero, the levels of a T that splits, after the loop and from what LDS
  // holds: values kept in registers beside the pairs would leave orders 17 to 32 two
  // waves per SIMD instead of three
  const double s1 = sturm_scale(tnorm);
  double emax2 = 0.0, floored = 0.0;
  for (int i = t; i < N; i += TPM) {
    emax2 = fmax(emax2, se2[i]);
    if (i + 1 < N && below_floor(se2[i] * s1 * s1)) floored = 1.0;
  }
  const double pivmin = DBL_MIN * fmax(1.0, grp_max<TPM>(emax2));
  if (grp_max<TPM>(floored) != 0.0) {
#pragma unroll 1
    for (int k0 = t; k0 < m + 4; k0 += TPM) {
      const double v = slam[k0] * s1, i1 = 1.0 / s1, n1 = tnorm * s1;
      bool conv = true;
      if (fabs(v) <= kLowLevel)
        slam[k0] = low_level(sd, se2, N, index(k0), v, n1, i1, pivmin, eps * eps * n1, max_it, conv) * i1;
      if (!conv) st |= BE_ST_NONCONVERGED;
    }
  }
  wave_lds_sync();
  const double *lam = slam + 4;
  if (live)
    for (int c = t; c < m + 2; c += TPM)
      evals[q * (m + 2) + c] = bad ? NAN : c == 0 ? slam[2] : c == m + 1 ? slam[3] : lam[c - 1];
  if (m > 0) {
    const double scale = fmax(1.0, fmax(fabs(slam[0]), fabs(slam[1])));
    double g = INFINITY;
    if (lo > 0) g = fmin(g, lam[0] - slam[2]);
    if (hi < N) g = fmin(g, slam[3] - lam[m - 1]);
    if (g < 1e-9 * scale) st |= BE_ST_GAP_CLOSED;
  }
  if (m > 0) {
    // ---- inverse iteration, a lane per vector (as tri_invit)
    int nblk = 0;
    if (t == 0) {
      const double splittol = tol_split(tnorm);
      sblk[nblk++] = 0;
      for (int i = 1; i < N; ++i)
        if (fabs(se[i - 1]) <= splittol) sblk[nblk++] = i;
      sblk[nblk] = N;
    }
    nblk = __shfl(nblk, lane - t, 64);
    for (int c = t; c < m; c += TPM) smark[c] = sbad[c] = 0;
    wave_lds_sync();
    const double tiny = eps * fmax(tnorm, DBL_MIN), dclu = tol_cluster(tnorm, clu_rel);
    for (int c = t; c < m; c += TPM) {
      const InvitBlock ib = invit_block(sd, se2, lam, m, c, sblk, nblk, N, tnorm, clu_rel, pivmin);
      if (ib.shared) smark[c] = ib.bs + 2;
      if (!ib.found) sbad[ib.c0] = 1;
      for (int i = 0; i < N; ++i)
        if (i < ib.bs || i >= ib.bt) X0[i * m + c] = 0.0;
      if (!invit_vector<false>(sd, se, ib.bs, ib.bt, ib.lm, tiny, c, X0, ZG, m)) st |= BE_ST_NONCONVERGED;
    }
    wave_lds_sync();
    for (int c = t; c < m; c += TPM) {  // a cluster with a lane that found no block is one group
      int c0 = c;
      while (c0 > 0 && lam[c0] - lam[c0 - 1] <= dclu) --c0;
      if (sbad[c0]) smark[c] = 1;
    }
    wave_lds_sync();
    // ---- groups of a cluster that share a block: modified Gram-Schmidt, two passes, lanes over rows
    for (int c0 = 0; c0 < m;) {
      const int c1 = group_end(lam, smark, m, c0, dclu);
      if (c1 - c0 > 1)
        for (int pass = 0; pass < 2; ++pass)
          for (int c = c0; c < c1; ++c) {
            for (int s2 = c0; s2 <= c; ++s2) {  // s2 == c: normalize
              double d = 0.0;
              for (int i = t; i < N; i += TPM) d = fma(X0[i * m + s2], X0[i * m + c], d);
              d = grp_sum<TPM>(d);
              const double inv = d > 0.0 ? 1.0 / sqrt(d) : 0.0;
              for (int i = t; i < N; i += TPM)
                X0[i * m + c] = s2 == c ? X0[i * m + c] * inv : X0[i * m + c] - d * X0[i * m + s2];
              wave_lds_sync();
            }
          }
      c0 = c1;
    }
    wave_lds_sync();
    // ---- symmetric orthonormalization (as the general path's Newton-Schulz steps)
    double *G = ZG + N * m;  // m x m, beside the second iterate
    double err = 0.0;
    bool act = true, done2 = false;
    for (int it = 0; it < 8 && __any(act); ++it) {
      double e2 = 0.0;
      for (int e = t; e < m * m; e += TPM) {
        const int r = e % m, c = e / m;
        double g = 0.0;
        for (int i = 0; i < N; ++i) g = fma(X0[i * m + r], X0[i * m + c], g);
        const double off = fabs(g - (r == c ? 1.0 : 0.0));
        e2 = off == off ? fmax(e2, off) : INFINITY;
        if (act) G[e] = (r == c ? 1.5 : 0.0) - 0.5 * g;
      }
      e2 = grp_max<TPM>(e2);
      if (act) {
        err = e2;
        done2 = err < 1e-8;
        act = err > tol_orth && !(err > 1.0);
      }
      wave_lds_sync();
      const bool step = act;
      for (int e = t; e < N * m; e += TPM) {
        const int c = e % m, i = e / m;
        double x = 0.0;
        for (int k = 0; k < m; ++k) x = fma(G[c + k * m], X0[i * m + k], x);
        if (step) ZG[e] = x;
      }
      wave_lds_sync();
      if (step) {
        for (int e = t; e < N * m; e += TPM) X0[e] = ZG[e];
        if (done2) {
          act = false;
          err = 0.0;
        }
      }
      wave_lds_sync();
    }
    if (!(err <= fmax(tol_orth, 1e-10))) st |= BE_ST_NONCONVERGED;
    // ---- U = H_0 ... H_{N-2} Z, a lane per column; written coalesced
    if constexpr (FULL) {
      double2 *Uc = reinterpret_cast<double2 *>(ZG);  // column c at c (N + 1)
      if ((reinterpret_cast<uintptr_t>(ZG) & 15) != 0) Uc = reinterpret_cast<double2 *>(ZG + 1);
      for (int c = t; c < m; c += TPM) {
        double2 *u = Uc + c * (N + 1);
        for (int i = 0; i < N; ++i) u[i] = make_double2(X0[i * m + c], 0.0);
        for (int j = N - 2; j >= 0; --j) {
          double2 s = make_double2(0.0, 0.0);
#pragma unroll 4
          for (int i = j + 1; i < N; ++i) s = be::cadd(s, be::cmulc(A[i + j * N], u[i]));
          s = be::cmul(stau[j], s);
#pragma unroll 4
          for (int i = j + 1; i < N; ++i) u[i] = be::csub(u[i], be::cmul(A[i + j * N], s));
        }
      }
      wave_lds_sync();
      if (live)
        for (int e = t; e < N * m; e += TPM) {
          const int r = e % N, c = e / N;
          U[q * sU + r + int64_t(c) * ldu] = bad ? OUT{NAN, NAN} : OUT{Uc[c * (N + 1) + r].x, Uc[c * (N + 1) + r].y};
        }
    } else if constexpr (MODE == kFullC64) {
      // U = Z - V (T (V^H Z)) over rows 1 .. N-1, Z rounded to FP32
      float2 *Z = reinterpret_cast<float2 *>(ZG), *X = Z + N * m, *Y = Wf;  // W is done with, m <= N
      for (int e = t; e < N * m; e += TPM) Z[e] = make_float2(float(X0[e % N * m + e / N]), 0.f);
      wave_lds_sync();
      for (int e = t; e < N * m; e += TPM) X[e] = product_c64<true>(Af + 1 + e % N * N, 1, Z + 1 + e / N * N, N - 1);
      wave_lds_sync();
      for (int e = t; e < N * m; e += TPM) Y[e] = product_c64<false>(Tf + e % N, N, X + e / N * N, N);
      wave_lds_sync();
      for (int e = t; e < N * m; e += TPM) {
        const int r = e % N, c = e / N;
        float2 z = Z[e];
        if (r > 0) {
          const float2 p = product_c64<false>(Af + r, N, Y + c * N, N);
          z.x -= p.x;
          z.y -= p.y;
        }
        if (live) U[q * sU + r + int64_t(c) * ldu] = bad ? OUT{NAN, NAN} : OUT{z.x, z.y};
      }
    } else if (live) {
      typedef decltype(OUT{}.x) F;
      for (int e = t; e < N * m; e += TPM) {
        const int r = e % N, c = e / N;
        U[q * sU + r + int64_t(c) * ldu] = bad ? OUT{F(NAN), F(NAN)} : OUT{F(X0[r * m + c]), F(0)};
      }
    }
  }
  if (bad) st = BE_ST_NAN_INF;
#pragma unroll
  for (int o = TPM / 2; o > 0; o >>= 1) st |= uint32_t(__shfl_xor(int(st), o, 64));
  if (live && t == 0) status[q] = st;
}

template <int TPM, int NM, SmallMode MODE, typename IN, typename OUT>
int launch_small(be_ctx *ctx, IN *H, int64_t sH, int ld, const double *d, const double *e, int64_t sDE, int N,
                 int lo, int m, int64_t n_mat, double clu_rel, double tol_orth, double *evals, OUT *U, int ldu,
                 int64_t sU, uint32_t *status, hipStream_t stream) {
  constexpr int MPB = 64 / TPM;
  const size_t lds = size_t(MPB) * small_doubles(N, m, MODE) * sizeof(double) + 16;
  auto kern = &eigh_small_kernel<TPM, NM, MODE, IN, OUT>;
  hipLaunchKernelGGL(kern, dim3(static_cast<uint32_t>((n_mat + MPB - 1) / MPB)), dim3(64), lds, stream, H, sH, ld, d, e,
                     sDE, N, lo, m, n_mat, clu_rel, tol_orth, ctx->dbg_bisect_max_iter, evals, U, ldu, sU, status);
  return be::check_launch(ctx, "eigh_small");
}

}  // namespace

namespace be {

int eigh_small_fp64(be_ctx *ctx, double2 *H, int N, int ld, int64_t ms, int64_t n_mat, int lo, int hi, double *evals,
                    double2 *U, int ldu, int64_t us, uint32_t *status, hipStream_t stream, double clu_rel) {
  ProfScope prof(ctx, "eigh_small", stream);
  auto go = N <= 4    ? &launch_small<8, 4, kFull, double2, double2>
            : N <= 8  ? &launch_small<8, 8, kFull, double2, double2>
            : N <= 16 ? &launch_small<16, 16, kFull, double2, double2>
                      : &launch_small<64, 32, kFull, double2, double2>;
  return go(ctx, H, ms, ld, nullptr, nullptr, 0, N, lo, hi - lo, n_mat, clu_rel, 1e-14, evals, U, ldu, us, status, stream);
}

int eigh_small_c64(be_ctx *ctx, float2 *H, int N, int ld, int64_t ms, int64_t n_mat, int lo, int hi, double *evals,
                   double2 *U, int ldu, int64_t us, uint32_t *status, hipStream_t stream, double clu_rel) {
  ProfScope prof(ctx, "eigh_small_c64", stream);
  auto go = N <= 4   ? &launch_small<8, 4, kFullC64, float2, double2>
            : N <= 8 ? &launch_small<8, 8, kFullC64, float2, double2>
                     : &launch_small<16, 16, kFullC64, float2, double2>;
  return go(ctx, H, ms, ld, nullptr, nullptr, 0, N, lo, hi - lo, n_mat, clu_rel, 2e-7, evals, U, ldu, us, status, stream);
}

int tri_small_c64(be_ctx *ctx, const double *d, const double *e, int N, int64_t n_mat, int lo, int hi, double *evals,
                  float2 *Z, int ldz, int64_t sz, uint32_t *status, hipStream_t stream, double clu_rel, double tol_orth) {
  ProfScope prof(ctx, "tri_small", stream);
  auto go = N <= 4    ? &launch_small<8, 4, kTri, float2, float2>
            : N <= 8  ? &launch_small<8, 8, kTri, float2, float2>
            : N <= 16 ? &launch_small<16, 16, kTri, float2, float2>
                      : &launch_small<64, 32, kTri, float2, float2>;
  return go(ctx, static_cast<float2 *>(nullptr), 0, 0, d, e, N, N, lo, hi - lo, n_mat, clu_rel, tol_orth, evals, Z, ldz, sz, status, stream);
}

}  // namespace be
