// Berry flux through the plaquettes of a k-grid (the coupling-matrix method
// of the disordered quadrupolar-insulator example, Sec. IV: the zone is cut
// into plaquettes and the Berry flux through each is integrated along its
// closed boundary; applied to the occupied bands or to one spin sector).
//
// Link variables between neighbouring grid points, along the loop direction
// and across it (both periodic), det(U(k')^H U(k)):
//   links    batched MFMA GEMMs U(k')^H U(k) (the across-direction batch runs
//            with the transverse index innermost and cyclic),
//   phases   k_det_phase_r, k_det_phase: blocked LU with partial pivoting, one workgroup per link,
//            arg det = sum of the pivots' arguments (+ pi per row swap),
//            log |det| = sum of log |pivot|. A link is singular, its
//            variable det/|det| undetermined, when its smallest singular
//            value is below 1e-8 (the test the Wilson loop applies to its
//            overlaps). No singular value of an overlap of orthonormal bases
//            exceeds 1, so |det| <= sigma_min: |det| >= 1e-8 proves the link
//            regular. Otherwise (a near-singular link, or only a high order:
//            0.97^640 < 1e-8) sigma_min is estimated from the LU factors by
//            inverse iteration on (M^H M)^{-1}, whose Rayleigh quotient
//            bounds 1/sigma_min^2 from below,
//   flux     k_plaquette: F(i, j) = wrap(phi_par(i+1, j) - phi_par(i, j)
//            + phi_perp(i, j) - phi_perp(i, j+1)) in (-pi, pi], oriented so
//            that the sum over the zone is 2 pi times the winding of eq. 6;
//            each link enters two plaquettes with opposite signs, so the sum
//            is an exact multiple of 2 pi (the Chern number).
#include <algorithm>
#include <cfloat>
#include <cmath>
#include <mutex>
#include <string>
#include <type_traits>

#include "common.hpp"
#include "lanes.hpp"

namespace {

constexpr int DT = 256;  // threads per determinant
constexpr double kPi = 3.14159265358979323846;
constexpr double kLogSingular = -18.420680743952367;  // log(1e-8)

__device__ __forceinline__ double wrap_pi(double x) {
  x -= 2.0 * kPi * rint(x / (2.0 * kPi));
  return x <= -kPi ? kPi : x;
}

// Sum over the NT threads of the block (NT a multiple of 64); red: NT/64
// doubles of LDS (unused for one wave). Every thread gets the sum.
template <int NT>
__device__ __forceinline__ double block_sum(double v, double *red) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  if constexpr (NT > 64) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) red[wave] = v;
    __syncthreads();
    v = 0.0;
    for (int w = 0; w < NT / 64; ++w) v += red[w];
  }
  return v;
}

// Smallest singular value of an m x m matrix from its LU factors P M = L U,
// stored in place (row-major rows of length m; unit lower L strictly below
// the diagonal, U on and above it). Row interchanges do not
// change singular values, so sigma_min(M) = sigma_min(L U). Two steps of
// inverse iteration on (LU)^{-1} (LU)^{-H} from a fixed start vector whose
// entries have modulus one, then the Rayleigh quotient rq = |(LU)^{-H} x|^2
// of the normalized iterate: rq <= 1/sigma_min^2, so the returned 1/sqrt(rq)
// is an upper bound of sigma_min, equal to it once the iterate has converged
// (each step scales the other singular directions down by
// (sigma_min/sigma_k)^2 against the smallest one). Returns 0 when a solve
// overflows (singular to working precision).
// Triangular solves are column-oriented with a fixed owner per row (thread
// r mod NT), one barrier per column: the pivot column's value is published
// through a double-buffered LDS slot. Solves with U^H and L^H read rows of
// the factors (coalesced); solves with L and U read columns.
// x: m double2 of LDS, slot: 2 double2 of LDS, red: as for block_sum.
template <int NT>
__device__ double lu_smin(const double2 *A, int m, double2 *x, double2 *slot, double *red) {
  const int tid = threadIdx.x;
  auto rowp = [&](int i) { return A + int64_t(i) * m; };
  auto first_above = [&](int c) {  // smallest r > c owned by this thread
    int r = tid;
    if (r <= c) r += ((c - r) / NT + 1) * NT;
    return r;
  };
  for (int i = tid; i < m; i += NT) {
    const uint32_t h = uint32_t(i + 1) * 2654435761u;
    double sn, cs;
    sincospi(double(h) * (2.0 / 4294967296.0), &sn, &cs);
    x[i] = make_double2(cs, sn);
  }
  for (int it = 0;; ++it) {
    // normalize
    double ss = 0.0;
    for (int i = tid; i < m; i += NT) ss += x[i].x * x[i].x + x[i].y * x[i].y;
    ss = block_sum<NT>(ss, red);
    if (!(ss > 0.0) || !isfinite(ss)) return 0.0;
    const double inv = 1.0 / sqrt(ss);
    for (int i = tid; i < m; i += NT) x[i] = make_double2(x[i].x * inv, x[i].y * inv);
    __syncthreads();
    // U^H t = x, forward: t_c = x_c / conj(u_cc), x_r -= conj(U(c, r)) t_c (r > c)
    for (int c = 0; c < m; ++c) {
      const double2 *Ac = rowp(c);
      if (tid == c % NT) {
        const double2 u = Ac[c], xc = x[c];
        const double den = u.x * u.x + u.y * u.y;
        const double2 t = make_double2((xc.x * u.x - xc.y * u.y) / den, (xc.x * u.y + xc.y * u.x) / den);
        x[c] = t;
        slot[c & 1] = t;
      }
      __syncthreads();
      const double2 t = slot[c & 1];
      for (int r = first_above(c); r < m; r += NT) {
        const double2 a = Ac[r];
        x[r] = make_double2(x[r].x - (a.x * t.x + a.y * t.y), x[r].y - (a.x * t.y - a.y * t.x));
      }
    }
    __syncthreads();
    // L^H y = t, backward (unit diagonal): t_r -= conj(L(c, r)) y_c (r < c)
    for (int c = m - 1; c >= 0; --c) {
      const double2 *Ac = rowp(c);
      if (tid == c % NT) slot[c & 1] = x[c];
      __syncthreads();
      const double2 y = slot[c & 1];
      for (int r = tid; r < c; r += NT) {
        const double2 a = Ac[r];
        x[r] = make_double2(x[r].x - (a.x * y.x + a.y * y.y), x[r].y - (a.x * y.y - a.y * y.x));
      }
    }
    __syncthreads();
    double rq = 0.0;
    for (int i = tid; i < m; i += NT) rq += x[i].x * x[i].x + x[i].y * x[i].y;
    rq = block_sum<NT>(rq, red);
    if (!(rq > 0.0) || !isfinite(rq)) return 0.0;
    if (it == 2) return 1.0 / sqrt(rq);
    // L v = y, forward (unit diagonal): y_r -= L(r, c) v_c (r > c)
    for (int c = 0; c < m; ++c) {
      if (tid == c % NT) slot[c & 1] = x[c];
      __syncthreads();
      const double2 v = slot[c & 1];
      for (int r = first_above(c); r < m; r += NT) {
        const double2 a = rowp(r)[c];
        x[r] = make_double2(x[r].x - (a.x * v.x - a.y * v.y), x[r].y - (a.x * v.y + a.y * v.x));
      }
    }
    __syncthreads();
    // U z = v, backward: z_c = v_c / u_cc, v_r -= U(r, c) z_c (r < c)
    for (int c = m - 1; c >= 0; --c) {
      if (tid == c % NT) {
        const double2 u = rowp(c)[c], vc = x[c];
        const double den = u.x * u.x + u.y * u.y;
        const double2 z = make_double2((vc.x * u.x + vc.y * u.y) / den, (vc.y * u.x - vc.x * u.y) / den);
        x[c] = z;
        slot[c & 1] = z;
      }
      __syncthreads();
      const double2 z = slot[c & 1];
      for (int r = tid; r < c; r += NT) {
        const double2 a = rowp(r)[c];
        x[r] = make_double2(x[r].x - (a.x * z.x - a.y * z.y), x[r].y - (a.x * z.y + a.y * z.x));
      }
    }
    __syncthreads();
  }
}

// Largest value of the lanes of a wave and its index (the smallest of equals)
template <int O>
__device__ __forceinline__ void best_step(double &best, int &bi) {
  double ov = best;
  int oi = bi;
  if constexpr (O >= 16) {  // both halves' values in every lane
    const uint2 l = lane_swap<O>(uint32_t(__double2loint(best)), uint32_t(__double2loint(best)));
    const uint2 h = lane_swap<O>(uint32_t(__double2hiint(best)), uint32_t(__double2hiint(best)));
    const uint2 i = lane_swap<O>(uint32_t(bi), uint32_t(bi));
    best = __hiloint2double(int(h.x), int(l.x));
    ov = __hiloint2double(int(h.y), int(l.y));
    bi = int(i.x);
    oi = int(i.y);
  } else {
    ov = lane_xor<O>(best);
    oi = __float_as_int(lane_xor<O>(__int_as_float(bi)));
  }
  const bool take = ov > best || (ov == best && oi < bi);
  best = take ? ov : best;
  bi = take ? oi : bi;
}
__device__ __forceinline__ void lane_best(double &best, int &bi) {
  best_step<32>(best, bi);
  best_step<16>(best, bi);
  best_step<8>(best, bi);
  best_step<4>(best, bi);
  best_step<2>(best, bi);
  best_step<1>(best, bi);
}

// Singular-value certificate of a link from its LU: log |det| when that is at
// least log(1e-8) (then sigma_min >= |det| >= 1e-8), else log of the inverse
// iteration's upper bound of sigma_min (-inf for a zero pivot). The link is
// flagged singular when the certificate is below log(1e-8).
//
// arg det and log |det| of A_q (m x m, ld m) by blocked LU with partial
// pivoting, in place. The factorization runs on M = A_q^T (det M = det A_q),
// whose rows are contiguous in memory, so that row interchanges, the block
// row of U and the trailing update are all coalesced. Per panel of NB columns:
//   1. load rows k0.. of the panel into LDS (column by column), find the
//      first pivot while loading;
//   2. factor the panel in LDS, column by column (pivot, interchange within
//      the panel, multipliers, rank-1 update of the panel's later columns,
//      search for the next pivot fused with the update: two barriers per
//      column);
//   3. one thread per trailing column: apply the panel's interchanges and
//      solve with the unit lower triangle L11 (the panel's block row of U);
//   4. trailing update M22 -= L21 U12: a wave per row stream, lanes over
//      consecutive columns, U12 in registers, L21 broadcast from LDS.
// The factored panel is written back and its interchanges are applied to the
// columns left of it, so M ends holding the LU factors of its row-permuted
// self (read by lu_smin when |det| < 1e-8).
// phase[q] = sum of the pivots' arguments (+ pi per interchange), wrapped to
// (-pi, pi]; lsig[q] = the singular-value certificate above. A zero pivot
// leaves a zero column below it: nothing is eliminated.
template <int NB>
__global__ __launch_bounds__(DT) void k_det_phase(double2 *A, int m, int64_t sA, double *phase, double *lsig) {
  extern __shared__ double2 sP[];  // panel, column-major: sP[c * rows + r]
  __shared__ double s_v[DT / 64];
  __shared__ int s_i[DT / 64];
  __shared__ int s_piv[NB];
  __shared__ double s_la;
  double2 *M = A + int64_t(blockIdx.x) * sA;  // M[r][c] = M[r * m + c]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  double ph = 0.0, la = 0.0;

  auto wave_best = [&](double best, int bi) {
    for (int o = 32; o > 0; o >>= 1) {
      const double ov = __shfl_xor(best, o, 64);
      const int oi = __shfl_xor(bi, o, 64);
      if (ov > best || (ov == best && oi < bi)) {
        best = ov;
        bi = oi;
      }
    }
    if (lane == 0) {
      s_v[wave] = best;
      s_i[wave] = bi;
    }
  };

  for (int k0 = 0; k0 < m; k0 += NB) {
    const int nbp = min(NB, m - k0), rows = m - k0;
    // ---- 1. panel load, pivot search of its first column
    {
      double best = -1.0;
      int bi = 0;
      for (int e = tid; e < rows * nbp; e += DT) {
        const int r = e / nbp, c = e - r * nbp;
        const double2 v = M[int64_t(k0 + r) * m + k0 + c];
        sP[c * rows + r] = v;
        if (c == 0) {
          const double a2 = v.x * v.x + v.y * v.y;
          if (a2 > best || (a2 == best && r < bi)) {
            best = a2;
            bi = r;
          }
        }
      }
      wave_best(best, bi);
    }
    __syncthreads();
    // ---- 2. panel factorization
    for (int c = 0; c < nbp; ++c) {
      double b = s_v[0];
      int p = s_i[0];
      for (int w = 1; w < DT / 64; ++w)
        if (s_v[w] > b || (s_v[w] == b && s_i[w] < p)) {
          b = s_v[w];
          p = s_i[w];
        }
      if (b < 0.0) p = c;  // no rows (cannot happen for c < rows)
      if (p != c)
        for (int cc = tid; cc < nbp; cc += DT) {
          const double2 t = sP[cc * rows + c];
          sP[cc * rows + c] = sP[cc * rows + p];
          sP[cc * rows + p] = t;
        }
      if (tid == 0) s_piv[c] = p;
      __syncthreads();
      const double2 piv = sP[c * rows + c];
      const double den = piv.x * piv.x + piv.y * piv.y;
      if (tid == 0) {
        ph += atan2(piv.y, piv.x) + (p != c ? kPi : 0.0);
        la += 0.5 * log(den);
      }
      const double2 ipv = den > 0.0 ? make_double2(piv.x / den, -piv.y / den) : make_double2(0.0, 0.0);
      double best = -1.0;
      int bi = c + 1;
      for (int r = c + 1 + tid; r < rows; r += DT) {
        const double2 a = sP[c * rows + r];
        const double2 l = make_double2(a.x * ipv.x - a.y * ipv.y, a.x * ipv.y + a.y * ipv.x);
        sP[c * rows + r] = l;
        for (int cc = c + 1; cc < nbp; ++cc) {
          const double2 u = sP[cc * rows + c];
          double2 x = sP[cc * rows + r];
          x.x -= l.x * u.x - l.y * u.y;
          x.y -= l.x * u.y + l.y * u.x;
          sP[cc * rows + r] = x;
          if (cc == c + 1) {
            const double a2 = x.x * x.x + x.y * x.y;
            if (a2 > best) {
              best = a2;
              bi = r;
            }
          }
        }
      }
      wave_best(best, bi);
      __syncthreads();
    }
    // the factored panel (L21 below, U11 on and above the diagonal) back to
    // M, and its interchanges applied to the columns left of it, so that M
    // ends as the LU factors of the row-permuted matrix (for sigma_min)
    for (int e = tid; e < rows * nbp; e += DT) {
      const int r = e / nbp, c = e - r * nbp;
      M[int64_t(k0 + r) * m + k0 + c] = sP[c * rows + r];
    }
#pragma unroll 1
    for (int jj = tid; jj < k0; jj += DT) {
#pragma unroll 1
      for (int c = 0; c < nbp; ++c) {
        const int p = s_piv[c];
        if (p != c) {
          const double2 t = M[int64_t(k0 + c) * m + jj];
          M[int64_t(k0 + c) * m + jj] = M[int64_t(k0 + p) * m + jj];
          M[int64_t(k0 + p) * m + jj] = t;
        }
      }
    }
    if (k0 + nbp >= m) break;
    // ---- 3. interchanges and U12 = L11^{-1} (P A12), one thread per trailing column
    const int j0 = k0 + nbp, C = m - j0;
#pragma unroll 1
    for (int jj = tid; jj < C; jj += DT) {
      const int j = j0 + jj;
#pragma unroll 1
      for (int c = 0; c < nbp; ++c) {
        const int p = s_piv[c];
        if (p != c) {
          const double2 t = M[int64_t(k0 + c) * m + j];
          M[int64_t(k0 + c) * m + j] = M[int64_t(k0 + p) * m + j];
          M[int64_t(k0 + p) * m + j] = t;
        }
      }
      double2 u[NB];
#pragma unroll
      for (int c = 0; c < NB; ++c) {
        if (c < nbp) {
          double2 x = M[int64_t(k0 + c) * m + j];
#pragma unroll
          for (int cc = 0; cc < c; ++cc) {
            const double2 l = sP[cc * rows + c];
            x.x -= l.x * u[cc].x - l.y * u[cc].y;
            x.y -= l.x * u[cc].y + l.y * u[cc].x;
          }
          u[c] = x;
          M[int64_t(k0 + c) * m + j] = x;
        }
      }
    }
    __syncthreads();
    // ---- 4. trailing update M22 -= L21 U12
    for (int jb = 0; jb < C; jb += 64) {
      const int j = j0 + jb + lane;
      const bool ok = jb + lane < C;
      double2 u[NB];
#pragma unroll
      for (int c = 0; c < NB; ++c) u[c] = (ok && c < nbp) ? M[int64_t(k0 + c) * m + j] : make_double2(0.0, 0.0);
#pragma unroll 1
      for (int r = nbp + wave; r < rows; r += DT / 64) {
        if (!ok) continue;
        double2 x = M[int64_t(k0 + r) * m + j];
#pragma unroll
        for (int c = 0; c < NB; ++c) {
          const double2 l = sP[c * rows + r];  // same address across the wave
          x.x -= l.x * u[c].x - l.y * u[c].y;
          x.y -= l.x * u[c].y + l.y * u[c].x;
        }
        M[int64_t(k0 + r) * m + j] = x;
      }
    }
    __syncthreads();
  }
  if (tid == 0) {
    phase[blockIdx.x] = m > 0 ? wrap_pi(ph) : 0.0;
    s_la = la;
  }
  __syncthreads();
  la = s_la;
  if (la < kLogSingular && la > -INFINITY) {
    const double sg = lu_smin<DT>(M, m, sP, sP + m, s_v);
    la = sg > 0.0 ? log(sg) : -INFINITY;
  }
  if (tid == 0) lsig[blockIdx.x] = la;
}

// The same factorization for orders up to NT: a thread per row of the panel of NB
// columns, which it holds in registers, so that a column costs two barriers, a search
// over lanes by moves between them and one LDS read of the pivot row. The
// panel's interchanges reach the other columns as one gather (all rows of a
// column loaded before any is stored), and the trailing update runs on the
// matrix cores: k_det_phase waited out a memory access per interchange and per
// row, a single wave per link below order 128 besides. Bound by the latency of
// the columns' steps. 400 links, a wave or a workgroup per link before -> now:
// order 16 39 -> 25 us, 48 154 -> 91, 79 382 -> 188, 128 1,198 -> 376; 500 of
// order 166 996 -> 637; 300 of order 256 2.42 -> 1.32 ms. lsig and phase as there (the sums over the
// pivots in another order).
template <int NT, int NB>
__global__ __launch_bounds__(NT, 2) void k_det_phase_r(double2 *A, int m, int64_t sA, double *phase, double *lsig) {
  constexpr int NW = NT / 64, KT = NB / 4;  // KT: matrix-core steps of a panel's columns
  constexpr int LP = NB + 1;       // pitch: lanes that read a column of 16 rows meet different banks
  extern __shared__ double2 sL[];  // factored panel, row by row: sL[r * LP + c]
  __shared__ double2 s_row[2][NB];  // the pivot's row, the row it takes the place of
  __shared__ double2 s_piv[NB];
  __shared__ double s_v[NW];
  __shared__ int s_i[NW], s_p[NB], s_src[NT];
  double2 *M = A + int64_t(blockIdx.x) * sA;  // M[r][c] = M[r * m + c]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lk = lane >> 4, wv = __builtin_amdgcn_readfirstlane(wave);
  double ph = 0.0, la = 0.0;  // lane c < NB: of the pivots of columns c, NB + c, ...
  for (int k0 = 0; k0 < m; k0 += NB) {
    const int nbp = min(NB, m - k0), rows = m - k0;
    double2 x[NB];
    unrolled<NB>([&](auto CC) {
      constexpr int c = CC;
      const double2 v = M[int64_t(k0 + min(tid, rows - 1)) * m + k0 + min(c, nbp - 1)];
      x[c] = make_double2(c < nbp ? v.x : 0.0, c < nbp ? v.y : 0.0);
    });
    s_src[tid] = tid;
    unrolled<NB>([&](auto CC) {
      constexpr int c = CC;
      if (c < nbp) {
        // pivot: the largest |x_c| of rows c .., the first of equal ones (none: row c)
        const double a2 = x[c].x * x[c].x + x[c].y * x[c].y;
        double best = tid >= c && tid < rows && a2 > -1.0 ? a2 : -1.0;
        int bi = tid;
        lane_best(best, bi);
        if (lane == 0) {
          s_v[wave] = best;
          s_i[wave] = bi;
        }
        __syncthreads();
        best = s_v[0];
        int p = s_i[0];
        for (int w = 1; w < NW; ++w)
          if (s_v[w] > best || (s_v[w] == best && s_i[w] < p)) {
            best = s_v[w];
            p = s_i[w];
          }
        if (best < 0.0) p = c;
        if (tid == p || tid == c) {  // (row c is the pivot's own where p = c)
          double2 *const to = s_row[tid != p];
          unrolled<NB>([&](auto D) { to[D] = x[D]; });
        }
        if (tid == 0) {
          s_p[c] = p;
          const int t = s_src[c];
          s_src[c] = s_src[p];
          s_src[p] = t;
        }
        __syncthreads();
        const bool swap = p != c && (tid == c || tid == p);
        if (__any(swap)) {
          const double2 *const from = s_row[tid == p];
          unrolled<NB>([&](auto D) {
            const double2 o = from[D];
            x[D] = make_double2(swap ? o.x : x[D].x, swap ? o.y : x[D].y);
          });
        }
        const double2 pv = s_row[0][c];
        const double den = pv.x * pv.x + pv.y * pv.y;
        if (tid == 0) s_piv[c] = pv;
        const double2 ipv = den > 0.0 ? make_double2(pv.x / den, -pv.y / den) : make_double2(0.0, 0.0);
        const double2 l0 = be::cmul(x[c], ipv);
        const bool below = tid > c;  // rows up to c stay: their multiplier is zero
        const double2 l = make_double2(below ? l0.x : 0.0, below ? l0.y : 0.0);
        x[c] = make_double2(below ? l.x : x[c].x, below ? l.y : x[c].y);
        unrolled<NB - 1 - c>([&](auto D) {
          constexpr int cc = c + 1 + D;
          x[cc] = be::csub(x[cc], be::cmul(l, s_row[0][cc]));
        });
      }
    });
    // the factored panel to LDS (L11 and L21 of the steps below) and back to M
    if (tid < rows)
      unrolled<NB>([&](auto D) {
        sL[tid * LP + D] = x[D];
        if (D < nbp) M[int64_t(k0 + tid) * m + k0 + D] = x[D];
      });
    __syncthreads();
    if (tid < nbp) {
      const double2 pv = s_piv[tid];
      ph += atan2(pv.y, pv.x) + (s_p[tid] != tid ? kPi : 0.0);
      la += 0.5 * log(pv.x * pv.x + pv.y * pv.y);
    }
    // interchanges of the other columns, a thread per column: the first nbp rows
    // and the pivots' old rows change (a pivot from the first rows, or a column
    // past the last panel's, stores what the rows' own stores then replace);
    // right of the panel also U12 = L11^{-1} (P A12)
    const int j0 = k0 + nbp, C = m - j0;
    auto interchange = [&](int j, auto solve) {
      double2 u[NB];
      double vx[NB], vy[NB];
      unrolled<NB>([&](auto D) {  // the rows are the same in every thread: scalar addresses
        const int cc = min(int(D), nbp - 1);
        const int ru = __builtin_amdgcn_readfirstlane(s_src[cc]), rv = __builtin_amdgcn_readfirstlane(s_src[s_p[cc]]);
        u[D] = (M + int64_t(k0 + ru) * m)[j];
        const double2 v = (M + int64_t(k0 + rv) * m)[j];
        vx[D] = v.x;
        vy[D] = v.y;
      });
      unrolled<NB>([&](auto D) {
        const int r = __builtin_amdgcn_readfirstlane(s_p[min(int(D), nbp - 1)]);
        (M + int64_t(k0 + r) * m)[j] = make_double2(vx[D], vy[D]);
      });
      // L11 is read when the rows' registers are free again (read ahead of the
      // stores it made registers spill)
      __builtin_amdgcn_sched_barrier(0);
      unrolled<NB>([&](auto D) {
        constexpr int c = D;
        if constexpr (c % 4 == 0) __builtin_amdgcn_sched_barrier(0);
        double2 y = u[c];
        if constexpr (decltype(solve)::value)
          unrolled<c>([&](auto E) { y = be::csub(y, be::cmul(sL[c * LP + E], u[E])); });
        u[c] = y;
        (M + int64_t(k0 + min(c, nbp - 1)) * m)[j] = y;
      });
    };
    for (int j = tid; j < k0; j += NT) interchange(j, std::false_type{});
    for (int j = j0 + tid; j < m; j += NT) interchange(j, std::true_type{});
    __syncthreads();
    // trailing update M22 -= L21 U12 on the matrix cores (broadcasts of L21 to a
    // lane per column kept the LDS busier than the FP64 units): a wave per
    // 16 columns, whose U12 it holds
    const int nct = (C + 15) / 16, nrt = (rows - nbp + 15) / 16;
    for (int ct = wv; ct < nct; ct += NW) {
      const int jc = 16 * ct + li, j = j0 + min(jc, C - 1);
      double2 u[KT];
#pragma unroll
      for (int t = 0; t < KT; ++t) u[t] = M[int64_t(k0 + 4 * t + lk) * m + j];  // C > 0: nbp = NB
      double2 *Mj = M + int64_t(j0) * m + j;
      const int rmax = rows - nbp - 1;
      double2 y[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) y[r] = Mj[int64_t(min(lk + 4 * r, rmax)) * m];
      for (int rt = 0; rt < nrt; ++rt) {
        v4d re, im;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          re[r] = y[r].x;
          im[r] = y[r].y;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) y[r] = Mj[int64_t(min(16 * (rt + 1) + lk + 4 * r, rmax)) * m];  // the next tile
        const double2 *Lr = sL + (nbp + min(16 * rt + li, rmax)) * LP + lk;
#pragma unroll
        for (int t = 0; t < KT; ++t) {
          const double2 l = Lr[4 * t];
          re = __builtin_amdgcn_mfma_f64_16x16x4f64(-l.x, u[t].x, re, 0, 0, 0);
          im = __builtin_amdgcn_mfma_f64_16x16x4f64(-l.x, u[t].y, im, 0, 0, 0);
          re = __builtin_amdgcn_mfma_f64_16x16x4f64(l.y, u[t].y, re, 0, 0, 0);
          im = __builtin_amdgcn_mfma_f64_16x16x4f64(-l.y, u[t].x, im, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int i = 16 * rt + lk + 4 * r;
          if (i <= rmax && jc < C) Mj[int64_t(i) * m] = make_double2(re[r], im[r]);
        }
      }
    }
    __syncthreads();
  }
  if (wave == 0) {  // sums over the NB lanes that hold pivots
    ph = lane < NB ? ph : 0.0;
    la = lane < NB ? la : 0.0;
#pragma unroll
    for (int o = NB / 2; o > 0; o >>= 1) {
      ph += __shfl_xor(ph, o, 64);
      la += __shfl_xor(la, o, 64);
    }
    if (lane == 0) {
      phase[blockIdx.x] = m > 0 ? wrap_pi(ph) : 0.0;
      s_v[0] = la;
    }
  }
  __syncthreads();
  la = s_v[0];
  __syncthreads();
  if (la < kLogSingular && la > -INFINITY) {
    const double sg = lu_smin<NT>(M, m, sL, sL + m, s_v);
    la = sg > 0.0 ? log(sg) : -INFINITY;
  }
  if (tid == 0) lsig[blockIdx.x] = la;
}

// Largest order of the kernel with a row per thread, and the panel width of the
// other for order m (a panel of at most 160 KiB of LDS; 64 where that fits).
constexpr int kDetRows = 256;
// Panel columns of the kernel with a row per thread. A panel holds its columns in
// registers and takes them all to their end, also those past the matrix: small
// orders take the narrowest that covers them; narrow panels leave registers for
// more links per compute unit, wide ones pass over the trailing matrix less often.
// Whole calls, 16 -> 8 columns (4 at order 4): 10,240 links of order 4 94 -> 65 us,
// 8 132 -> 94, 17 323 -> 233, 48 854 -> 774, 65 2.87 -> 2.39 ms, 80 3.16 -> 2.94, 96
// 4.18 -> 4.21; 40,960 of 64 4.94 -> 5.25; 64 links of order 9 59 -> 62 us, 17 102 -> 87,
// 65 323 -> 282, 128 678 -> 693.
int det_panel_cols(int m) {
  if (m <= 4) return 4;
  if (m <= 8) return 8;
  if (m <= 12) return 16;
  return m <= 60 || (m > 64 && m <= 80) ? 8 : 16;
}
int det_panel_width(int m) {
  if (m <= 512) return 8;
  if (m <= 2544) return 4;
  return 0;
}

// One workgroup per system: flux of every plaquette, its sum, Chern number
// and status. phi_par[(s n_perp + i) n_par + j]; phi_perp[(s n_par + j) n_perp + i].
__global__ __launch_bounds__(256) void k_plaquette(const double *phi_par, const double *phi_perp, const double *ls_par,
                                                   const double *ls_perp, int n_par, int n_perp, double *flux,
                                                   int32_t *chern, double *total, uint32_t *status) {
  const int64_t s = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t kps = int64_t(n_par) * n_perp;
  double sum = 0.0, fmx = 0.0, mpmin = INFINITY;
  for (int64_t e = tid; e < kps; e += 256) {
    const int i = int(e / n_par), j = int(e % n_par);
    const int i1 = i + 1 == n_perp ? 0 : i + 1, j1 = j + 1 == n_par ? 0 : j + 1;
    const double *pp = phi_par + s * kps;
    const double *pq = phi_perp + s * kps;
    const double F = wrap_pi(pp[int64_t(i1) * n_par + j] - pp[int64_t(i) * n_par + j] + pq[int64_t(j) * n_perp + i] -
                             pq[int64_t(j1) * n_perp + i]);
    flux[s * kps + e] = F;
    sum += F;
    fmx = fmax(fmx, fabs(F));
    mpmin = fmin(mpmin, fmin(ls_par[s * kps + e], ls_perp[s * kps + int64_t(j) * n_perp + i]));
  }
  for (int o = 32; o > 0; o >>= 1) {
    sum += __shfl_xor(sum, o, 64);
    fmx = fmax(fmx, __shfl_xor(fmx, o, 64));
    mpmin = fmin(mpmin, __shfl_xor(mpmin, o, 64));
  }
  __shared__ double r[3][4];
  if (lane == 0) {
    r[0][wave] = sum;
    r[1][wave] = fmx;
    r[2][wave] = mpmin;
  }
  __syncthreads();
  if (tid == 0) {
    double a = 0.0, b = 0.0, c = INFINITY;
    for (int w = 0; w < 4; ++w) {
      a += r[0][w];
      b = fmax(b, r[1][w]);
      c = fmin(c, r[2][w]);
    }
    const double t = a / (2.0 * kPi);
    const double rt = rint(t);
    uint32_t st = 0;
    if (c < kLogSingular) st |= BE_ST_OVERLAP_SINGULAR;
    if (b > 0.8 * kPi || fabs(t - rt) > 1e-6) st |= BE_ST_WINDING_UNRESOLVED;
    const bool fin = isfinite(t) && fabs(t) < 1e9;
    if (!fin) st |= BE_ST_NAN_INF;
    total[s] = t;
    chern[s] = fin ? int32_t(rt) : 0;
    status[s] |= st;
  }
}

__global__ void k_zero_st(uint32_t *p, int64_t n) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

}  // namespace

// ---------------------------------------------------------------- scratch without allocation
// Fixed device scratch of be_plaquette_flux_noalloc (one copy per device,
// held for the life of the process). Host code never uses the array's name
// as an address: its device address comes from hipGetSymbolAddress, taken
// once per device at context creation.
static __device__ __align__(256) unsigned char scratch[BE_NOALLOC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};
}  // namespace

namespace be {
// Called by be_create with `device` current.
int noalloc_scratch_init(be_ctx *ctx, int device) {
  if (device < 0 || device >= kMaxDevices) return set_err(ctx, BE_EINVAL, "device index beyond the scratch table");
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (g_scratch_ptr[device]) return BE_OK;
  void *ptr = nullptr;
  const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
  if (e != hipSuccess || !ptr) {
    (void)hipGetLastError();
    return set_err(ctx, BE_EHIP, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
  }
  g_scratch_ptr[device] = ptr;
  return BE_OK;
}
}  // namespace be

namespace {

// Scratch of one flux call: the links of one direction for spp systems and
// four per-link arrays (phases and singular-value certificates, both directions).
struct FluxScratch {
  double2 *L = nullptr;
  double *ph_par = nullptr, *ph_perp = nullptr, *ls_par = nullptr, *ls_perp = nullptr;
  void declare(be::Carve &cv, int64_t spp, int64_t kps, int64_t mm) {
    cv.add(&L, size_t(spp * kps * mm));
    cv.add(&ph_par, size_t(spp * kps));
    cv.add(&ph_perp, size_t(spp * kps));
    cv.add(&ls_par, size_t(spp * kps));
    cv.add(&ls_perp, size_t(spp * kps));
  }
};

int check_flux_args(be_ctx *ctx, const void *U, int32_t N, int32_t m, int32_t ldu, int64_t u_stride, int32_t n_sys,
                    int32_t n_par, int32_t n_perp, double *flux, int32_t *chern, double *total, uint32_t *status) {
  using namespace be;
  BE_CHECK_ARG(ctx, ctx && U && flux && chern && total && status, "be_plaquette_flux: null argument");
  BE_CHECK_ARG(ctx, N >= 1 && m >= 0 && m <= N, "be_plaquette_flux: need 0 <= m <= N");
  BE_CHECK_ARG(ctx, ldu >= N && u_stride >= int64_t(ldu) * std::max(m, 1), "be_plaquette_flux: ldu < N or u_stride < ldu*m");
  BE_CHECK_ARG(ctx, n_sys >= 0 && n_par >= 1 && n_perp >= 1, "be_plaquette_flux: need n_sys >= 0, n_par, n_perp >= 1");
  BE_CHECK_ARG(ctx, det_panel_width(m) > 0, "be_plaquette_flux: m > 2544 not supported");
  return BE_OK;
}

// The flux computation on scratch `fs` holding the links of spp systems.
int flux_run(be_ctx *ctx, const void *U, int32_t N, int32_t m, int32_t ldu, int64_t u_stride, int32_t n_sys,
             int32_t n_par, int32_t n_perp, double *flux, int32_t *chern, double *total, uint32_t *status,
             const FluxScratch &fs, int64_t spp, hipStream_t stream) {
  using namespace be;
  const int nbw = det_panel_width(m);
  // dynamic LDS up to the panel size of the width in use (set on every call:
  // a cheap host call, valid for whichever device is current)
  if (nbw == 4)
    BE_HIP_TRY(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(&k_det_phase<4>),
                                        hipFuncAttributeMaxDynamicSharedMemorySize, 2544 * 4 * 16));
  else if (m > kDetRows)
    BE_HIP_TRY(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(&k_det_phase<8>),
                                        hipFuncAttributeMaxDynamicSharedMemorySize, 512 * 8 * 16));
  const int64_t kps = int64_t(n_par) * n_perp;
  const int64_t mm = int64_t(std::max(m, 1)) * std::max(m, 1);
  hipLaunchKernelGGL(k_zero_st, dim3((n_sys + 255) / 256), dim3(256), 0, stream, status, int64_t(n_sys));
  BE_RET_IF(check_launch(ctx, "zero"));
  double2 *L = fs.L;
  const double2 *Ud = static_cast<const double2 *>(U);
  for (int64_t s0 = 0; s0 < n_sys; s0 += spp) {
    const int64_t ns = std::min<int64_t>(spp, n_sys - s0);
    const int64_t nk = ns * kps;
    const double2 *Us = Ud + s0 * kps * u_stride;
    for (int dir = 0; dir < 2; ++dir) {
      if (m > 0) {
        ZGemm g;  // links U(k')^H U(k)
        g.M = m;
        g.N = m;
        g.K = N;
        g.opA = 1;
        g.A = Us;
        g.lda = ldu;
        g.B = Us;
        g.ldb = ldu;
        if (dir == 0) {  // k' = k(i, j+1): batch (s, i, j), j innermost and cyclic
          g.bA = ZBatch::cyclic(u_stride, n_par, 1, int64_t(n_par) * u_stride);
          g.bB = ZBatch::strided(u_stride);
        } else {  // k' = k(i+1, j): batch (s, j, i), i innermost and cyclic
          ZBatch a = ZBatch::cyclic(int64_t(n_par) * u_stride, n_perp, 1, kps * u_stride);
          a.s1 = u_stride;
          a.n1 = n_par;
          ZBatch b = a;
          b.shift = 0;
          g.bA = a;
          g.bB = b;
        }
        g.C = L;
        g.ldc = m;
        g.bC = ZBatch::strided(mm);
        g.batch = nk;
        g.tag = "flux_links";
        BE_RET_IF(zgemm(ctx, g, stream));
      }
      {
        ProfScope prof(ctx, "det_phase", stream);
        const size_t lds = size_t(std::max(m, 1)) * nbw * sizeof(double2);
        double *ph = dir == 0 ? fs.ph_par : fs.ph_perp, *ls = dir == 0 ? fs.ls_par : fs.ls_perp;
        const dim3 grid(static_cast<uint32_t>(nk));
        if (m <= kDetRows) {
          const int nt = m <= 64 ? 64 : m <= 128 ? 128 : 256, nb = det_panel_cols(m);
          const size_t sm = size_t(std::max(m, 1)) * (nb + 1) * sizeof(double2);
          auto kern = nt == 256 ? &k_det_phase_r<256, 16>
                      : nt == 128 ? (nb == 8 ? &k_det_phase_r<128, 8> : &k_det_phase_r<128, 16>)
                      : nb == 4   ? &k_det_phase_r<64, 4>
                      : nb == 8   ? &k_det_phase_r<64, 8>
                                  : &k_det_phase_r<64, 16>;
          if (sm > 65536)
            BE_HIP_TRY(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                                hipFuncAttributeMaxDynamicSharedMemorySize, int(sm)));
          hipLaunchKernelGGL(kern, grid, dim3(nt), sm, stream, L, m, mm, ph, ls);
        }
        else if (nbw == 8)
          hipLaunchKernelGGL(k_det_phase<8>, grid, dim3(DT), lds, stream, L, m, mm, ph, ls);
        else
          hipLaunchKernelGGL(k_det_phase<4>, grid, dim3(DT), lds, stream, L, m, mm, ph, ls);
      }
      BE_RET_IF(check_launch(ctx, "det_phase"));
    }
    hipLaunchKernelGGL(k_plaquette, dim3(static_cast<uint32_t>(ns)), dim3(256), 0, stream, fs.ph_par, fs.ph_perp,
                       fs.ls_par, fs.ls_perp, n_par, n_perp, flux + s0 * kps, chern + s0, total + s0, status + s0);
    BE_RET_IF(check_launch(ctx, "plaquette"));
  }
  return BE_OK;
}

}  // namespace

extern "C" int be_plaquette_flux(be_ctx *ctx, const void *U, int32_t N, int32_t m, int32_t ldu, int64_t u_stride,
                                 int32_t n_sys, int32_t n_par, int32_t n_perp, double *flux, int32_t *chern,
                                 double *total, uint32_t *status, hipStream_t stream) {
  using namespace be;
  BE_RET_IF(check_flux_args(ctx, U, N, m, ldu, u_stride, n_sys, n_par, n_perp, flux, chern, total, status));
  if (n_sys == 0) return BE_OK;
  const int64_t kps = int64_t(n_par) * n_perp;
  const int64_t mm = int64_t(std::max(m, 1)) * std::max(m, 1);
  // systems per pass: the links of one direction within about 1 GiB
  const int64_t per = std::max<int64_t>(1, (int64_t(1) << 30) / (kps * mm * int64_t(sizeof(double2))));
  const int64_t spp = std::min<int64_t>(per, n_sys);
  FluxScratch fs;
  Carve cv;
  fs.declare(cv, spp, kps, mm);
  BE_RET_IF(cv.commit(ctx, stream, WS_WILSON));
  return flux_run(ctx, U, N, m, ldu, u_stride, n_sys, n_par, n_perp, flux, chern, total, status, fs, spp, stream);
}

extern "C" int be_plaquette_flux_noalloc(be_ctx *ctx, const void *U, int32_t N, int32_t m, int32_t ldu,
                                         int64_t u_stride, int32_t n_sys, int32_t n_par, int32_t n_perp, double *flux,
                                         int32_t *chern, double *total, uint32_t *status, hipStream_t stream) {
  using namespace be;
  BE_RET_IF(check_flux_args(ctx, U, N, m, ldu, u_stride, n_sys, n_par, n_perp, flux, chern, total, status));
  if (n_sys == 0) return BE_OK;
  void *base = nullptr;
  {
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    base = (ctx->device >= 0 && ctx->device < kMaxDevices) ? g_scratch_ptr[ctx->device] : nullptr;
  }
  if (!base) return set_err(ctx, BE_EHIP, "be_plaquette_flux_noalloc: no scratch address for this device");
  const int64_t kps = int64_t(n_par) * n_perp;
  const int64_t mm = int64_t(std::max(m, 1)) * std::max(m, 1);
  // as many systems per pass as the fixed scratch holds (at least one)
  auto bytes = [&](int64_t spp) {
    FluxScratch f;
    Carve c;
    f.declare(c, spp, kps, mm);
    return c.total();
  };
  const size_t cap = size_t(BE_NOALLOC_SCRATCH_BYTES);
  if (bytes(1) > cap)
    return set_err(ctx, BE_EINVAL, "be_plaquette_flux_noalloc: one system needs " + std::to_string(bytes(1)) +
                                       " bytes of scratch, more than the fixed " + std::to_string(cap));
  int64_t spp = std::min<int64_t>(n_sys, std::max<int64_t>(1, int64_t(cap / bytes(1))));
  while (spp > 1 && bytes(spp) > cap) --spp;
  FluxScratch fs;
  Carve cv;
  fs.declare(cv, spp, kps, mm);
  cv.place(base);
  return flux_run(ctx, U, N, m, ldu, u_stride, n_sys, n_par, n_perp, flux, chern, total, status, fs, spp, stream);
}
