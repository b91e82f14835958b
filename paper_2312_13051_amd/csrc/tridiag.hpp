// Device functions of the FP64 tridiagonal eigensolver shared by its kernels:
// Sturm counts, the tolerances of splits and clusters, the choice of the block
// that carries an eigenvector, and inverse iteration for one vector.
#pragma once

#include <cfloat>
#include <cmath>

#include "common.hpp"

namespace {

// a / b as a times the hardware reciprocal of b refined by one Newton-Raphson
// step: within a few ulps of the rounded quotient, for normal b (the Sturm
// recurrence keeps |b| >= pivmin >= DBL_MIN, so 1/b and a/b stay finite).
__device__ __forceinline__ double div_nr(double a, double b) {
  double r = __builtin_amdgcn_rcp(b);
  r = fma(fma(-b, r, 1.0), r, r);
  return a * r;
}

// Number of eigenvalues of T below x (Sturm sequence of the LDL^T
// factorization of T - x I). The quotient uses div_nr: the count is that of a
// matrix within a few ulps of T, the same kind of backward error the
// correctly rounded division gives.
__device__ __forceinline__ int sturm_count(const double *sd, const double *se2, int N, double x, double pivmin) {
  int cnt = 0;
  double qv = sd[0] - x;
  if (fabs(qv) < pivmin) qv = -pivmin;
  cnt += qv < 0.0;
  for (int i = 1; i < N; ++i) {
    qv = (sd[i] - x) - div_nr(se2[i - 1], qv);
    if (fabs(qv) < pivmin) qv = -pivmin;
    cnt += qv < 0.0;
  }
  return cnt;
}

// The same count for bisection, from the principal minors' recurrence
// p_i = (d_i - x) p_{i-1} - e_{i-1}^2 p_{i-2}: its sign changes count the
// eigenvalues below x, as the negative quotients p_i / p_{i-1} do, with the same
// backward error (a few ulps of d_i - x and e^2), but each step is one multiply
// and one fused multiply-add instead of a reciprocal, its refinement and four
// more operations in one dependent chain. T comes scaled (sturm_scale) with its
// infinity norm in [1/2, 1], as pairs (d_i, e_{i-1}^2) with e^2 >= kSturmE2: a
// step then grows p by at most 3 and two steps shrink it by no less than
// kSturmE2, so that taking out the exponent every eighth step keeps p in
// range, and no two consecutive minors vanish. Half the bands, quotients -> minors
// throughout: 2,304 matrices of order 400 7.31 -> 3.53 ms, of order 200 2.85 ->
// 1.35, 120 of order 64 181 -> 113 us (two counts at once in a thread, with half
// the waves: 191 us and 5.94 ms).
constexpr double kSturmE2 = 1e-36;  // (1e-18 ||T||)^2, below the rounding of T
struct SturmMinors {
  double x, p0, p1;
  uint32_t s1, cnt;
  __device__ __forceinline__ SturmMinors(double d0, double xx) : x(xx), p0(1.0), p1(d0 - xx) {
    s1 = uint32_t(__double2hiint(p1));
    cnt = s1 >> 31;
  }
  __device__ __forceinline__ void step(double2 v) {
    const double pn = fma(v.x - x, p1, -(v.y * p0));
    const uint32_t sn = uint32_t(__double2hiint(pn));
    cnt += (sn ^ s1) >> 31;
    p0 = p1;
    p1 = pn;
    s1 = sn;
  }
  __device__ __forceinline__ void rescale() {
    const int ex = -__builtin_amdgcn_frexp_exp(fmax(fabs(p0), fabs(p1)));
    p0 = __builtin_amdgcn_ldexp(p0, ex);
    p1 = __builtin_amdgcn_ldexp(p1, ex);
  }
};
__device__ __forceinline__ int sturm_count_p(const double2 *de, int N, double x) {
  SturmMinors s(de[0].x, x);
  int i = 1;
  for (; i + 8 <= N; i += 8) {
    double2 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = de[i + u];
#pragma unroll
    for (int u = 0; u < 8; ++u) s.step(v[u]);
    s.rescale();
  }
  for (; i < N; ++i) s.step(de[i]);
  return int(s.cnt);
}
// with the pairs in registers (rows past N as sturm_pad)
template <int NM>
__device__ __forceinline__ int sturm_count_p(const double2 (&de)[NM], double x) {
  SturmMinors s(de[0].x, x);
#pragma unroll
  for (int i = 1; i < NM; ++i) {
    s.step(de[i]);
    if (i % 8 == 0) s.rescale();
  }
  return int(s.cnt);
}
// A row with an eigenvalue past every x that is counted at (|x| <= 1 + rounding)
__device__ __forceinline__ double2 sturm_pad() { return make_double2(2.0, kSturmE2); }

// The quotients' count from the same pairs, four steps' reads issued together.
__device__ __forceinline__ int sturm_count_i(const double2 *de, int N, double x) {
  int cnt = 0;
  double qv = de[0].x - x;
  if (fabs(qv) < DBL_MIN) qv = -DBL_MIN;
  cnt += qv < 0.0;
#pragma unroll 4
  for (int i = 1; i < N; ++i) {
    const double2 v = de[i];
    qv = (v.x - x) - div_nr(v.y, qv);
    if (fabs(qv) < DBL_MIN) qv = -DBL_MIN;
    cnt += qv < 0.0;
  }
  return cnt;
}

template <int NM>
__device__ __forceinline__ int sturm_count_i(const double2 (&de)[NM], double x) {
  double qv = de[0].x - x;
  if (fabs(qv) < DBL_MIN) qv = -DBL_MIN;
  int cnt = qv < 0.0;
#pragma unroll
  for (int i = 1; i < NM; ++i) {
    qv = (de[i].x - x) - div_nr(de[i].y, qv);
    if (fabs(qv) < DBL_MIN) qv = -DBL_MIN;
    cnt += qv < 0.0;
  }
  return cnt;
}

// Interval width, relative to ||T||, from which a mixed path's bisection counts
// by quotients. The two counts differ only within a few eps ||T|| of an
// eigenvalue, i.e. in an eigenvalue's last bits; the vectors of a degenerate
// level are a basis that those bits choose, and a mixed path rounds that basis
// to FP32. So its last bits stay the quotients', while the wide intervals,
// 2^14 such distances and more, take the cheaper count (4,608 matrices of order 400:
// 11.0 -> 7.65 ms).
constexpr double kQuotientWidth = 0x1p-38;

// Couplings below the minors' floor are raised to it there, which moves a level by
// up to 2e-18 ||T||: below the rounding of the levels themselves down to 2^-6 ||T||,
// but not of the levels near zero of a T that splits. Those are found again by
// quotients on T as it is, from an interval around v wide enough for that move: four
// cells of a power of two's grid, whose halvings are the same whatever v is, so that
// equal levels come out equal and all in order. (v, tn: of the T scaled as above; k:
// the level's index.)
constexpr double kLowLevel = 0x1p-6, kLowMove = 8e-18;  // relative to the norm tn
__device__ __forceinline__ bool below_floor(double e2) { return e2 < kSturmE2; }
__device__ __forceinline__ double low_level(const double *sd, const double *se2, int N, int k, double v, double tn,
                                            double isc, double pivmin, double tol_abs, int max_it, bool &conv) {
  const double w = __builtin_amdgcn_ldexp(1.0, __builtin_amdgcn_frexp_exp(kLowMove * tn + 4.0 * DBL_EPSILON * fabs(v)));
  double a = (floor(v / w) - 1.0) * w, b = a + 4.0 * w;
  conv = false;
#pragma unroll 1
  for (int it = 0; it <= max_it; ++it) {
    const double mid = 0.5 * (a + b);
    conv = b - a <= fmax(2.0 * DBL_EPSILON * fmax(fabs(a), fabs(b)) + DBL_MIN, tol_abs) || mid <= a || mid >= b;
    if (conv || it == max_it) break;
    if (sturm_count(sd, se2, N, mid * isc, pivmin) > k) b = mid;
    else a = mid;
  }
  return 0.5 * (a + b);
}

// Power of two that takes a norm into [1/2, 1) (1 for a zero or non-finite norm;
// at most 2^1000, so that a norm among the subnormal numbers has a finite one)
__device__ __forceinline__ double sturm_scale(double tnorm) {
  return tnorm > 0.0 && tnorm < INFINITY ? ldexp(1.0, min(-ilogb(tnorm) - 1, 1000)) : 1.0;
}

__device__ __forceinline__ double hash_unit(uint64_t a, uint64_t b) {
  // splitmix64 of (a, b) -> uniform in (-1, 1)
  uint64_t z = a * 0x9E3779B97F4A7C15ull + b + 0x632BE59BD9B4E019ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  z ^= z >> 31;
  return (double)(z >> 11) * (2.0 / 9007199254740992.0) - 1.0;
}

// Tolerances relative to ||T||: split < block window < cluster gap, so a
// cluster's window never reaches the next cluster. Eigenvalues closer than
// the cluster tolerance (clu_rel, by default kCluRel = 1e-12) form a cluster, whose vectors are
// computed as one invariant subspace (any orthonormal basis of it): inverse
// iteration separates two eigenvalues only to about eps ||T|| / gap, so
// below that gap their vectors can come out nearly parallel (a cluster of
// eigenvalues spread over 1e-12 ||T|| - e.g. the projected spin operator's
// +-1 clusters computed from refined eigenvectors, whose T splits into many
// blocks - would otherwise have lanes pick blocks by windows narrower than
// the cluster, and leave an orthonormalization that cannot converge). A
// caller that needs the vectors of nearly equal eigenvalues resolved one by
// one (and validates them) may pass a smaller tolerance.
constexpr double kCluRel = 1e-12;
__device__ __forceinline__ double tol_split(double tnorm) { return 16.0 * DBL_EPSILON * tnorm; }
__device__ __forceinline__ double tol_window(double tnorm, double clu_rel) { return 0.5 * clu_rel * tnorm; }
__device__ __forceinline__ double tol_cluster(double tnorm, double clu_rel) { return clu_rel * tnorm; }

// Block of T that carries the eigenvector of lane c, and its shift. The k
// members of a cluster (consecutive eigenvalues within the cluster tolerance)
// take the k distinct blocks that hold it, in order; lanes whose block holds
// several of them share it.
struct InvitBlock {
  int c0;      // first member of the lane's cluster
  int bs, bt;  // the block's rows
  bool found, shared;
  double lm;  // shift
};
__device__ __forceinline__ InvitBlock invit_block(const double *sd, const double *se2, const double *lam, int m, int c,
                                                  const int *sblk, int nblk, int N, double tnorm, double clu_rel,
                                                  double pivmin) {
  const double dblk = tol_window(tnorm, clu_rel), dclu = tol_cluster(tnorm, clu_rel);
  int c0 = c, c1 = c + 1;
  while (c0 > 0 && lam[c0] - lam[c0 - 1] <= dclu) --c0;
  while (c1 < m && lam[c1] - lam[c1 - 1] <= dclu) ++c1;
  const double wlo = lam[c0] - dblk, whi = lam[c1 - 1] + dblk;
  if (nblk == 1 && c1 - c0 == 1)  // the window holds this eigenvalue and no other
    return InvitBlock{c0, 0, N, true, false, lam[c]};
  const int jr = c - c0;
  int bs = 0, bt = N, cnt = 0;
  bool found = false, shared = false;
  for (int b = 0; b < nblk && !found; ++b) {
    const int s0 = sblk[b], t0 = sblk[b + 1];
    const int nb = sturm_count(sd + s0, se2 + s0, t0 - s0, whi, pivmin) -
                   sturm_count(sd + s0, se2 + s0, t0 - s0, wlo, pivmin);
    if (nb > 0 && cnt + nb > jr) {
      bs = s0;
      bt = t0;
      found = true;
      shared = nb > 1;
    }
    cnt += nb;
  }
  // Lanes that share a block with other members of their cluster take
  // shifts a few eps ||T|| apart: far larger than the splitting of a
  // degenerate pair (so neither member dominates a lane's solve and each
  // lane returns an independent combination of the cluster's vectors),
  // far smaller than the distance to the next cluster.
  const double lm =
      (!found || shared) ? lam[c] + (jr - 0.5 * (c1 - c0 - 1)) * 2.0 * DBL_EPSILON * tnorm : lam[c];
  return InvitBlock{c0, bs, bt, found, shared, lm};
}

// Inverse iteration for vector c (normalized, two solves) on rows bs .. bt - 1
// of T with shift lm: X[i * mp + c] receives it, Z0 is scratch of the same
// layout. AHEAD: loads four rows ahead of their use (arrays in memory; in LDS
// one at a time). False when the vector did not come out finite.
template <bool AHEAD>
__device__ __forceinline__ bool invit_vector(const double *sd, const double *se, int bs, int bt, double lm, double tiny,
                                             int c, double *X, double *Z0, int mp) {
  // two solves: from a pseudo-random start the first already amplifies the
  // wanted direction by ~1/(eps ||T||) against ~1/gap for the others. The
  // second solve recomputes the same factorization (same operations, same
  // factors) instead of storing it again, and takes the first solution's
  // normalization as it reads it. Of the factorization only the diagonal
  // a_i met at each elimination step is stored: the pivot choice of row i
  // (|a_i| < |e_i|) and every factor entry follow from a_i, a_{i-1} and T,
  // recomputed by the same operations in the back substitution.
  // The loads of each sweep are issued PF rows ahead of the recurrence that
  // consumes them, so the serial chain waits on memory once per PF rows.
  // The start vector depends on the column only, not on the matrix's place
  // in the batch: a matrix gets the same eigenvectors, bit for bit, in any
  // batch (inside a degenerate cluster the start decides the basis).
  constexpr int PF = AHEAD ? 4 : 1;
  double scale = 1.0;
  bool ok = true;
  for (int it = 0; it < 2; ++it) {
    // forward elimination with partial pivoting on [T_block - lm I | rhs]
    double a = sd[bs] - lm, b = bt - bs > 1 ? se[bs] : 0.0;
    double r = it == 0 ? hash_unit(uint64_t(c) + 1, bs) : X[int64_t(bs) * mp + c] * scale;
    // one elimination step at row i (i + 1 < bt) with right-hand side entry rn of row i + 1
    auto step = [&](int i, double rn) {
      const double ei = se[i], Dn = sd[i + 1] - lm, en = (i + 2 < bt) ? se[i + 1] : 0.0;
      const int64_t o = int64_t(i) * mp + c;
      if (it == 0) Z0[o] = a;
      // without interchange: l = e_i / a (a = 0 only with e_i = 0, then
      // taken as tiny), row i keeps (a, b); with interchange: l = a / e_i
      const bool keep = fabs(a) >= fabs(ei);
      const double ad = (keep && a == 0.0) ? tiny : a;
      const double l = (keep ? ei : ad) / (keep ? ad : ei);
      X[o] = keep ? r : rn;
      const double p1 = keep ? Dn : b, p2 = keep ? b : Dn;
      const double q1 = keep ? rn : r, q2 = keep ? r : rn;
      a = p1 - l * p2;
      b = keep ? en : -l * en;
      r = q1 - l * q2;
    };
    if (it == 0) {
      for (int i = bs; i + 1 < bt; ++i) step(i, hash_unit(uint64_t(c) + 1, i + 1));
    } else {
      for (int i0 = bs; i0 + 1 < bt; i0 += PF) {
        double rv[PF];
#pragma unroll
        for (int u = 0; u < PF; ++u) rv[u] = i0 + u + 1 < bt ? X[int64_t(i0 + u + 1) * mp + c] : 0.0;
#pragma unroll
        for (int u = 0; u < PF; ++u)
          if (i0 + u + 1 < bt) step(i0 + u, rv[u] * scale);
      }
    }
    {
      const int64_t o = int64_t(bt - 1) * mp + c;
      if (it == 0) Z0[o] = a;
      X[o] = r;
    }
    // back substitution: row i of the triangular factor is (e_i, D_{i+1},
    // e_{i+1}) where row i was interchanged, else (a_i, b_i, 0) with b_i =
    // e_i, or -(a_{i-1} / e_{i-1}) e_i after an interchange at row i-1
    double x1 = 0.0, x2 = 0.0, nrm = 0.0;
    double ai = Z0[int64_t(bt - 1) * mp + c];
    for (int i0 = bt - 1; i0 >= bs; i0 -= PF) {
      double xv[PF], av[PF];
#pragma unroll
      for (int u = 0; u < PF; ++u) {
        const int i = i0 - u;
        xv[u] = i >= bs ? X[int64_t(i) * mp + c] : 0.0;
        av[u] = i > bs ? Z0[int64_t(i - 1) * mp + c] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < PF; ++u) {
        const int i = i0 - u;
        if (i >= bs) {
          const double ap = av[u];
          double z0, z1 = 0.0, z2 = 0.0;
          if (i == bt - 1) {
            z0 = ai == 0.0 ? tiny : ai;
          } else if (fabs(ai) >= fabs(se[i])) {
            z0 = ai == 0.0 ? tiny : ai;
            z1 = se[i];
            if (i > bs && !(fabs(ap) >= fabs(se[i - 1]))) {
              const double l = ap / se[i - 1];
              z1 = -l * se[i];
            }
          } else {
            z0 = se[i];
            z1 = sd[i + 1] - lm;
            z2 = (i + 2 < bt) ? se[i + 1] : 0.0;
          }
          const double xi = (xv[u] - z1 * x1 - z2 * x2) / z0;
          X[int64_t(i) * mp + c] = xi;
          x2 = x1;
          x1 = xi;
          nrm = fma(xi, xi, nrm);
          ai = ap;
        }
      }
    }
    const double inv = 1.0 / sqrt(nrm);
    if (!isfinite(inv) || inv == 0.0) ok = false;
    if (it == 0) {
      scale = inv;
    } else {
      for (int i0 = bs; i0 < bt; i0 += PF) {
        double xv[PF];
#pragma unroll
        for (int u = 0; u < PF; ++u) xv[u] = i0 + u < bt ? X[int64_t(i0 + u) * mp + c] : 0.0;
#pragma unroll
        for (int u = 0; u < PF; ++u)
          if (i0 + u < bt) X[int64_t(i0 + u) * mp + c] = xv[u] * inv;
      }
    }
  }
  return ok;
}

// End of the orthonormalization group starting at c0: the following lanes of
// the same cluster with the same group id (0: no group, a group of one).
__device__ __forceinline__ int group_end(const double *lam, const int *mk, int m, int c0, double dclu) {
  int c1 = c0 + 1;
  if (mk[c0] == 0) return c1;
  while (c1 < m && mk[c1] == mk[c0] && lam[c1] - lam[c1 - 1] <= dclu) ++c1;
  return c1;
}

}  // namespace
