// Householder reduction of Hermitian matrices that fit one compute unit, FP64.
//
// The panel kernel streams the trailing matrix from memory once per column
// (and the panel's V and W twice). A matrix of order 192 is 295 KB as a
// triangle: it fits the 512 KB of a compute unit's registers. Here a workgroup
// of 512 threads holds the triangle there for the whole reduction, multiplies
// it with each reflector and applies the rank-2 update at once: no panel, no
// V and W, no separate trailing update, four barriers per column.
//
// Thread (tx, ty), tx < 32, ty < 16, holds the elements (32 a + tx, 16 b + ty)
// of the blocks that reach the lower triangle (b <= 2 a + 1), zeros above the
// diagonal. A column belongs to one half-wave, so column sums need lane moves
// only; a row is spread over the 16 half-waves, whose partial sums meet in LDS.
// Orders past 192 keep their first columns (up to 24) in LDS.
// Bound by the latency of the column's chain (norm, square root and reciprocals,
// product, combination, update: 2.6 us a column at order 64, 5.3 at 192, of
// which the FP64 arithmetic is a third). Panel kernel and trailing update ->
// this kernel and larft: order 64, 120 matrices 793 -> 205 us; 128, 2,048: 9.46
// -> 4.09 ms; 200, 2,304: 30.4 -> 12.9 ms; the last 208 columns of 2,304 matrices
// of order 400: 27 -> 13 ms. Up to order 96 two matrices share a compute unit.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "common.hpp"
#include "hetrd_resident.hpp"
#include "lanes.hpp"

namespace {

constexpr int RT = 512, RWV = RT / 64;  // threads and waves

// Workgroup barrier that orders LDS accesses only: __syncthreads would also wait
// for the reflector's stores to memory, which nothing in the loop reads back.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Index of block (a, b), b <= 2 a + 1, among a thread's elements: by columns b
__host__ __device__ constexpr int blk(int NA, int a, int b) {
  int k = 0;
  for (int c = 0; c < b; ++c) k += NA - c / 2;
  return k + a - b / 2;
}

constexpr int kStrip = 24;  // columns in LDS, at most (orders past 192)

// Rows of the kernel's vectors in LDS
__host__ __device__ constexpr int resident_rows(int NA) { return 32 * NA + (NA == 6 ? kStrip : 0); }

// LDS in double2: column j, u, v, w and the strip's row and column sums (NX
// each), the block's column sums (32 NA), row partials (RWV x NA x 32), the
// wave sums of u^H A u (RWV doubles), and the strip (S n).
__host__ __device__ inline int resident_lds(int NA, int S, int n) {
  return 6 * resident_rows(NA) + 32 * NA + RWV * NA * 32 + RWV / 2 + S * n;
}

template <int NA, int GB>
__global__ __launch_bounds__(RT, NA <= 3 ? 4 : 2) void hetrd_resident_kernel(double2 *A, int64_t sA, int lda, int N,
                                                                              int p0, int S, double *d, double *e,
                                                                              int64_t sDE, double2 *taus) {
  extern __shared__ double2 sm[];
  constexpr int NX = resident_rows(NA);
  const int n = N - p0, nb = n - S;
  double2 *const sx = sm, *const su = sm + NX, *const sv = sm + 2 * NX, *const sw = sm + 3 * NX, *const yS = sm + 4 * NX,
          *const yK = sm + 5 * NX, *const yC = sm + 6 * NX;
  double *const part = reinterpret_cast<double *>(yC + 32 * NA);  // [wave][a][64]
  double *sq = part + RWV * NA * 64;
  double2 *strip = reinterpret_cast<double2 *>(sq + RWV);  // column k at k n
  const int64_t q = blockIdx.x;
  double2 *Aq = A + q * sA + p0 + int64_t(p0) * lda;  // element (0, 0) of the trailing matrix
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tx = lane & 31, ty = 2 * wave + (lane >> 5);
  // element against the diagonal in blocks b = 2 a and b = 2 a + 1
  const bool on0 = tx == ty, on1 = tx == ty + 16, up0 = tx < ty, up1 = tx < ty + 16;

  double2 m[NA * (NA + 1)];
  double mx = 0.0;
  unrolled<2 * NA>([&](auto B) {
    constexpr int b = B, a0 = b / 2;
    unrolled<NA - a0>([&](auto D) {
      constexpr int a = a0 + D;
      const int i = 32 * a + tx, k = 16 * b + ty;
      double2 v = make_double2(0.0, 0.0);
      if (i < nb && k <= i) v = Aq[S + i + int64_t(S + k) * lda];
      if (i == k) v.y = 0.0;
      m[blk(NA, a, b)] = v;
      mx = fmax(mx, fmax(fabs(v.x), fabs(v.y)));
      if (b == 0 && S == 0 && ty == 0) sx[i] = v;
    });
  });
  for (int t = tid; t < S * n; t += RT) {
    const int k = t / n, i = t - k * n;
    double2 v = make_double2(0.0, 0.0);
    if (i >= k) v = Aq[i + int64_t(k) * lda];
    if (i == k) v.y = 0.0;
    mx = fmax(mx, fmax(fabs(v.x), fabs(v.y)));
    strip[t] = v;
  }
  for (int i = tid; i < NX; i += RT) yS[i] = make_double2(0.0, 0.0);
  mx = fold_max<16>(fold_max<32>(mx));
  mx = fmax(mx, lane_xor<8>(mx));
  mx = fmax(mx, lane_xor<4>(mx));
  mx = fmax(mx, lane_xor<2>(mx));
  mx = fmax(mx, lane_xor<1>(mx));
  if (lane == 0) sq[wave] = mx;
  __syncthreads();
  // Products of three factors of u, A and u below would leave the range of FP64 for
  // matrices of norm 1e103 or 1e-105: one that far from one is reduced scaled by a
  // power of two (d and e are scaled back). A column of norm below 2^-450 then counts
  // as zero: the square of scal would leave the range, and leaving it out changes the
  // matrix by 2^-350 of its norm at most.
  for (int w2 = 0; w2 < RWV; ++w2) mx = fmax(mx, sq[w2]);
  const int ex = __builtin_amdgcn_frexp_exp(mx);  // 0 for zero and non-finite values
  const int sh = ex > 100 || ex < -100 ? -ex : 0;
  if (sh != 0) {
    unrolled<2 * NA>([&](auto B) {
      constexpr int b = B, a0 = b / 2;
      unrolled<NA - a0>([&](auto D) {
        constexpr int a = a0 + D;
        double2 &v = m[blk(NA, a, b)];
        v = make_double2(__builtin_amdgcn_ldexp(v.x, sh), __builtin_amdgcn_ldexp(v.y, sh));
        if (b == 0 && S == 0 && ty == 0) sx[32 * a + tx] = v;
      });
    });
    for (int t = tid; t < S * n; t += RT)
      strip[t] = make_double2(__builtin_amdgcn_ldexp(strip[t].x, sh), __builtin_amdgcn_ldexp(strip[t].y, sh));
    __syncthreads();
  }
  if (S > 0 && tid < n) sx[tid] = strip[tid];  // column 0 (else written with the loads)
  __syncthreads();
  for (int j = 0; j + 1 < n; ++j) {
    // ---- reflector of column j (every wave by itself); u = x - beta e_{j+1}, v = scal u
    double xn = 0.0;
    for (int i = j + 2 + lane; i < n; i += 64) {
      const double2 x = sx[i];
      xn = fma(x.x, x.x, fma(x.y, x.y, xn));
    }
    xn = wave_sum(xn);
    const double2 alpha = sx[j + 1];
    double2 tau = make_double2(0.0, 0.0), scal = tau, ub = tau;
    double beta = alpha.x;
    const double nn = alpha.x * alpha.x + alpha.y * alpha.y + xn;
    if ((xn != 0.0 || alpha.y != 0.0) && !(nn < 0x1p-900)) {
      const double nrm = sqrt(nn);
      beta = alpha.x >= 0.0 ? -nrm : nrm;
      tau = make_double2((beta - alpha.x) / beta, -alpha.y / beta);
      ub = make_double2(alpha.x - beta, alpha.y);
      const double den = ub.x * ub.x + ub.y * ub.y;
      scal = make_double2(ub.x / den, -ub.y / den);
    }
    if (tid < NX) {
      double2 u = make_double2(0.0, 0.0);
      if (tid > j && tid < n) u = tid == j + 1 ? ub : sx[tid];
      su[tid] = u;
    }
    lds_barrier();
    // ---- y = A u: row sums per thread, column sums per half-wave, and u^H A u
    double qs = 0.0;
    {
      double2 ui[NA], yr[NA];
#pragma unroll
      for (int a = 0; a < NA; ++a) {
        ui[a] = su[S + 32 * a + tx];
        yr[a] = make_double2(0.0, 0.0);
      }
      // column blocks GB at a time: their LDS reads and lane sums overlap
      unrolled<(2 * NA + GB - 1) / GB>([&](auto BG) {
        constexpr int b0 = BG * GB;
        if (S + 16 * (b0 + GB - 1) + 15 <= j) return;  // columns all reduced (uniform)
        double2 uk[GB], yc[GB];
        unrolled<GB>([&](auto V) {
          if constexpr (b0 + V < 2 * NA) uk[V] = su[S + 16 * (b0 + V) + ty];
          yc[V] = make_double2(0.0, 0.0);
        });
        unrolled<NA>([&](auto Ar) {
          unrolled<GB>([&](auto V) {
            constexpr int a = Ar, b = b0 + V, a0 = b / 2;
            if constexpr (b < 2 * NA && a >= a0) {
              const double2 x = m[blk(NA, a, b)];
              double2 c = ui[a];
              yr[a].x = fma(x.x, uk[V].x, fma(-x.y, uk[V].y, yr[a].x));
              yr[a].y = fma(x.x, uk[V].y, fma(x.y, uk[V].x, yr[a].y));
              if (a == a0 && (b % 2 ? on1 : on0)) {  // the diagonal is in the row part
                qs -= (c.x * c.x + c.y * c.y) * x.x;
                c = make_double2(0.0, 0.0);
              }
              yc[V].x = fma(x.x, c.x, fma(x.y, c.y, yc[V].x));
              yc[V].y = fma(x.x, c.y, fma(-x.y, c.x, yc[V].y));
            }
          });
        });
        // sums over the 32 lanes of a half-wave: rows of 16 lanes hold the real
        // and the imaginary part, then each exchange halves the columns a lane holds
        double t[GB];
        unrolled<GB>([&](auto V) { t[V] = fold<16>(yc[V].x, yc[V].y); });
        if constexpr (GB == 4) {
          const bool up = (lane & 4) != 0;
          unrolled<2>([&](auto V) {
            const double keep = up ? t[V + 2] : t[V], send = up ? t[V] : t[V + 2];
            t[V] = keep + lane_xor<4>(send);
          });
        }
        {
          const bool up = (lane & 8) != 0;
          const double keep = up ? t[1] : t[0], send = up ? t[0] : t[1];
          t[0] = keep + lane_xor<8>(send);
        }
        if constexpr (GB == 2) t[0] += lane_xor<4>(t[0]);
        t[0] += lane_xor<2>(t[0]);
        t[0] += lane_xor<1>(t[0]);
        const int c = GB == 4 ? ((lane >> 3) & 1) + ((lane >> 2) & 1) * 2 : (lane >> 3) & 1;  // column of the group
        if ((lane & (GB == 4 ? 3 : 7)) == 0 && b0 + c < 2 * NA)
          reinterpret_cast<double *>(yC + 16 * (b0 + c) + ty)[(lane >> 4) & 1] = t[0];
      });
#pragma unroll
      for (int a = 0; a < NA; ++a) {
        qs += 2.0 * (ui[a].x * yr[a].x + ui[a].y * yr[a].y);
        if (S + 32 * a + 31 > j) part[(wave * NA + a) * 64 + lane] = fold<32>(yr[a].x, yr[a].y);
      }
    }
    if (j + 1 < S) {  // the strip's columns: a thread per row, a wave per column
      if (tid < n) {
        const int i = tid;
        double2 y = make_double2(0.0, 0.0);
        const double2 c = su[i];
        for (int k = j + 1; k <= min(i, S - 1); ++k) y = be::cadd(y, be::cmul(strip[k * n + i], su[k]));
        yS[i] = y;
        qs += 2.0 * (c.x * y.x + c.y * y.y);
        if (i > j && i < S) qs -= (c.x * c.x + c.y * c.y) * strip[i * n + i].x;
      }
      for (int k = j + 1 + wave; k < S; k += RWV) {
        double2 y = make_double2(0.0, 0.0);
        for (int i = k + 1 + lane; i < n; i += 64) y = be::cadd(y, be::cmulc(strip[k * n + i], su[i]));
        y.x = wave_sum(y.x);
        y.y = wave_sum(y.y);
        if (lane == 0) yK[k] = y;
      }
    }
    qs = wave_sum(qs);
    if (lane == 0) sq[wave] = qs;
    lds_barrier();
    // ---- v and w = tau y - (tau y)^H v / 2 tau v; v^H A v is real, so the last factor is too
    if (tid < NX) {
      const int i = tid;
      double2 v = make_double2(0.0, 0.0), w = v;
      if (i > j && i < n) {
        double2 y = make_double2(0.0, 0.0);
        if (i >= S) {
          const int r = i - S;
          y = yC[r];
          const double *pr = part + (r >> 5) * 64 + (r & 31);
#pragma unroll
          for (int w2 = 0; w2 < RWV; ++w2) {
            y.x += pr[w2 * NA * 64];
            y.y += pr[w2 * NA * 64 + 32];
          }
        } else {
          y = yK[i];
        }
        if (j + 1 < S) y = be::cadd(y, yS[i]);
        double qq = 0.0;
#pragma unroll
        for (int w2 = 0; w2 < RWV; ++w2) qq += sq[w2];
        v = i == j + 1 ? make_double2(1.0, 0.0) : be::cmul(su[i], scal);
        const double al = -0.5 * (tau.x * tau.x + tau.y * tau.y) * (scal.x * scal.x + scal.y * scal.y) * qq;
        w = be::cmul(be::cmul(tau, scal), y);
        w.x = fma(al, v.x, w.x);
        w.y = fma(al, v.y, w.y);
      }
      sv[i] = v;
      sw[i] = w;
      if (i < n) Aq[i + int64_t(j) * lda] = v;
    }
    for (int r = tid; r < p0; r += RT) Aq[r - p0 + int64_t(j) * lda] = make_double2(0.0, 0.0);
    if (tid == 0) {
      d[q * sDE + p0 + j] = __builtin_amdgcn_ldexp(sx[j].x, -sh);
      e[q * sDE + p0 + j] = __builtin_amdgcn_ldexp(beta, -sh);
      taus[q * N + p0 + j] = tau;
    }
    lds_barrier();
    // ---- A -= v w^H + w v^H; the next column goes to sx
    {
      const int jn = j + 1 - S, jb = jn >> 4;  // its index in the register block
      const bool mine = jn >= 0 && ty == (jn & 15);
      double2 vi[NA], wi[NA];
#pragma unroll
      for (int a = 0; a < NA; ++a) {
        vi[a] = sv[S + 32 * a + tx];
        wi[a] = sw[S + 32 * a + tx];
      }
      unrolled<NA>([&](auto BG) {
        constexpr int b0 = 2 * BG;
        if (S + 16 * b0 + 31 <= j) return;
        double2 vk[2], wk[2];
        unrolled<2>([&](auto V) {
          vk[V] = sv[S + 16 * (b0 + V) + ty];
          wk[V] = sw[S + 16 * (b0 + V) + ty];
        });
        unrolled<NA>([&](auto Ar) {
          unrolled<2>([&](auto V) {
            constexpr int a = Ar, b = b0 + V, a0 = b / 2;
            if constexpr (a >= a0) {
              double2 x = m[blk(NA, a, b)];
              x.x = fma(-vi[a].x, wk[V].x, fma(-vi[a].y, wk[V].y, fma(-wi[a].x, vk[V].x, fma(-wi[a].y, vk[V].y, x.x))));
              x.y = fma(-vi[a].y, wk[V].x, fma(vi[a].x, wk[V].y, fma(-wi[a].y, vk[V].x, fma(wi[a].x, vk[V].y, x.y))));
              if (a == a0) {
                if (b % 2 ? up1 : up0) x = make_double2(0.0, 0.0);
                if (b % 2 ? on1 : on0) x.y = 0.0;
              }
              m[blk(NA, a, b)] = x;
              if (b == jb && mine) sx[S + 32 * a + tx] = x;  // rows above the column's diagonal are not used
            }
          });
        });
      });
      if (j + 1 < S && tid > j && tid < n) {
        const int i = tid;
        const double2 v = sv[i], w = sw[i];
        for (int k = j + 1; k <= min(i, S - 1); ++k) {
          double2 x = be::csub(strip[k * n + i], be::cadd(be::cmulc(sw[k], v), be::cmulc(sv[k], w)));
          if (i == k) x.y = 0.0;
          strip[k * n + i] = x;
          if (k == j + 1) sx[i] = x;
        }
      }
    }
    lds_barrier();
  }
  // last column: no reflector
  if (tid == 0) {
    d[q * sDE + N - 1] = __builtin_amdgcn_ldexp(sx[n - 1].x, -sh);
    taus[q * N + N - 1] = make_double2(0.0, 0.0);
  }
  for (int r = tid; r < N; r += RT) Aq[r - p0 + int64_t(n - 1) * lda] = make_double2(0.0, 0.0);
}

// Compact-WY factor of a panel of reflectors (H_0 .. H_{nb-1} = I - V T V^H):
// T(0:j, j) = -tau_j T(0:j, 0:j) (V^H v_j)(0:j), T(j, j) = tau_j. One workgroup
// per panel and matrix; V^H V from row tiles staged in LDS.
constexpr int LB = 32;
__global__ __launch_bounds__(256) void larft_kernel(const double2 *A, int64_t sA, int lda, int N, int p_first,
                                                    const double2 *taus, double2 *Tm, int64_t sT) {
  __shared__ double2 tile[LB][LB + 1], G[LB][LB + 1], T[LB][LB + 1];
  const int p = p_first + blockIdx.x, c0 = p * LB, nbp = min(LB, N - c0);
  const int64_t q = blockIdx.y;
  const double2 *Aq = A + q * sA + int64_t(c0) * lda;
  const int tid = threadIdx.x;
  double2 acc[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) acc[u] = make_double2(0.0, 0.0);
  const int c2 = tid >> 3, cb = (tid & 7) * 4;  // column pair (cb + u, c2)
  for (int r0 = c0 + 1; r0 < N; r0 += LB) {
    for (int t = tid; t < LB * LB; t += 256) {
      const int r = t % LB, c = t / LB;
      tile[r][c] = (r0 + r < N && c < nbp) ? Aq[r0 + r + int64_t(c) * lda] : make_double2(0.0, 0.0);
    }
    __syncthreads();
    if (cb < c2)
      for (int r = 0; r < LB; ++r) {
        const double2 v = tile[r][c2];
#pragma unroll
        for (int u = 0; u < 4; ++u) acc[u] = be::cadd(acc[u], be::cmulc(tile[r][cb + u], v));
      }
    __syncthreads();
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) G[cb + u][c2] = acc[u];
  for (int t = tid; t < LB * LB; t += 256) T[t % LB][t / LB] = make_double2(0.0, 0.0);
  __syncthreads();
  for (int j = 0; j < nbp; ++j) {
    const double2 tau = taus[q * N + c0 + j];
    if (tid < j) {
      double2 x = make_double2(0.0, 0.0);
      for (int c = tid; c < j; ++c) x = be::cadd(x, be::cmul(T[tid][c], G[c][j]));
      x = be::cmul(tau, x);
      T[tid][j] = make_double2(-x.x, -x.y);
    }
    if (tid == j) T[j][j] = tau;
    __syncthreads();
  }
  double2 *Tq = Tm + q * sT + int64_t(p) * LB * LB;
  for (int t = tid; t < LB * LB; t += 256) Tq[t] = T[t % LB][t / LB];
}

typedef void (*ResidentFn)(double2 *, int64_t, int, int, int, int, double *, double *, int64_t, double2 *);

// The kernel for order n and its strip: rows and columns held in registers in steps of 32
ResidentFn resident_fn(int n, int *S, int *NA) {
  *NA = std::min(6, std::max(2, (n + 31) / 32));
  *S = std::max(0, n - 192);
  switch (*NA) {
    case 2: return &hetrd_resident_kernel<2, 4>;
    case 3: return &hetrd_resident_kernel<3, 2>;
    case 4: return &hetrd_resident_kernel<4, 4>;
    case 5: return &hetrd_resident_kernel<5, 2>;
    default: return &hetrd_resident_kernel<6, 2>;
  }
}

}  // namespace

namespace be {

int hetrd_resident(be_ctx *ctx, double2 *H, int64_t ms, int ld, int N, int p0, int64_t n_mat, double *d, double *e,
                   int64_t sDE, double2 *tau, hipStream_t stream) {
  int S = 0, NA = 0;
  ResidentFn fn = resident_fn(N - p0, &S, &NA);
  const size_t lds = size_t(resident_lds(NA, S, N - p0)) * sizeof(double2);
  if (lds > 65536)
    BE_HIP_TRY(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(fn), hipFuncAttributeMaxDynamicSharedMemorySize,
                                        int(lds)));
  ProfScope prof(ctx, "hetrd_resident", stream);
  hipLaunchKernelGGL(fn, dim3(static_cast<uint32_t>(n_mat)), dim3(RT), lds, stream, H, ms, ld, N, p0, S, d, e, sDE, tau);
  return check_launch(ctx, "hetrd_resident");
}

int larft(be_ctx *ctx, const double2 *H, int64_t ms, int ld, int N, int p_first, int64_t n_mat, const double2 *tau,
          double2 *Tm, int64_t sT, hipStream_t stream) {
  ProfScope prof(ctx, "larft", stream);
  hipLaunchKernelGGL(larft_kernel, dim3(static_cast<uint32_t>((N + LB - 1) / LB - p_first), static_cast<uint32_t>(n_mat)),
                     dim3(256), 0, stream, H, ms, ld, N, p_first, tau, Tm, sT);
  return check_launch(ctx, "larft");
}

int64_t resident_slots(be_ctx *ctx, int n) {
  int S = 0, NA = 0, per_cu = 0;
  ResidentFn fn = resident_fn(n, &S, &NA);
  const size_t lds = size_t(resident_lds(NA, S, n)) * sizeof(double2);
  if (lds > 65536 && hipFuncSetAttribute(reinterpret_cast<const void *>(fn), hipFuncAttributeMaxDynamicSharedMemorySize,
                                         int(lds)) != hipSuccess)
    (void)hipGetLastError();
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void *>(fn), RT, lds) != hipSuccess) {
    (void)hipGetLastError();
    per_cu = 0;
  }
  return int64_t(std::max(per_cu, 1)) * ctx->n_cu;
}

}  // namespace be
