// Rows (a1) and (a2): hopping list -> device plan -> Bloch Hamiltonians.
//
// The host packer merges duplicate keys, checks Hermiticity and keeps the
// upper triangle grouped into (row, col) pairs, sorted by column then row,
// so that consecutive threads of the scatter kernel write consecutive rows of
// one column. The device side is two kernels per call: a zero fill of every
// matrix and a phase-weighted scatter with one thread per (pair, matrix):
//   H[r, c] = sum_e t_e exp(2 pi i kappa . R_e),  H[c, r] = conj(H[r, c]).
// The diagonal is written with an exactly zero imaginary part, so H is
// bitwise Hermitian, and each element is summed by one thread in a fixed
// order, so the result is deterministic.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <memory>
#include <type_traits>
#include <utility>

#include "common.hpp"
#include "hk_pack.hpp"

static_assert(sizeof(be::hkpack::PairRC) == sizeof(int2) && sizeof(be::hkpack::EntR) == sizeof(int4) &&
                  sizeof(be::hkpack::EntT) == sizeof(double2),
              "packed host arrays are uploaded as int2 / int4 / double2");

struct be_hk_plan {
  int device = 0;
  int n_sys = 0;
  std::vector<int32_t> N;        // per system
  std::vector<int32_t> dim;      // per system
  std::vector<int64_t> pair_off; // per system, into pair arrays
  std::vector<int32_t> n_pairs;  // per system
  int64_t total_pairs = 0;
  int64_t total_ents = 0;
  void *d_all = nullptr;          // one allocation that holds the arrays below
  int2 *d_pair_rc = nullptr;      // (row, col), row <= col
  int32_t *d_pair_start = nullptr;// entry start per pair (+1 sentinel per system, global index)
  int4 *d_ent_R = nullptr;        // R (x, y, z) and its index among the system's distinct vectors
  double2 *d_ent_t = nullptr;     // amplitude
  // per-system descriptors on the device
  int32_t *d_sys_dim = nullptr;
  int64_t *d_sys_pair_off = nullptr;
  int32_t *d_sys_npairs = nullptr;
  std::vector<int32_t> n_R;       // distinct lattice vectors per system
  int4 *d_R = nullptr;            // the distinct vectors of all systems
  int64_t *d_sys_R_off = nullptr; // per system, into d_R
  int32_t *d_sys_n_R = nullptr;
};

namespace {

__global__ void hk_zero_c128(double2 *H, int64_t stride, int32_t ld, int32_t N, int64_t n_k) {
  int64_t per = int64_t(N) * N;
  int64_t q = blockIdx.y;
  for (; q < n_k; q += gridDim.y) {
    double2 *Hq = H + q * stride;
    for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < per; e += int64_t(gridDim.x) * blockDim.x) {
      int64_t c = e / N, r = e - c * N;
      Hq[r + c * ld] = make_double2(0.0, 0.0);
    }
  }
}

__global__ void hk_zero_c64(float2 *H, int64_t stride, int32_t ld, int32_t N, int64_t n_k) {
  int64_t per = int64_t(N) * N;
  int64_t q = blockIdx.y;
  for (; q < n_k; q += gridDim.y) {
    float2 *Hq = H + q * stride;
    for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < per; e += int64_t(gridDim.x) * blockDim.x) {
      int64_t c = e / N, r = e - c * N;
      Hq[r + c * ld] = make_float2(0.f, 0.f);
    }
  }
}

// exp(2 pi i kappa.R) as (cos, sin); the argument is reduced to [-1/2, 1/2]
// before sincospi.
__device__ __forceinline__ double2 bloch_phase(int4 r, double k0, double k1, double k2, int dim) {
  double x = k0 * r.x;
  if (dim > 1) x = fma(k1, double(r.y), x);
  if (dim > 2) x = fma(k2, double(r.z), x);
  x -= rint(x);
  double s, c;
  sincospi(2.0 * x, &s, &c);
  return make_double2(c, s);
}

__device__ __forceinline__ double2 add_hop(double2 acc, double2 te, double2 ph) {
  acc.x = fma(te.x, ph.x, fma(-te.y, ph.y, acc.x));
  acc.y = fma(te.x, ph.y, fma(te.y, ph.x, acc.y));
  return acc;
}

// Sum of t exp(2 pi i kappa.R) over the entries of one pair.
__device__ __forceinline__ double2 pair_sum(const int32_t *start, int64_t p, const int4 *R, const double2 *t,
                                            double k0, double k1, double k2, int dim) {
  double2 acc = make_double2(0.0, 0.0);
  int32_t e0 = start[p], e1 = start[p + 1];
  for (int32_t e = e0; e < e1; ++e) acc = add_hop(acc, t[e], bloch_phase(R[e], k0, k1, k2, dim));
  return acc;
}

template <typename OUT>
__device__ __forceinline__ void put(OUT *Hq, int64_t idx, double2 v);
template <>
__device__ __forceinline__ void put<double2>(double2 *Hq, int64_t idx, double2 v) { Hq[idx] = v; }
template <>
__device__ __forceinline__ void put<float2>(float2 *Hq, int64_t idx, double2 v) {
  Hq[idx] = make_float2(float(v.x), float(v.y));
}

// Element (row, col) of the upper triangle and its conjugate below it.
template <typename OUT>
__device__ __forceinline__ void put_pair(OUT *Hq, int2 rc, int32_t ld, double2 v) {
  if (rc.x == rc.y) v.y = 0.0;
  put<OUT>(Hq, rc.x + int64_t(rc.y) * ld, v);
  if (rc.x != rc.y) put<OUT>(Hq, rc.y + int64_t(rc.x) * ld, be::cconj(v));
}

template <typename OUT>
__global__ void hk_scatter(OUT *H, int64_t stride, int32_t ld, int32_t sys_first, const double *kappa, int32_t n_kap,
                           int64_t n_mat, const int2 *pair_rc, const int32_t *pair_start, const int4 *ent_R,
                           const double2 *ent_t, const int32_t *sys_dim, const int64_t *sys_pair_off,
                           const int32_t *sys_npairs) {
  for (int64_t q = blockIdx.y; q < n_mat; q += gridDim.y) {
    int s = sys_first + static_cast<int>(q / n_kap);
    int k = static_cast<int>(q % n_kap);
    int np = sys_npairs[s];
    int64_t p = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (p >= np) continue;
    p += sys_pair_off[s];
    int2 rc = pair_rc[p];
    double2 v = pair_sum(pair_start, p, ent_R, ent_t, kappa[3 * k], kappa[3 * k + 1], kappa[3 * k + 2], sys_dim[s]);
    put_pair<OUT>(H + q * stride, rc, ld, v);
  }
}

// The same with the phases of a k-point's distinct lattice vectors taken once
// per workgroup into LDS: a list of many orbitals repeats each vector in
// thousands of entries, and sincospi in FP64 bounds hk_scatter. A workgroup of
// 256 threads takes 256 / pp groups of KB k-points, pp lanes each: a power of
// two that covers the pairs of small matrices (KB = 1), so that their threads
// are not idle, or all 256 and four k-points per entry read (KB = 4; the
// entries' bytes from L2 bound the sums with one: 603 us against 260 us for
// 96 orbitals, 29 vectors, 1,024 k-points, 1.39e8 entries, 1,850 us without
// the table). 210,000 matrices of order 4: 357 -> 60 us. Larger lists take
// further rounds over blockIdx.x. The sums are those of hk_scatter, bit for bit.
constexpr int kPhaseTable = 2048;  // phases in LDS (32 KB)

template <int KB, typename OUT>
__global__ __launch_bounds__(256) void hk_scatter_table(OUT *H, int64_t stride, int32_t ld, int32_t sys_first,
                                                        const double *kappa, int32_t n_kap, int32_t n_sys, int pp,
                                                        int nr_max, const int2 *pair_rc, const int32_t *pair_start,
                                                        const int4 *ent_R, const double2 *ent_t,
                                                        const int32_t *sys_dim, const int64_t *sys_pair_off,
                                                        const int32_t *sys_npairs, const int4 *Rs,
                                                        const int64_t *sys_R_off, const int32_t *sys_n_R) {
  extern __shared__ double2 tab[];  // phases [group][k-point][nr_max]
  const int per = 256 / pp, sub = threadIdx.x / pp, l = threadIdx.x % pp;
  double2 *T = tab + sub * KB * nr_max;
  const int nkb = (n_kap + KB - 1) / KB;  // groups per system
  const int64_t n_grp = int64_t(n_sys) * nkb;
  for (int64_t b0 = int64_t(blockIdx.y) * per; b0 < n_grp; b0 += int64_t(gridDim.y) * per) {
    const bool live = b0 + sub < n_grp;
    const int sl = live ? static_cast<int>((b0 + sub) / nkb) : 0, s = sys_first + sl;
    const int k0 = live ? static_cast<int>((b0 + sub) % nkb) * KB : 0;
    const int nk = live ? min(KB, n_kap - k0) : 0;
    const int nr = sys_n_R[s];
    for (int e = l; e < nk * nr; e += pp) {
      const int u = e / nr, r = e - u * nr;
      const double *kp = kappa + 3 * int64_t(k0 + u);
      T[u * nr_max + r] = bloch_phase(Rs[sys_R_off[s] + r], kp[0], kp[1], kp[2], sys_dim[s]);
    }
    __syncthreads();
    const int np = live ? sys_npairs[s] : 0;
    OUT *Hq = H + (int64_t(sl) * n_kap + k0) * stride;
    for (int p0 = blockIdx.x * pp + l; p0 < np; p0 += gridDim.x * pp) {
      const int64_t p = sys_pair_off[s] + p0;
      double2 v[KB];
#pragma unroll
      for (int u = 0; u < KB; ++u) v[u] = make_double2(0.0, 0.0);
      const int32_t e1 = pair_start[p + 1];
#pragma unroll 2
      for (int32_t e = pair_start[p]; e < e1; ++e) {
        const double2 te = ent_t[e];
        const double2 *ph = T + ent_R[e].w;
#pragma unroll
        for (int u = 0; u < KB; ++u) v[u] = add_hop(v[u], te, ph[u * nr_max]);  // slots past nk hold no result
      }
      const int2 rc = pair_rc[p];
#pragma unroll
      for (int u = 0; u < KB; ++u)
        if (u < nk) put_pair<OUT>(Hq + u * stride, rc, ld, v[u]);
    }
    __syncthreads();
  }
}

}  // namespace

extern "C" {

int be_hk_plan_create(be_ctx *ctx, const be_hoplist *sys_h, int32_t n_sys, be_hk_plan **plan) {
  using namespace be;
  BE_CHECK_ARG(ctx, ctx && sys_h && plan && n_sys > 0, "be_hk_plan_create: null argument or n_sys <= 0");
  *plan = nullptr;
  auto *P = new be_hk_plan();
  P->device = ctx->device;
  P->n_sys = n_sys;
  be::hkpack::Packed pk;
  for (int s = 0; s < n_sys; ++s) {
    const be_hoplist &h = sys_h[s];
    int32_t np = 0;
    const std::string why = be::hkpack::pack_system(h.N, h.dim, h.nnz, h.i, h.j, h.R, h.t, pk, &np);
    if (!why.empty()) {
      delete P;
      return set_err(ctx, BE_EINVAL, "be_hk_plan_create: system " + std::to_string(s) + ": " + why);
    }
    // A list with most of its pairs gets the others as pairs without entries:
    // the sums then write every element, and the launch that clears H goes (36
    // of 93 us for 210,000 matrices of order 4; Wilson loop of 1 band on 64 x 64
    // points 159 -> 115 us). From half the pairs on: a pair without entries costs
    // no more than the two elements' share of the clearing launch.
    const int64_t all = int64_t(h.N) * (h.N + 1) / 2;
    if (np < all && all <= 2 * int64_t(np) + 8) {
      const size_t first = pk.rc.size() - np;
      std::vector<char> seen(size_t(h.N) * h.N, 0);
      for (size_t a = first; a < pk.rc.size(); ++a) seen[size_t(pk.rc[a].c) * h.N + pk.rc[a].r] = 1;
      for (int32_t c = 0; c < h.N; ++c)
        for (int32_t r = 0; r <= c; ++r)
          if (!seen[size_t(c) * h.N + r]) {
            pk.rc.push_back({r, c});
            pk.start.push_back(static_cast<int32_t>(pk.R.size()));
            ++np;
          }
    }
    P->N.push_back(h.N);
    P->dim.push_back(h.dim);
    P->pair_off.push_back(static_cast<int64_t>(pk.rc.size()) - np);
    P->n_pairs.push_back(np);
  }
  pk.start.push_back(static_cast<int32_t>(pk.R.size()));
  const be::hkpack::DistinctR dr = be::hkpack::index_vectors(pk, P->pair_off, P->n_pairs);
  P->n_R = dr.count;
  P->total_pairs = static_cast<int64_t>(pk.rc.size());
  P->total_ents = static_cast<int64_t>(pk.R.size());
  // one allocation and one copy for all arrays: each hipMalloc, synchronous
  // copy and hipFree costs a small model more than its kernels (ten of them:
  // 2-band model, whole call 299 us; one: 171 us)
  struct Array {
    void **dst;
    const void *src;
    size_t bytes, off;
  };
  std::vector<Array> arrays;
  size_t total = 0;
  auto add = [&](auto **dst, const void *src, size_t count) {
    const size_t bytes = count * sizeof(**dst);
    arrays.push_back({reinterpret_cast<void **>(dst), src, bytes, total});
    total += (std::max<size_t>(bytes, 16) + 255) & ~size_t(255);
  };
  add(&P->d_pair_rc, pk.rc.data(), pk.rc.size());
  add(&P->d_pair_start, pk.start.data(), pk.start.size());
  add(&P->d_ent_R, pk.R.data(), pk.R.size());
  add(&P->d_ent_t, pk.t.data(), pk.t.size());
  add(&P->d_sys_dim, P->dim.data(), P->dim.size());
  add(&P->d_sys_pair_off, P->pair_off.data(), P->pair_off.size());
  add(&P->d_sys_npairs, P->n_pairs.data(), P->n_pairs.size());
  add(&P->d_R, dr.R.data(), dr.R.size());
  add(&P->d_sys_R_off, dr.off.data(), dr.off.size());
  add(&P->d_sys_n_R, dr.count.data(), dr.count.size());
  const std::unique_ptr<unsigned char[]> host(new unsigned char[total]);  // padding stays as it is
  for (const Array &x : arrays)
    if (x.bytes) std::memcpy(host.get() + x.off, x.src, x.bytes);
  if (hipMalloc(&P->d_all, total) != hipSuccess ||
      hipMemcpy(P->d_all, host.get(), total, hipMemcpyHostToDevice) != hipSuccess) {
    (void)hipGetLastError();
    be_hk_plan_destroy(P);
    return set_err(ctx, BE_ENOMEM, "be_hk_plan_create: device upload failed");
  }
  for (const Array &x : arrays) *x.dst = static_cast<unsigned char *>(P->d_all) + x.off;
  *plan = P;
  return BE_OK;
}

int be_hk_plan_destroy(be_hk_plan *P) {
  if (!P) return BE_EINVAL;
  (void)hipSetDevice(P->device);
  if (P->d_all) (void)hipFree(P->d_all);
  delete P;
  return BE_OK;
}

int32_t be_hk_plan_N(const be_hk_plan *P, int32_t s) {
  if (!P || s < 0 || s >= P->n_sys) return -1;
  return P->N[s];
}

int be_build_hk(be_ctx *ctx, const be_hk_plan *P, int32_t sys_first, int32_t n_sys_call, const double *kappa,
                int32_t n_kap, void *H, int64_t mat_stride, int32_t ld, int32_t dtype, hipStream_t stream) {
  using namespace be;
  BE_CHECK_ARG(ctx, ctx && P && kappa && H, "be_build_hk: null argument");
  BE_CHECK_ARG(ctx, n_kap >= 0 && n_sys_call >= 0, "be_build_hk: negative count");
  BE_CHECK_ARG(ctx, sys_first >= 0 && sys_first + n_sys_call <= P->n_sys, "be_build_hk: system range out of the plan");
  BE_CHECK_ARG(ctx, dtype == BE_C128 || dtype == BE_C64, "be_build_hk: dtype must be BE_C128 or BE_C64");
  if (n_kap == 0 || n_sys_call == 0) return BE_OK;
  int32_t N = P->N[sys_first], maxp = 0, max_R = 0;
  bool covers = true;  // the pairs are the whole upper triangle
  for (int32_t s = sys_first; s < sys_first + n_sys_call; ++s) {
    BE_CHECK_ARG(ctx, P->N[s] == N, "be_build_hk: all systems of one call must have the same N");
    maxp = std::max(maxp, P->n_pairs[s]);
    covers = covers && P->n_pairs[s] == int64_t(N) * (N + 1) / 2;
    max_R = std::max(max_R, P->n_R[s]);
  }
  BE_CHECK_ARG(ctx, ld >= N, "be_build_hk: ld < N");
  BE_CHECK_ARG(ctx, mat_stride >= int64_t(ld) * N, "be_build_hk: mat_stride < ld*N");
  int64_t n_mat = int64_t(n_sys_call) * n_kap;
  int64_t per = int64_t(N) * N;
  dim3 zb(256), zg(static_cast<uint32_t>(std::min<int64_t>((per + 255) / 256, 4096)),
                   static_cast<uint32_t>(std::min<int64_t>(n_mat, 65535)));
  ProfScope prof(ctx, "hk_build", stream);
  if (!covers) {
    if (dtype == BE_C128)
      hipLaunchKernelGGL(hk_zero_c128, zg, zb, 0, stream, static_cast<double2 *>(H), mat_stride, ld, N, n_mat);
    else
      hipLaunchKernelGGL(hk_zero_c64, zg, zb, 0, stream, static_cast<float2 *>(H), mat_stride, ld, N, n_mat);
    BE_RET_IF(check_launch(ctx, "hk_zero"));
  }
  // lanes per matrix; the phase table unless the list has too many distinct vectors for it
  int pp = 8;
  while (pp < 256 && pp < maxp) pp *= 2;
  // workgroups (x, y) with kb k-points per entry read and r rounds of pairs per
  // workgroup, which share its phases. Four k-points where the entries' reads bound
  // the sums, lists of four entries a pair and more (48 orbitals, 256 k-points 38 us,
  // 59 with one), else where they leave every compute unit work, and as many rounds,
  // up to four, as do (order 1024, five entries for four pairs, c64, one k-point: 22.5
  // us in hk_scatter, 26.8 with four of each, 23.6 so; 16: 46.2, 52.5, 47.7)
  auto grid = [&](int kb, int r) {
    const int64_t groups = (int64_t(n_sys_call) * ((n_kap + kb - 1) / kb) + 256 / pp - 1) / (256 / pp);
    return dim3(static_cast<uint32_t>(std::max(1, (maxp + r * pp - 1) / (r * pp))),
                static_cast<uint32_t>(std::min<int64_t>(groups, 65535)));
  };
  auto fills = [&](dim3 g) { return int64_t(g.x) * g.y >= 2 * ctx->n_cu; };
  const bool many = P->total_ents >= 4 * P->total_pairs && n_kap >= 4;  // entries
  const int kb = pp == 256 && 4 * int64_t(max_R) <= kPhaseTable && (many || fills(grid(4, 1))) ? 4 : 1;
  int rounds = 4;
  while (rounds > 1 && !fills(grid(kb, rounds))) rounds /= 2;
  auto go = [&](auto *Ht) {
    typedef std::remove_pointer_t<decltype(Ht)> OUT;
    const int64_t phases = (256 / pp) * int64_t(kb) * max_R;
    if (phases <= kPhaseTable) {
      const dim3 g = grid(kb, rounds);
      auto kern = kb == 4 ? &hk_scatter_table<4, OUT> : &hk_scatter_table<1, OUT>;
      hipLaunchKernelGGL(kern, g, dim3(256), size_t(phases) * sizeof(double2), stream, Ht, mat_stride, ld, sys_first,
                         kappa, n_kap, n_sys_call, pp, max_R, P->d_pair_rc, P->d_pair_start, P->d_ent_R, P->d_ent_t,
                         P->d_sys_dim, P->d_sys_pair_off, P->d_sys_npairs, P->d_R, P->d_sys_R_off, P->d_sys_n_R);
    } else {
      const dim3 g(static_cast<uint32_t>(std::max(1, (maxp + 255) / 256)),
                   static_cast<uint32_t>(std::min<int64_t>(n_mat, 65535)));
      hipLaunchKernelGGL(hk_scatter<OUT>, g, dim3(256), 0, stream, Ht, mat_stride, ld, sys_first, kappa, n_kap, n_mat,
                         P->d_pair_rc, P->d_pair_start, P->d_ent_R, P->d_ent_t, P->d_sys_dim, P->d_sys_pair_off,
                         P->d_sys_npairs);
    }
  };
  if (dtype == BE_C128) go(static_cast<double2 *>(H));
  else go(static_cast<float2 *>(H));
  return check_launch(ctx, "hk_scatter");
}

}  // extern "C"
