// Key switching with the inner products formed where their result is used, for the rings of the split transform
// (N = 2^13 .. 2^16).
//
// A key switch ends with the ModDown: of the extended basis' rows only the special ones (and, merged with a modulus
// switch, the top data row) are transformed back and converted; the data rows meet the converted rows w in the
// finish, out_i = (y_i - t w_i) P^-1.  So the inner products y of the rows that go back are computed by a kernel that
// runs their inverse row pass before it writes them, and those of the data rows by the finish itself, in registers:
// they are never written or read.  A rotation at six limbs moved 118 rows per job with the inner products, the row
// pass, the column pass and the finish apart; it moves 78 so, in one launch less.
#include <algorithm>

#include "internal.hpp"
#include "rowtile.hpp"

namespace copse {

// One hoisted rotation: digits' own limbs from `in` (NTT form, nl limbs), the other rows from `ext` [D][nE][N], the
// key [D][Ltot][N], polynomial 0 of the unrotated ciphertext, and the result (2 polys of nl limbs).
struct RotPack {
  static constexpr int kMax = 32;   // 32 x 56 B of kernel arguments
  KsRot j[kMax];
};

// Place of a workgroup: the tile index fastest (the eight XCDs keep to their tiles of N = 32768), then the
// polynomial, whose two workgroups read the same digits, then the job, since consecutive jobs read the same key: what
// the first of them fetches the others find in that XCD's L2.
struct KsPlace {
  int row, job, poly;
  size_t t0;
};
__device__ __forceinline__ KsPlace ks_place(int njobs) {
  const unsigned lin = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
  const unsigned rest = lin / gridDim.x;
  KsPlace p;
  p.t0 = (size_t)(lin % gridDim.x) * 4096;
  p.poly = (int)(rest & 1u);
  p.job = (int)((rest >> 1) % (unsigned)njobs);
  p.row = (int)((rest >> 1) / (unsigned)njobs);
  return p;
}

// a += sum over the digits of digit x key (key: the polynomial's half of it), on the positions t + 512 k of a tile of
// extended row o (global prime `prime`).  Each product is within 0.69 q; from |a| < 2 q the sum is folded back after
// every eight (below 7.5 q), so that any number of digits (48 at most, one prime each) ends below 6.1 q or, without a
// fold, below 7.5 q.
__device__ __forceinline__ void rot_digits(double (&a)[8], const KsRot& jb, const double* key, int D, int o, int own,
                                           int prime, int nE, const AutoTile& at, size_t t0, size_t N, size_t key_ds,
                                           const DevPrime& pr) {
  key += (size_t)prime * N + t0;
  for (int j = 0; j < D; ++j) {
    const double* row = j == own ? jb.in + (size_t)o * N : jb.ext + ((size_t)j * nE + o) * N;   // uniform
    double e[8], kv[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      e[k] = auto_load(row, at, k);
      kv[k] = tile_load(key + (size_t)j * key_ds, k);
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) a[k] += mul_lazy(e[k], kv[k], pr.q, pr.qinv);
    if ((j & 7) == 7) red8(a, pr);   // uniform
  }
}

// Special rows: the sum of one polynomial's special row, then its inverse row pass, to acc [job][2][alpha][N].  Bytes
// and arithmetic are even here (3.3 us of each per workgroup and unit, 5.5 measured), so what counts is that one
// workgroup's transform covers another's loads: at 62 registers four share a compute unit.  32 jobs of the 32-tree
// forest's reshuffle: 44 us a launch (the separate inner products and row pass of these rows: 52).
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(6))) void ks_rot_special_kernel(
    RotPack jobs, int njobs, double* __restrict__ acc, int D, int nE, int nl, int L, int alpha, int logN, size_t key_ds,
    const DevPrime* __restrict__ P) {
  __shared__ double sh[kLdsTile4];
  const size_t N = (size_t)1 << logN;
  const KsPlace pl = ks_place(njobs);
  const KsRot jb = jobs.j[pl.job];
  const int prime = L + 1 + pl.row;
  const DevPrime pr = P[prime];
  const AutoTile at = auto_tile(pl.t0, jb.g, logN);
  double a[8], x[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) a[k] = 0.0;
  rot_digits(a, jb, pl.poly == 0 ? jb.kb : jb.ka, D, nl + pl.row, -1, prime, nE, at, pl.t0, N, key_ds, pr);
  red8(a, pr);
  row4_inv_tile(nullptr, pl.t0, logN - 12, pr, sh, x, a);
  if (pr.q >= kInvOpen) red8(x, pr);   // uniform
  double* o = acc + (((size_t)pl.job * 2 + pl.poly) * alpha + pl.row) * N + pl.t0;
#pragma unroll
  for (int k = 0; k < 8; ++k) tile_store(o, k, x[k]);
}

// Data row i of one polynomial: the forward row pass of its converted row w, the inner product added to -t w in
// registers, out_0 = (sum - t w) P^-1 + sigma(c0), out_1 = (sum - t w) P^-1.  Bound by HBM, at 5 TB/s: 73 us a launch of
// 32 jobs (the inner products of the data rows and the finish apart: 92).
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(6))) void ks_rot_finish_kernel(
    RotPack jobs, int njobs, const double* __restrict__ w, const double* __restrict__ pinv, double t_mod, int D, int nE,
    int nl, int alpha, int logN, size_t key_ds, const DevPrime* __restrict__ P, bool packed) {
  __shared__ double sh[kLdsTile4];
  const size_t N = (size_t)1 << logN;
  const KsPlace pl = ks_place(njobs);
  const KsRot jb = jobs.j[pl.job];
  const int i = pl.row;
  const DevPrime pr = P[i];
  double a[8];
  row4_fwd_tile(TileSrc{row_at(w, ((size_t)pl.job * 2 + pl.poly) * nl + i, N, packed), pl.t0, N, packed}, logN - 12, pr, sh,
                a);
#pragma unroll
  for (int k = 0; k < 8; ++k) a[k] = -mul_lazy(a[k], t_mod, pr.q, pr.qinv);
  const AutoTile at = auto_tile(pl.t0, jb.g, logN);
  rot_digits(a, jb, pl.poly == 0 ? jb.kb : jb.ka, D, i, i / alpha, i, nE, at, pl.t0, N, key_ds, pr);
  // |a| < 7.5 q, the product below 2 q
  const double pi = pinv[i];
#pragma unroll
  for (int k = 0; k < 8; ++k) a[k] = mul_lazy(a[k], pi, pr.q, pr.qinv);
  if (pl.poly == 0) {   // uniform
#pragma unroll
    for (int k = 0; k < 8; ++k) a[k] += auto_load(jb.c0 + (size_t)i * N, at, k);
  }
  double* o = jb.out + ((size_t)pl.poly * nl + i) * N + pl.t0;
#pragma unroll
  for (int k = 0; k < 8; ++k) tile_store(o, k, canon(reduce_sym(a[k], pr.q, pr.qinv), pr.q));
}

static size_t rot_per_launch(const Context& c) {
  return c.tune.ks_jobs > 0 ? (size_t)std::min(c.tune.ks_jobs, RotPack::kMax) : RotPack::kMax;
}
static int distinct_keys(const RotPack& pk, int cnt) {
  int keys = 0;
  for (int k = 0; k < cnt; ++k) {
    bool seen = false;
    for (int k2 = 0; k2 < k; ++k2) seen |= pk.j[k2].kb == pk.j[k].kb;
    keys += !seen;
  }
  return keys;
}
static RotPack rot_pack(const std::vector<KsRot>& jobs, size_t first, int cnt) {
  RotPack pk;
  for (int k = 0; k < cnt; ++k) pk.j[k] = jobs[first + k];
  return pk;
}
static void check_split(const Context& c) {
  if (c.log_n < 13) fail(COPSE_EINVAL, "internal: split transform needs N >= 8192");
}

void launch_ks_rot_special(Context& c, const std::vector<KsRot>& jobs, double* acc, int D, int nE, int level,
                           size_t key_ds) {
  check_split(c);
  const size_t per = rot_per_launch(c);
  for (size_t first = 0; first < jobs.size(); first += per) {
    const int cnt = (int)std::min<size_t>(per, jobs.size() - first);
    const RotPack pk = rot_pack(jobs, first, cnt);
    hipEvent_t ev;
    prof_begin(c, 4, &ev);
    hipLaunchKernelGGL(ks_rot_special_kernel, dim3((unsigned)(c.N / 4096), c.alpha, 2 * cnt), dim3(512), 0, c.stream,
                       pk, cnt, acc + first * 2 * c.alpha * c.N, D, nE, level + 1, c.L, c.alpha, (int)c.log_n, key_ds,
                       c.d_primes);
    COPSE_HIP(hipGetLastError());
    prof_end(c, 4, ev, ((double)(D + 2) * cnt + 2.0 * D * distinct_keys(pk, cnt)) * c.alpha * (double)c.N * 8.0);
  }
}

void launch_ks_rot_finish(Context& c, const std::vector<KsRot>& jobs, const double* w, const double* pinv, int D,
                          int nE, int level, size_t key_ds) {
  check_split(c);
  const int nl = level + 1;
  const size_t per = rot_per_launch(c);
  for (size_t first = 0; first < jobs.size(); first += per) {
    const int cnt = (int)std::min<size_t>(per, jobs.size() - first);
    const RotPack pk = rot_pack(jobs, first, cnt);
    hipEvent_t ev;
    prof_begin(c, 7, &ev);
    hipLaunchKernelGGL(ks_rot_finish_kernel, dim3((unsigned)(c.N / 4096), nl, 2 * cnt), dim3(512), 0, c.stream, pk,
                       cnt, w + first * 2 * nl * c.row_doubles(), pinv, (double)c.t, D, nE, nl, c.alpha, (int)c.log_n, key_ds,
                       c.d_primes, c.packed);
    COPSE_HIP(hipGetLastError());
    prof_end(c, 7, ev, ((double)(D + 5) * cnt + 2.0 * D * distinct_keys(pk, cnt)) * nl * (double)c.N * 8.0);
  }
}

// ------------------------------------------------------------------ relinearizations
struct RelinPack {
  static constexpr int kMax = 32;   // 32 x 64 B of kernel arguments
  KsRelin j[kMax];
};

// Data row i of both polynomials of one job.  The finish is out_k = (sum_k - cw w_k + ca add_k) m1 (cw = t, ca = P,
// m1 = P^-1 for a ModDown; t P, P and (P q_l)^-1 merged with the switch), so the sums start from -cw w_k + ca add_k
// and everything stays in registers: the inner products are never written, and of a product's operands each row is
// read once for the addend (a0 b0, a0 b1 + a1 b0) and for the row's own digit a1 b1.  Both rows w are transformed as
// one pair, the other digits' rows one at a time with the sums live (128 registers, two workgroups per compute unit).
__global__ __launch_bounds__(512, 4) void ks_relin_finish_kernel(RelinPack jobs, int njobs,
                                                                 const double* __restrict__ w,
                                                                 const double* __restrict__ m1,
                                                                 const double* __restrict__ cw,
                                                                 const double* __restrict__ ca, double t_mod, int nout,
                                                                 int D, int nE, int nl, int alpha, int logN,
                                                                 size_t key_ds, const DevPrime* __restrict__ P,
                                                                 bool packed) {
  __shared__ double sh[kLdsTile4], sh2[kLdsTile4];
  const size_t N = (size_t)1 << logN;
  const unsigned lin = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
  const unsigned rest = lin / gridDim.x;
  const size_t t0 = (size_t)(lin % gridDim.x) * 4096;
  const int job = (int)(rest % (unsigned)njobs), i = (int)(rest / (unsigned)njobs);
  const KsRelin jb = jobs.j[job];
  const DevPrime pr = cload_prime(P + i);
  const int S1 = logN - 12, own = i / alpha;
  const size_t ro = (size_t)i * N + t0, ps = (size_t)nl * N;
  double a0[8], a1[8];
  const size_t r0 = (size_t)job * 2 * nout + i;
  row4_fwd_tile2(TileSrc{row_at(w, r0, N, packed), t0, N, packed}, TileSrc{row_at(w, r0 + nout, N, packed), t0, N, packed},
                 S1, pr, sh, sh2, a0, a1);
  const double c1 = cw != nullptr ? cload(cw + i) : t_mod, c2 = cload(ca + i);
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    a0[k] = -mul_lazy(a0[k], c1, pr.q, pr.qinv);
    a1[k] = -mul_lazy(a1[k], c1, pr.q, pr.qinv);
  }
  auto mac = [&](int j, double(&x)[8]) {
    const size_t ko = (size_t)j * key_ds + ro;
    double kv[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) kv[k] = tile_load(jb.kb + ko, k);
    if (pr.q >= kFwdLazy) red8(x, pr);   // uniform
#pragma unroll
    for (int k = 0; k < 8; ++k) a0[k] += mul_lazy(x[k], kv[k], pr.q, pr.qinv);
#pragma unroll
    for (int k = 0; k < 8; ++k) kv[k] = tile_load(jb.ka + ko, k);
#pragma unroll
    for (int k = 0; k < 8; ++k) a1[k] += mul_lazy(x[k], kv[k], pr.q, pr.qinv);
  };
  // the addend, and the row's own digit
  {
    double x[8];
    const double* d0 = jb.add + ro;
    const double* d1 = d0 + ps;
    if (jb.add_b != nullptr) {   // uniform
      const double* e0 = jb.add_b + ro;
      const double* e1 = e0 + ps;
      // in an order that keeps three rows live
      double u[8], v[8], y[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        u[k] = tile_load(d0, k);
        v[k] = tile_load(e0, k);
      }
#pragma unroll
      for (int k = 0; k < 8; ++k)
        a0[k] += mul_lazy(mul_lazy(u[k], v[k], pr.q, pr.qinv), c2, pr.q, pr.qinv);
#pragma unroll
      for (int k = 0; k < 8; ++k) y[k] = tile_load(e1, k);
#pragma unroll
      for (int k = 0; k < 8; ++k) u[k] = mul_lazy(u[k], y[k], pr.q, pr.qinv);
#pragma unroll
      for (int k = 0; k < 8; ++k) x[k] = tile_load(d1, k);
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        a1[k] += mul_lazy(u[k] + mul_lazy(x[k], v[k], pr.q, pr.qinv), c2, pr.q, pr.qinv);
        x[k] = mul_lazy(x[k], y[k], pr.q, pr.qinv);
      }
    } else {
      double u[8], v[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        u[k] = tile_load(d0, k);
        v[k] = tile_load(d1, k);
        x[k] = tile_load(jb.in + ro, k);
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        a0[k] += mul_lazy(u[k], c2, pr.q, pr.qinv);
        a1[k] += mul_lazy(v[k], c2, pr.q, pr.qinv);
      }
    }
    mac(own, x);
  }
  for (int j = 0; j < D; ++j) {   // uniform
    if (j == own) continue;
    double x[8];
    lds_barrier();   // the tile buffer's previous use is over in every wave
    row4_fwd_tile(TileSrc{jb.ext + ((size_t)j * nE + i) * N, t0, N, false}, S1, pr, sh, x);
    mac(j, x);
  }
  // at most eight digits: |a| < 10 q, the product below 2.5 q
  const double m = cload(m1 + i);
  double* o = jb.out + ro;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    tile_store(o, k, canon(reduce_sym(mul_lazy(a0[k], m, pr.q, pr.qinv), pr.q, pr.qinv), pr.q));
    tile_store(o + (size_t)nout * N, k, canon(reduce_sym(mul_lazy(a1[k], m, pr.q, pr.qinv), pr.q, pr.qinv), pr.q));
  }
}

void launch_ks_relin_finish(Context& c, const std::vector<KsRelin>& jobs, const double* w, const double* m1,
                            const double* cw, const double* ca, int nout, int D, int nE, int level, size_t key_ds) {
  check_split(c);
  if (D > 8) fail(COPSE_EINVAL, "internal: too many digits for the fused inner product");
  if (nout < 1 || nout > level + 1) fail(COPSE_EINVAL, "internal: relinearization without output limbs");
  const size_t per = c.tune.ks_jobs > 0 ? (size_t)std::min(c.tune.ks_jobs, RelinPack::kMax) : RelinPack::kMax;
  for (size_t first = 0; first < jobs.size(); first += per) {
    const int cnt = (int)std::min<size_t>(per, jobs.size() - first);
    RelinPack pk;
    double rows = 0;
    for (int k = 0; k < cnt; ++k) {
      pk.j[k] = jobs[first + k];
      rows += D - 1 + 2 + 2 + (pk.j[k].add_b != nullptr ? 4 : 3);
    }
    hipEvent_t ev;
    prof_begin(c, 7, &ev);
    hipLaunchKernelGGL(ks_relin_finish_kernel, dim3((unsigned)(c.N / 4096), nout, cnt), dim3(512), 0, c.stream, pk, cnt,
                       w + first * 2 * nout * c.row_doubles(), m1, cw, ca, (double)c.t, nout, D, nE, level + 1, c.alpha,
                       (int)c.log_n, key_ds, c.d_primes, c.packed);
    COPSE_HIP(hipGetLastError());
    prof_end(c, 7, ev, (rows + 2.0 * D) * nout * (double)c.N * 8.0);
  }
}

}  // namespace copse
