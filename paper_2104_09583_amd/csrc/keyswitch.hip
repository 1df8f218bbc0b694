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
// extended row o (global prime `prime`)
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
    int nl, int alpha, int logN, size_t key_ds, const DevPrime* __restrict__ P) {
  __shared__ double sh[kLdsTile4];
  const size_t N = (size_t)1 << logN;
  const KsPlace pl = ks_place(njobs);
  const KsRot jb = jobs.j[pl.job];
  const int i = pl.row;
  const DevPrime pr = P[i];
  double a[8];
  row4_fwd_tile(w + (((size_t)pl.job * 2 + pl.poly) * nl + i) * N + pl.t0, pl.t0, logN - 12, pr, sh, a);
#pragma unroll
  for (int k = 0; k < 8; ++k) a[k] = -mul_lazy(a[k], t_mod, pr.q, pr.qinv);
  const AutoTile at = auto_tile(pl.t0, jb.g, logN);
  rot_digits(a, jb, pl.poly == 0 ? jb.kb : jb.ka, D, i, i / alpha, i, nE, at, pl.t0, N, key_ds, pr);
  // at most eight digits: |a| < 10 q, the product below 2.5 q
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
static void check_rot(const Context& c, int D) {
  if (c.log_n < 13) fail(COPSE_EINVAL, "internal: split transform needs N >= 8192");
  if (D < 1 || D > 8) fail(COPSE_EINVAL, "internal: too many digits for the fused rotation");
}

void launch_ks_rot_special(Context& c, const std::vector<KsRot>& jobs, double* acc, int D, int nE, int level,
                           size_t key_ds) {
  check_rot(c, D);
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
  check_rot(c, D);
  const int nl = level + 1;
  const size_t per = rot_per_launch(c);
  for (size_t first = 0; first < jobs.size(); first += per) {
    const int cnt = (int)std::min<size_t>(per, jobs.size() - first);
    const RotPack pk = rot_pack(jobs, first, cnt);
    hipEvent_t ev;
    prof_begin(c, 7, &ev);
    hipLaunchKernelGGL(ks_rot_finish_kernel, dim3((unsigned)(c.N / 4096), nl, 2 * cnt), dim3(512), 0, c.stream, pk,
                       cnt, w + first * 2 * nl * c.N, pinv, (double)c.t, D, nE, nl, c.alpha, (int)c.log_n, key_ds,
                       c.d_primes);
    COPSE_HIP(hipGetLastError());
    prof_end(c, 7, ev, ((double)(D + 5) * cnt + 2.0 * D * distinct_keys(pk, cnt)) * nl * (double)c.N * 8.0);
  }
}

}  // namespace copse
