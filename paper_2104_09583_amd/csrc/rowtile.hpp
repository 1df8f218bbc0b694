// The transform's row pass on one tile of 4096 elements, and the automorphism's index in the evaluation domain:
// the device functions that the row kernels and the fused key-switching kernels share.
#pragma once

#include "modarith.hpp"

namespace copse {

// ------------------------------------------------------------------ automorphism (evaluation domain)
// Slot k holds a(psi^e) with e = 2 bitrev(k) + 1.  sigma_g(a)(psi^e) = a(psi^(g e)), so the
// output slot k reads the input slot holding exponent g e mod 2N.
__device__ __forceinline__ uint32_t auto_src(uint32_t k, uint64_t g, int logN) {
  // g, e < 2 N: only the product's low logN + 1 bits are used, so a 24-bit product (full rate) serves N < 2^23
  uint32_t e = 2 * (__builtin_bitreverse32(k) >> (32 - logN)) + 1;
  uint32_t ge = __umul24((uint32_t)g, e) & (uint32_t)((2ULL << logN) - 1);
  return __builtin_bitreverse32(ge >> 1) >> (32 - logN);
}

// The same for a tile of 4096 positions t + 512 k (t the thread, N = 2^logN, logN >= 12): with h = logN - 12, tile
// index i and br the bit reversal, sigma_g takes position t + 512 k of tile i from index
//   br_logN(u_k + g 2^(3+h) br9(t)),  u_k = (g - 1) / 2 + g (2^h br3(k) + br_h(i))   (mod N),
// whose low 3 + h bits (reversed: the 512-element block) are u_k's and the same for all threads.  So the block and
// the added constant are scalars, and a lane's offset inside the block is an add and a bit reversal.
struct AutoTile {
  uint32_t block[8];   // first element of the source block of position class k (uniform)
  uint32_t bytes[8];   // byte offset of the thread's element in it
};
__device__ __forceinline__ AutoTile auto_tile(size_t t0, uint64_t g64, int logN) {
  const uint32_t g = (uint32_t)g64, s = (uint32_t)(logN - 9), h = s - 3, tile = (uint32_t)(t0 >> 12);
  const uint32_t ti = h == 0 ? 0 : __builtin_bitreverse32(tile) >> (32 - h);
  const uint32_t lane = __umul24(g, __builtin_bitreverse32(threadIdx.x) >> 23) << 23;
  AutoTile a;
#pragma unroll
  for (uint32_t k = 0; k < 8; ++k) {
    const uint32_t kr = (k >> 2) | (k & 2) | ((k & 1) << 2);
    const uint32_t u = ((g - 1) >> 1) + g * ((kr << h) + ti);
    a.block[k] = (__builtin_bitreverse32(u & ((1u << s) - 1)) >> (32 - s)) << 9;
    a.bytes[k] = __builtin_bitreverse32(lane + ((u >> s) << 23)) << 3;
  }
  return a;
}
__device__ __forceinline__ double auto_load(const double* row, const AutoTile& a, int k) {
  return gload_off(uniform(row + a.block[k]), a.bytes[k]);
}

// ------------------------------------------------------------------ row tiles
// LDS place of tile position j: the bits that tell lanes apart in each of the four access patterns below (distances
// 512, 64, 8 and 1 between a thread's elements) are folded into the low five, so that in a one-address access 32
// consecutive lanes touch 32 different 8-byte slots in all of them.  The counters show 0.6 conflict cycles per LDS
// instruction in the kernels of one tile, of whose 52 accesses the compiler has joined 12 from two, and up to 1.6 in
// those of a pair of tiles, where half are joined (2.0 everywhere with one word of padding every 16).  The fold is linear over GF(2), so a thread computes one base per pattern and reaches its eight
// positions by constants.
__device__ __forceinline__ uint32_t lds_fold(uint32_t j) { return j ^ ((j >> 5) & 7u) ^ (((j >> 6) & 3u) << 3); }
struct LdsPlace {
  uint32_t a, b, c, d;
};
__device__ __forceinline__ LdsPlace lds_place() {
  const uint32_t t = threadIdx.x;
  return {lds_fold(t), lds_fold((t >> 6) * 512 + (t & 63)), lds_fold((t >> 3) * 64 + (t & 7)), lds_fold(8 * t)};
}
__device__ __forceinline__ uint32_t lds_a(const LdsPlace& p, uint32_t k) { return p.a + 512 * k; }
__device__ __forceinline__ uint32_t lds_b(const LdsPlace& p, uint32_t k) { return (p.b ^ (10 * (k & 3))) + 64 * k; }
__device__ __forceinline__ uint32_t lds_c(const LdsPlace& p, uint32_t k) {
  return (p.c ^ ((8 * (k & 3)) | (k >> 2))) + 32 * (k >> 2);
}
__device__ __forceinline__ uint32_t lds_d(const LdsPlace& p, uint32_t k) { return p.d ^ k; }

__device__ __forceinline__ void red8(double* x, const DevPrime& pr) {
#pragma unroll
  for (int k = 0; k < 8; ++k) x[k] = reduce_sym(x[k], pr.q, pr.qinv);
}

// Twiddles of one radix-8 round of a thread whose 8 elements gb + d k (k < 8) lie in one aligned block of
// 8 d at stage offset m (the round's three stages use 1, 2 and 4 of them).
struct Tw8 {
  double w0, w1a, w1b, w2[4];
};
// group g0 + v of the round whose three stages' tables start at m, 2 m and 4 m; g0 uniform, v the lane's part (below
// 2^9), so that every load is a scalar base and a 32-bit lane offset
__device__ __forceinline__ Tw8 tw8_load(const double* tab, uint32_t g0, uint32_t m, uint32_t v) {
  const double* p0 = uniform(tab + m + g0);
  const double* p1 = uniform(tab + 2 * (m + g0));
  const double* p2 = uniform(tab + 4 * (m + g0));
  Tw8 w;
  w.w0 = gload_off(p0, 8 * v);
  w.w1a = gload_off(p1, 16 * v);
  w.w1b = gload_off(p1, 16 * v + 8);
#pragma unroll
  for (int k = 0; k < 4; ++k) w.w2[k] = gload_off(p2, 32 * v + 8 * k);
  return w;
}
// the same for a group that the whole wave shares: scalar loads into scalar registers
__device__ __forceinline__ Tw8 tw8_scalar(const double* tab, uint32_t g0, uint32_t m) {
  Tw8 w;
  w.w0 = cload(tab + m + g0);
  w.w1a = cload(tab + 2 * (m + g0));
  w.w1b = cload(tab + 2 * (m + g0) + 1);
#pragma unroll
  for (int k = 0; k < 4; ++k) w.w2[k] = cload(tab + 4 * (m + g0) + k);
  return w;
}
// position t + 512 k of a tile (p: uniform)
__device__ __forceinline__ double tile_load(const double* p, int k) {
  return gload_off(uniform(p + 512 * k), 8 * threadIdx.x);
}
// A tile of a row that is plain or packed (see pack48): the row's start, the tile's first element, N
struct TileSrc {
  const double* row;
  size_t t0, N;
  bool packed;
};
__device__ __forceinline__ void tile_read(const TileSrc& s, double (&x)[8]) {
  if (s.packed) {   // uniform
    const uint32_t* lo = reinterpret_cast<const uint32_t*>(s.row);
    const uint16_t* hi = reinterpret_cast<const uint16_t*>(lo + s.N);
    uint32_t l[8], h[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      l[k] = gload32_off(uniform(lo + s.t0 + 512 * k), 4 * threadIdx.x);
      h[k] = gload16_off(uniform(hi + s.t0 + 512 * k), 2 * threadIdx.x);
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) x[k] = unpack48(l[k], h[k]);
  } else {
#pragma unroll
    for (int k = 0; k < 8; ++k) x[k] = tile_load(s.row + s.t0, k);
  }
}
__device__ __forceinline__ void tile_store(double* p, int k, double v) {
  auto* q = (__attribute__((address_space(1))) char*)uniform(p + 512 * k);
  *(__attribute__((address_space(1))) double*)(q + (size_t)(uint32_t)(8 * threadIdx.x)) = v;
}
__device__ __forceinline__ void radix8_ct_w(double* x, const Tw8& w, const DevPrime& pr) {
#pragma unroll
  for (int k = 0; k < 4; ++k) bfly_ct(x[k], x[k + 4], w.w0, pr.q, pr.qinv);
  bfly_ct(x[0], x[2], w.w1a, pr.q, pr.qinv);
  bfly_ct(x[1], x[3], w.w1a, pr.q, pr.qinv);
  bfly_ct(x[4], x[6], w.w1b, pr.q, pr.qinv);
  bfly_ct(x[5], x[7], w.w1b, pr.q, pr.qinv);
#pragma unroll
  for (int k = 0; k < 4; ++k) bfly_ct(x[2 * k], x[2 * k + 1], w.w2[k], pr.q, pr.qinv);
}
__device__ __forceinline__ void radix8_gs_w(double* x, const Tw8& w, const DevPrime& pr) {
#pragma unroll
  for (int k = 0; k < 4; ++k) bfly_gs(x[2 * k], x[2 * k + 1], w.w2[k], pr.q, pr.qinv);
  bfly_gs(x[0], x[2], w.w1a, pr.q, pr.qinv);
  bfly_gs(x[1], x[3], w.w1a, pr.q, pr.qinv);
  bfly_gs(x[4], x[6], w.w1b, pr.q, pr.qinv);
  bfly_gs(x[5], x[7], w.w1b, pr.q, pr.qinv);
#pragma unroll
  for (int k = 0; k < 4; ++k) bfly_gs(x[k], x[k + 4], w.w0, pr.q, pr.qinv);
}

// Row pass over a tile of 4096 contiguous elements (stages S1..S1+11): 512 threads x 8 registers,
// four radix-8 rounds (distances 2048/1024/512, 256/128/64, 32/16/8, 4/2/1) with three LDS exchanges.
constexpr int kLdsTile4 = 4096;

// One 4096-element tile of the row pass, 512 threads x 8 registers, four radix-8 rounds with LDS
// exchanges between them and one more so that global memory is always touched at t + 512 k (each
// load or store instruction covers 512 consecutive bytes per wave).  Both directions read src[t + 512 k]
// of the tile and leave the values of tile positions t + 512 k in x[k] (signed, not reduced).  gb0 is the
// tile's first index in the row (twiddle groups).  The first two rounds' twiddle groups are the same for a whole
// workgroup and a whole wave (distances 512 and 64): scalar loads, which cost neither vector registers nor lane
// addresses; those of the last two rounds are loaded one round ahead, so a small launch waits on memory once.
// With pre given, the forward tile also loads pre[t + 512 k] into y[k] during its third round (an
// epilogue's operand, so that its latency overlaps the transform).
__device__ __forceinline__ void row4_fwd_tile(const TileSrc& src, int S1, const DevPrime& pr,
                                              double* sh, double x[8], const double* pre = nullptr,
                                              double* y = nullptr) {
  const int t = threadIdx.x;
  const uint32_t mA = 1u << S1, mB = mA << 3, mC = mA << 6, mD = mA << 9, tile = (uint32_t)(src.t0 >> 12);
  const LdsPlace lp = lds_place();
  const uint32_t wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const Tw8 wa = tw8_scalar(pr.fwd, tile, mA);
  const Tw8 wb = tw8_scalar(pr.fwd, 8 * tile + wave, mB);
  tile_read(src, *reinterpret_cast<double (*)[8]>(x));
  radix8_ct_w(x, wa, pr);
  const Tw8 wc = tw8_load(pr.fwd, 64 * tile, mC, (uint32_t)t >> 3);
#pragma unroll
  for (int k = 0; k < 8; ++k) sh[lds_a(lp, k)] = x[k];
  lds_barrier();
#pragma unroll
  for (int k = 0; k < 8; ++k) x[k] = sh[lds_b(lp, k)];
  radix8_ct_w(x, wb, pr);
  const Tw8 wd = tw8_load(pr.fwd, 512 * tile, mD, (uint32_t)t);
  if (pr.q >= kFwdLazy) red8(x, pr);   // uniform
#pragma unroll
  for (int k = 0; k < 8; ++k) sh[lds_b(lp, k)] = x[k];
  lds_wave_sync();   // rounds B and C touch the same 512 elements of this wave's block
#pragma unroll
  for (int k = 0; k < 8; ++k) x[k] = sh[lds_c(lp, k)];
  if (pre != nullptr) {
#pragma unroll
    for (int k = 0; k < 8; ++k) y[k] = tile_load(pre, k);
  }
  radix8_ct_w(x, wc, pr);
#pragma unroll
  for (int k = 0; k < 8; ++k) sh[lds_c(lp, k)] = x[k];
  lds_wave_sync();   // and so do rounds C and D
#pragma unroll
  for (int k = 0; k < 8; ++k) x[k] = sh[lds_d(lp, k)];
  radix8_ct_w(x, wd, pr);
  // each thread overwrites only the LDS words it just read
#pragma unroll
  for (int k = 0; k < 8; ++k) sh[lds_d(lp, k)] = x[k];
  lds_barrier();
#pragma unroll
  for (int k = 0; k < 8; ++k) x[k] = sh[lds_a(lp, k)];
}

// With vals given, the tile's values at t + 512 k are vals[k] instead of src[t + 512 k].
__device__ __forceinline__ void row4_inv_tile(const double* __restrict__ src, size_t gb0, int S1, const DevPrime& pr,
                                              double* sh, double x[8], const double* vals = nullptr) {
  const int t = threadIdx.x;
  const uint32_t mA = 1u << S1, mB = mA << 3, mC = mA << 6, mD = mA << 9, tile = (uint32_t)(gb0 >> 12);
  const LdsPlace lp = lds_place();
  const uint32_t wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const Tw8 wd = tw8_load(pr.inv, 512 * tile, mD, (uint32_t)t);
  const Tw8 wc = tw8_load(pr.inv, 64 * tile, mC, (uint32_t)t >> 3);
#pragma unroll
  for (int k = 0; k < 8; ++k) sh[lds_a(lp, k)] = vals != nullptr ? vals[k] : tile_load(src, k);
  lds_barrier();
#pragma unroll
  for (int k = 0; k < 8; ++k) x[k] = sh[lds_d(lp, k)];
  radix8_gs_w(x, wd, pr);
  const Tw8 wb = tw8_scalar(pr.inv, 8 * tile + wave, mB);
  if (pr.q >= kInvLazy) red8(x, pr);   // uniform
#pragma unroll
  for (int k = 0; k < 8; ++k) sh[lds_d(lp, k)] = x[k];
  lds_wave_sync();   // rounds D and C touch the same 512 elements of this wave's block
#pragma unroll
  for (int k = 0; k < 8; ++k) x[k] = sh[lds_c(lp, k)];
  radix8_gs_w(x, wc, pr);
  const Tw8 wa = tw8_scalar(pr.inv, tile, mA);
  red8(x, pr);
#pragma unroll
  for (int k = 0; k < 8; ++k) sh[lds_c(lp, k)] = x[k];
  lds_wave_sync();   // and so do rounds C and B
#pragma unroll
  for (int k = 0; k < 8; ++k) x[k] = sh[lds_b(lp, k)];
  radix8_gs_w(x, wb, pr);
  if (pr.q >= kInvLazy) red8(x, pr);
#pragma unroll
  for (int k = 0; k < 8; ++k) sh[lds_b(lp, k)] = x[k];
  lds_barrier();
#pragma unroll
  for (int k = 0; k < 8; ++k) x[k] = sh[lds_a(lp, k)];
  radix8_gs_w(x, wa, pr);
}

// Two tiles of one row pass at once (the same prime and tile position, so the same twiddles): the rounds of
// both run between the same exchanges, so a workgroup waits at half the barriers per tile and has twice the
// independent work between them.  sh and sh2: one tile buffer each.  The forward pair reads srcA[t + 512 k]
// and srcB[t + 512 k]; the inverse pair takes the tiles' values at t + 512 k in va and vb.  Results as for
// one tile, in x and y.
__device__ __forceinline__ void row4_fwd_tile2(const TileSrc& srcA, const TileSrc& srcB, int S1,
                                               const DevPrime& pr, double* sh, double* sh2,
                                               double x[8], double y[8]) {
  const int t = threadIdx.x;
  const uint32_t mA = 1u << S1, mB = mA << 3, mC = mA << 6, mD = mA << 9, tile = (uint32_t)(srcA.t0 >> 12);
  const LdsPlace lp = lds_place();
  const uint32_t wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const Tw8 wa = tw8_scalar(pr.fwd, tile, mA);
  const Tw8 wb = tw8_scalar(pr.fwd, 8 * tile + wave, mB);
  tile_read(srcA, *reinterpret_cast<double (*)[8]>(x));
  tile_read(srcB, *reinterpret_cast<double (*)[8]>(y));
  radix8_ct_w(x, wa, pr);
  radix8_ct_w(y, wa, pr);
  const Tw8 wc = tw8_load(pr.fwd, 64 * tile, mC, (uint32_t)t >> 3);
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    sh[lds_a(lp, k)] = x[k];
    sh2[lds_a(lp, k)] = y[k];
  }
  lds_barrier();
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    x[k] = sh[lds_b(lp, k)];
    y[k] = sh2[lds_b(lp, k)];
  }
  radix8_ct_w(x, wb, pr);
  radix8_ct_w(y, wb, pr);
  const Tw8 wd = tw8_load(pr.fwd, 512 * tile, mD, (uint32_t)t);
  if (pr.q >= kFwdLazy) {   // uniform
    red8(x, pr);
    red8(y, pr);
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    sh[lds_b(lp, k)] = x[k];
    sh2[lds_b(lp, k)] = y[k];
  }
  lds_wave_sync();   // rounds B and C touch the same 512 elements of this wave's block
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    x[k] = sh[lds_c(lp, k)];
    y[k] = sh2[lds_c(lp, k)];
  }
  radix8_ct_w(x, wc, pr);
  radix8_ct_w(y, wc, pr);
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    sh[lds_c(lp, k)] = x[k];
    sh2[lds_c(lp, k)] = y[k];
  }
  lds_wave_sync();   // and so do rounds C and D
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    x[k] = sh[lds_d(lp, k)];
    y[k] = sh2[lds_d(lp, k)];
  }
  radix8_ct_w(x, wd, pr);
  radix8_ct_w(y, wd, pr);
  // each thread overwrites only the LDS words it just read
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    sh[lds_d(lp, k)] = x[k];
    sh2[lds_d(lp, k)] = y[k];
  }
  lds_barrier();
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    x[k] = sh[lds_a(lp, k)];
    y[k] = sh2[lds_a(lp, k)];
  }
}

__device__ __forceinline__ void row4_inv_tile2(size_t gb0, int S1, const DevPrime& pr, double* sh, double* sh2,
                                               const double va[8], const double vb[8], double x[8], double y[8]) {
  const int t = threadIdx.x;
  const uint32_t mA = 1u << S1, mB = mA << 3, mC = mA << 6, mD = mA << 9, tile = (uint32_t)(gb0 >> 12);
  const LdsPlace lp = lds_place();
  const uint32_t wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const Tw8 wd = tw8_load(pr.inv, 512 * tile, mD, (uint32_t)t);
  const Tw8 wc = tw8_load(pr.inv, 64 * tile, mC, (uint32_t)t >> 3);
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    sh[lds_a(lp, k)] = va[k];
    sh2[lds_a(lp, k)] = vb[k];
  }
  lds_barrier();
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    x[k] = sh[lds_d(lp, k)];
    y[k] = sh2[lds_d(lp, k)];
  }
  radix8_gs_w(x, wd, pr);
  radix8_gs_w(y, wd, pr);
  const Tw8 wb = tw8_scalar(pr.inv, 8 * tile + wave, mB);
  if (pr.q >= kInvLazy) {   // uniform
    red8(x, pr);
    red8(y, pr);
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    sh[lds_d(lp, k)] = x[k];
    sh2[lds_d(lp, k)] = y[k];
  }
  lds_wave_sync();   // rounds D and C touch the same 512 elements of this wave's block
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    x[k] = sh[lds_c(lp, k)];
    y[k] = sh2[lds_c(lp, k)];
  }
  radix8_gs_w(x, wc, pr);
  radix8_gs_w(y, wc, pr);
  const Tw8 wa = tw8_scalar(pr.inv, tile, mA);
  red8(x, pr);
  red8(y, pr);
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    sh[lds_c(lp, k)] = x[k];
    sh2[lds_c(lp, k)] = y[k];
  }
  lds_wave_sync();   // and so do rounds C and B
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    x[k] = sh[lds_b(lp, k)];
    y[k] = sh2[lds_b(lp, k)];
  }
  radix8_gs_w(x, wb, pr);
  radix8_gs_w(y, wb, pr);
  if (pr.q >= kInvLazy) {
    red8(x, pr);
    red8(y, pr);
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    sh[lds_b(lp, k)] = x[k];
    sh2[lds_b(lp, k)] = y[k];
  }
  lds_barrier();
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    x[k] = sh[lds_a(lp, k)];
    y[k] = sh2[lds_a(lp, k)];
  }
  radix8_gs_w(x, wa, pr);
  radix8_gs_w(y, wa, pr);
}

}  // namespace copse
