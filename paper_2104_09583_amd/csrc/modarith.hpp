// Device arithmetic shared by the kernel files: modular products and reductions on fp64 residues, loads of
// known address spaces, LDS waits.
#pragma once

#include <type_traits>

#include "internal.hpp"

namespace copse {

// ------------------------------------------------------------------ modular arithmetic in fp64
__device__ __forceinline__ double mod_mul(double a, double b, double q, double qinv) {
  double h = a * b;
  double l = __fma_rn(a, b, -h);
  double k = floor(h * qinv);
  double r = __fma_rn(-k, q, h) + l;
  r = (r < 0.0) ? r + q : r;
  r = (r >= q) ? r - q : r;
  return r;
}
__device__ __forceinline__ double mod_add(double a, double b, double q) {
  double s = a + b;
  return (s >= q) ? s - q : s;
}
__device__ __forceinline__ double mod_sub(double a, double b, double q) {
  double s = a - b;
  return (s < 0.0) ? s + q : s;
}
// reduce an exact integer |v| < 2^52 into [0, q)
__device__ __forceinline__ double mod_reduce(double v, double q, double qinv) {
  double k = floor(v * qinv);
  double r = __fma_rn(-k, q, v);
  r = (r < 0.0) ? r + q : r;
  r = (r >= q) ? r - q : r;
  return r;
}

// Lazy (signed) residues for the transforms, for q < 2^49 and |b| < q:
//   mul_lazy: k = rint(a b / q) is off by three roundings (of a b, of 1 / q, of their product), so r = a b - k q =
//   fma(-k, q, h) + l is an exact integer with |r| <= (0.5 + 3 x 2^-53 |a|) q: 0.69 q for |a| < q, 0.875 q for
//   |a| <= 2^50, and below q for |a| <= 4 q as well (for q > 2^48 the roundings are within 2^46 / q, 4 q^2 2^-102 and
//   2^-3, together 0.5 at 2^49);
//   reduce_sym: x - q rint(x / q) lies in [-q/2, q/2] for |x| < 8 q;
//   canon: maps [-q/2, q/2] to [0, q), and (-q, q) too.
// Forward, a stage adds one such product to |x|: from |x| <= q six stages reach at most 7.6 q < 2^52 for
// q = 2^49, every value still an exact integer, so the row pass folds back once, after its second radix-8
// round; for q < 2^46 (kFwdLazy) its twelve stages stay below 20 q even from 8 q, and it never does.  Inverse, a
// stage doubles the sums: 2^3 per round, folded back after every round, or for q < 2^44 (kInvLazy) after every second
// one (64 q <= 2^50).  For q < 2^42 (kInvOpen) the inverse row pass
// also leaves its output unreduced (32 q): three column stages that follow reach 256 q <= 2^50, where the
// next product is still within 0.875 q (four: 512 q, within 1.25 q and folded back there).
constexpr double kFwdLazy = 70368744177664.0;   // 2^46
constexpr double kInvLazy = 17592186044416.0;   // 2^44
constexpr double kInvOpen = 4398046511104.0;    // 2^42
__device__ __forceinline__ double mul_lazy(double a, double b, double q, double qinv) {
  double h = a * b;
  double l = __fma_rn(a, b, -h);
  double k = rint(h * qinv);
  return __fma_rn(-k, q, h) + l;
}
__device__ __forceinline__ double reduce_sym(double x, double q, double qinv) {
  return __fma_rn(-rint(x * qinv), q, x);
}
__device__ __forceinline__ double canon(double x, double q) { return __fma_rn(x < 0.0 ? 1.0 : 0.0, q, x); }

// A load known to be from global memory (not through a flat address).  Flat loads count on the same
// wait counter as LDS and scalar loads, so every LDS wait before a barrier would also wait for them;
// global loads count only on the vector-memory counter.
__device__ __forceinline__ double gload(const double* p) {
  return *(const __attribute__((address_space(1))) double*)(p);
}
// A pointer that is the same for the whole wave, kept in scalar registers: without this the compiler adds constant
// offsets beyond the instruction's range to a 64-bit address in every lane.
template <class T>
__device__ __forceinline__ T* uniform(T* p) {
  asm("" : "+s"(p));
  return p;
}
// global load from a uniform base and a 32-bit byte offset per lane
__device__ __forceinline__ double gload_off(const double* p, uint32_t bytes) {
  return *(const __attribute__((address_space(1))) double*)((const char*)p + (size_t)bytes);
}
// Packed rows: N values of |x| < 2^47 in six bytes each, as N 32-bit words followed by N 16-bit words of x + 2^47.
// 2^52 + 2^47 + x has the sum in its low mantissa bits, so packing is an addition and unpacking an or and a
// subtraction.
constexpr double kPackBias = 4503599627370496.0 + 140737488355328.0;   // 2^52 + 2^47
__device__ __forceinline__ double unpack48(uint32_t lo, uint32_t hi) {
  return __hiloint2double((int)(0x43300000u | hi), (int)lo) - kPackBias;
}
__device__ __forceinline__ void pack48(double x, uint32_t& lo, uint16_t& hi) {
  const double d = x + kPackBias;
  lo = (uint32_t)__double2loint(d);
  hi = (uint16_t)__double2hiint(d);
}
__device__ __forceinline__ uint32_t gload32_off(const uint32_t* p, uint32_t bytes) {
  return *(const __attribute__((address_space(1))) uint32_t*)((const char*)p + (size_t)bytes);
}
__device__ __forceinline__ uint32_t gload16_off(const uint16_t* p, uint32_t bytes) {
  return *(const __attribute__((address_space(1))) uint16_t*)((const char*)p + (size_t)bytes);
}
// row r of a block of packed or plain rows of N values
__device__ __forceinline__ const double* row_at(const double* base, size_t r, size_t N, bool packed) {
  return base + r * (packed ? N / 4 * 3 : N);
}
// A load of a value that is uniform across the wave from a table no kernel writes (twiddles, row
// descriptors, primes, conversion constants): read through the constant address space, so it is a scalar
// load into scalar registers.
template <class T>
__device__ __forceinline__ T cload(const T* p) {
  static_assert(std::is_scalar<T>::value, "scalar loads take numbers and pointers");
  return *(const __attribute__((address_space(4))) T*)(p);
}
__device__ __forceinline__ int2 cload_row(const int2* p) {
  const int* w = reinterpret_cast<const int*>(p);
  return make_int2(cload(w), cload(w + 1));
}
// the fields of a prime the transforms use (q, 1/q, twiddle tables, N^-1)
__device__ __forceinline__ DevPrime cload_prime(const DevPrime* p) {
  DevPrime r;
  r.q = cload(&p->q);
  r.qinv = cload(&p->qinv);
  r.fwd = cload(&p->fwd);
  r.inv = cload(&p->inv);
  r.ninv = cload(&p->ninv);
  return r;
}
// Workgroup barrier for LDS exchanges: waits for this wave's LDS accesses only, so global loads issued
// before it (the next round's twiddles, an epilogue's operands) stay in flight across it.  The memory
// clobber keeps the compiler from moving LDS accesses across it.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
// An LDS exchange among the lanes of one wave: its writes are complete before its next reads are issued
// (no other wave takes part, so no workgroup barrier)
__device__ __forceinline__ void lds_wave_sync() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// One column of the 2^S1 x C matrix view in registers: the transform's first S1 stages (forward) or its last
// (inverse), one butterfly at a time (see the transform's comment in kernels.hip).
__device__ __forceinline__ void bfly_ct(double& x, double& y, double w, double q, double qinv) {
  double v = mul_lazy(y, w, q, qinv);
  double u = x;
  x = u + v;
  y = u - v;
}
__device__ __forceinline__ void bfly_gs(double& x, double& y, double w, double q, double qinv) {
  double u = x, v = y;
  x = u + v;
  y = mul_lazy(u - v, w, q, qinv);
}

}  // namespace copse
