// Host utilities: errors, number theory, SHAKE-256 (FIPS 202) and the
// samplers, and the device memory pool.
#include <algorithm>
#include <cstring>

#include "internal.hpp"

namespace copse {

[[noreturn]] void fail(int code, const std::string& msg) { throw Error{code, msg}; }

// ------------------------------------------------------------------ number theory
uint64_t mulmod(uint64_t a, uint64_t b, uint64_t m) {
  return (uint64_t)((unsigned __int128)a * b % m);
}

uint64_t powmod(uint64_t a, uint64_t e, uint64_t m) {
  uint64_t r = 1 % m;
  a %= m;
  while (e) {
    if (e & 1) r = mulmod(r, a, m);
    a = mulmod(a, a, m);
    e >>= 1;
  }
  return r;
}

// Extended Euclid; m need not be prime.
uint64_t invmod(uint64_t a, uint64_t m) {
  __int128 t0 = 0, t1 = 1, r0 = m, r1 = a % m;
  while (r1 != 0) {
    __int128 qq = r0 / r1, tmp;
    tmp = r0 - qq * r1; r0 = r1; r1 = tmp;
    tmp = t0 - qq * t1; t0 = t1; t1 = tmp;
  }
  if (r0 != 1) fail(COPSE_EINVAL, "value not invertible");
  if (t0 < 0) t0 += m;
  return (uint64_t)t0;
}

// Miller-Rabin with the first twelve primes as bases: deterministic for all 64-bit n.
bool is_prime(uint64_t n) {
  static const uint64_t bases[] = {2, 3, 5, 7, 11, 13, 17, 19, 23, 29, 31, 37};
  if (n < 2) return false;
  for (uint64_t p : bases)
    if (n % p == 0) return n == p;
  uint64_t d = n - 1;
  int s = 0;
  while ((d & 1) == 0) { d >>= 1; ++s; }
  for (uint64_t a : bases) {
    uint64_t x = powmod(a, d, n);
    if (x == 1 || x == n - 1) continue;
    bool comp = true;
    for (int i = 1; i < s; ++i) {
      x = mulmod(x, x, n);
      if (x == n - 1) { comp = false; break; }
    }
    if (comp) return false;
  }
  return true;
}

// An element of exact multiplicative order `order` (a power of two here) mod prime q.
uint64_t root_of_unity(uint64_t order, uint64_t q) {
  if ((q - 1) % order) fail(COPSE_EINVAL, "order does not divide q-1");
  for (uint64_t g = 2; g < q; ++g) {
    uint64_t r = powmod(g, (q - 1) / order, q);
    // order is a power of two: r has exact order iff r^(order/2) = -1
    if (powmod(r, order / 2, q) == q - 1) return r;
  }
  fail(COPSE_EINVAL, "no root of unity");
}

uint32_t bitrev(uint32_t x, int bits) {
  uint32_t r = 0;
  for (int i = 0; i < bits; ++i) { r = (r << 1) | (x & 1); x >>= 1; }
  return r;
}

// ------------------------------------------------------------------ Keccak-f[1600] / SHAKE-256
namespace {
struct KeccakConsts {
  uint64_t rc[24] = {};
  int rho[25] = {};
  constexpr KeccakConsts() {
    // round constants from the LFSR rc(t) of FIPS 202, Algorithm 5
    for (int ir = 0; ir < 24; ++ir)
      for (int j = 0; j <= 6; ++j) {
        const int t = (j + 7 * ir) % 255;
        unsigned R = 0x01;  // bits R[0..7] = 1,0,...,0
        for (int i = 1; i <= t; ++i) {
          R <<= 1;                       // R = 0 || R   (R[8] is the old R[7])
          const unsigned r8 = (R >> 8) & 1;
          R ^= r8 | (r8 << 4) | (r8 << 5) | (r8 << 6);
          R &= 0xFF;
        }
        if (R & 1) rc[ir] |= 1ULL << ((1 << j) - 1);
      }
    // rho offsets (FIPS 202, Algorithm 2)
    int x = 1, y = 0;
    for (int t = 0; t < 24; ++t) {
      rho[x + 5 * y] = ((t + 1) * (t + 2) / 2) % 64;
      const int ny = (2 * x + 3 * y) % 5;
      x = y;
      y = ny;
    }
  }
};
constexpr KeccakConsts kKeccak;

// One state (V = uint64_t) or eight independent ones in the lanes of V.
typedef uint64_t Lanes8 __attribute__((vector_size(64)));
template <class V>
inline __attribute__((always_inline)) V rotl(V v, int r) { return r ? (v << r) | (v >> (64 - r)) : v; }

template <class V>
inline __attribute__((always_inline)) void keccak_rounds(V* st) {
  V A[25];
#pragma unroll
  for (int i = 0; i < 25; ++i) A[i] = st[i];
  for (int ir = 0; ir < 24; ++ir) {
    V C[5], D[5], B[25];
#pragma unroll
    for (int x = 0; x < 5; ++x) C[x] = A[x] ^ A[x + 5] ^ A[x + 10] ^ A[x + 15] ^ A[x + 20];
#pragma unroll
    for (int x = 0; x < 5; ++x) D[x] = C[(x + 4) % 5] ^ rotl(C[(x + 1) % 5], 1);
    // rho and pi: B[y, 2x+3y] = rot(A[x, y])
#pragma unroll
    for (int x = 0; x < 5; ++x)
#pragma unroll
      for (int y = 0; y < 5; ++y) B[y + 5 * ((2 * x + 3 * y) % 5)] = rotl(A[x + 5 * y] ^ D[x], kKeccak.rho[x + 5 * y]);
#pragma unroll
    for (int x = 0; x < 5; ++x)
#pragma unroll
      for (int y = 0; y < 5; ++y)
        A[x + 5 * y] = B[x + 5 * y] ^ (~B[(x + 1) % 5 + 5 * y] & B[(x + 2) % 5 + 5 * y]);
    A[0] ^= kKeccak.rc[ir];
  }
#pragma unroll
  for (int i = 0; i < 25; ++i) st[i] = A[i];
}
void keccak_f(uint64_t A[25]) { keccak_rounds<uint64_t>(A); }
// eight states at once, for the widest vectors that the processor has
__attribute__((target("avx512f"))) void keccak8_avx512(Lanes8* st) { keccak_rounds<Lanes8>(st); }
__attribute__((target("avx2"))) void keccak8_avx2(Lanes8* st) { keccak_rounds<Lanes8>(st); }
void keccak8_base(Lanes8* st) { keccak_rounds<Lanes8>(st); }
void keccak8(Lanes8* st) {
  static void (*const f)(Lanes8*) = __builtin_cpu_supports("avx512f") ? keccak8_avx512
                                    : __builtin_cpu_supports("avx2")  ? keccak8_avx2
                                                                      : keccak8_base;
  f(st);
}
constexpr size_t kRate = 136;

void absorb_all(uint64_t st[25], const uint8_t* msg, size_t len) {
  std::memset(st, 0, 25 * sizeof(uint64_t));
  uint8_t block[kRate];
  size_t off = 0;
  while (true) {
    size_t take = std::min(kRate, len - off);
    std::memset(block, 0, kRate);
    std::memcpy(block, msg + off, take);
    bool last = take < kRate;
    if (last) {
      block[take] ^= 0x1F;          // SHAKE domain bits + first pad bit
      block[kRate - 1] ^= 0x80;     // last pad bit
    }
    for (size_t i = 0; i < kRate / 8; ++i) {
      uint64_t lane = 0;
      for (int b = 0; b < 8; ++b) lane |= (uint64_t)block[8 * i + b] << (8 * b);
      st[i] ^= lane;
    }
    keccak_f(st);
    off += take;
    if (last) break;
  }
}
}  // namespace

void shake256(const uint8_t* msg, size_t len, uint8_t* out, size_t outlen) {
  uint64_t st[25];
  absorb_all(st, msg, len);
  size_t done = 0;
  while (done < outlen) {
    size_t take = std::min(kRate, outlen - done);
    for (size_t i = 0; i < take; ++i) out[done + i] = (uint8_t)(st[i / 8] >> (8 * (i % 8)));
    done += take;
    if (done < outlen) keccak_f(st);
  }
}

ShakeStream::ShakeStream(const uint8_t seed[32], const char* domain, uint64_t obj, uint32_t limb) {
  std::vector<uint8_t> msg(seed, seed + 32);
  for (const char* p = domain; *p; ++p) msg.push_back((uint8_t)*p);
  for (int i = 0; i < 8; ++i) msg.push_back((uint8_t)(obj >> (8 * i)));
  for (int i = 0; i < 4; ++i) msg.push_back((uint8_t)(limb >> (8 * i)));
  absorb_all(st_, msg.data(), msg.size());
  permute_block();
}

void ShakeStream::permute_block() {
  // st_ already permuted: expose its first rate bytes
  for (size_t i = 0; i < kRate; ++i) buf_[i] = (uint8_t)(st_[i / 8] >> (8 * (i % 8)));
  pos_ = 0;
}

void ShakeStream::read(uint8_t* out, size_t n) {
  for (size_t i = 0; i < n; ++i) {
    if (pos_ == kRate) {
      keccak_f(st_);
      permute_block();
    }
    out[i] = buf_[pos_++];
  }
}

namespace {
// Up to eight SHAKE-256 streams of SHAKE256(seed || domain || le64(object) || le32(limb)), squeezed together a block
// (136 bytes of every stream) at a time.  A stream is one chain of permutations, so the eight run in the lanes of one
// vector: with 512-bit registers a permutation of all eight takes 0.45 us, of one alone 0.43 us (on one host; eight
// plaintexts' randomness, N = 32768, takes 17.6 ms there one stream at a time, 1.8 ms so).
class ShakeStreams {
 public:
  ShakeStreams(const uint8_t seed[32], int n) : n_(n) { std::memcpy(seed_, seed, 32); }
  void set(int lane, const char* domain, uint64_t obj, uint32_t limb) {
    std::vector<uint8_t> msg(seed_, seed_ + 32);
    for (const char* p = domain; *p; ++p) msg.push_back((uint8_t)*p);
    for (int i = 0; i < 8; ++i) msg.push_back((uint8_t)(obj >> (8 * i)));
    for (int i = 0; i < 4; ++i) msg.push_back((uint8_t)(limb >> (8 * i)));
    uint64_t st[25];
    absorb_all(st, msg.data(), msg.size());
    for (int i = 0; i < 25; ++i) {
      if (n_ == 1) one_[i] = st[i];
      else st_[i][lane] = st[i];
    }
  }
  // the next `blocks` blocks of every stream: stream l's to out[l]
  void squeeze(uint8_t* const* out, size_t blocks) {
    for (size_t b = 0; b < blocks; ++b) {
      if (fresh_) fresh_ = false;
      else if (n_ == 1) keccak_f(one_);
      else keccak8(st_);
      for (int l = 0; l < n_; ++l) {
        uint64_t w[kRate / 8];
        for (size_t i = 0; i < kRate / 8; ++i) w[i] = n_ == 1 ? one_[i] : st_[i][l];
        std::memcpy(out[l] + b * kRate, w, kRate);
      }
    }
  }

 private:
  uint8_t seed_[32];
  int n_;
  bool fresh_ = true;   // absorbing leaves the first block in place
  uint64_t one_[25];
  Lanes8 st_[25] = {};
};
static_assert(__BYTE_ORDER__ == __ORDER_LITTLE_ENDIAN__, "blocks are copied out as little-endian words");

constexpr size_t blocks_of(size_t bytes) { return (bytes + kRate - 1) / kRate; }

// Draws from n <= 8 streams until each has `count` values: take(lane, block bytes) returns how many values the lane
// has so far.
template <class Take>
void draw_streams(ShakeStreams& s, int n, size_t first_blocks, size_t count, Take take) {
  std::vector<uint8_t> buf;
  for (size_t blocks = first_blocks;; blocks = 1) {
    buf.resize((size_t)n * blocks * kRate);
    uint8_t* out[8];
    for (int l = 0; l < n; ++l) out[l] = buf.data() + (size_t)l * blocks * kRate;
    s.squeeze(out, blocks);
    bool done = true;
    for (int l = 0; l < n; ++l) done = take(l, out[l], blocks * kRate) >= count && done;
    if (done) return;
  }
}

struct TernaryTable {
  int8_t v[256];
  constexpr TernaryTable() : v() {
    for (int b = 0; b < 256; ++b) v[b] = (int8_t)(b % 3 == 2 ? -1 : b % 3);
  }
};
constexpr TernaryTable kTernary;

void ternary_streams(ShakeStreams& s, int n, size_t count, int8_t* const* out) {
  size_t got[8] = {};
  draw_streams(s, n, blocks_of(count + count / 200 + 16), count, [&](int l, const uint8_t* b, size_t len) {
    size_t g = got[l];
    for (size_t i = 0; i < len && g < count; ++i) {
      out[l][g] = kTernary.v[b[i]];
      g += b[i] != 255;
    }
    return got[l] = g;
  });
}
}  // namespace

void sample_uniform_limbs(const uint8_t seed[32], const char* dom, uint64_t obj, uint32_t first_limb,
                          const std::vector<uint64_t>& q, size_t n, double* out) {
  for (size_t l0 = 0; l0 < q.size(); l0 += 8) {
    const int m = (int)std::min<size_t>(8, q.size() - l0);
    ShakeStreams s(seed, m);
    for (int l = 0; l < m; ++l) s.set(l, dom, obj, first_limb + (uint32_t)(l0 + l));
    size_t got[8] = {};
    draw_streams(s, m, blocks_of(8 * n + 8 * 17), n, [&](int l, const uint8_t* b, size_t len) {
      const uint64_t ql = q[l0 + l];
      const int bits = 64 - __builtin_clzll(ql);
      const uint64_t mask = bits >= 64 ? ~0ULL : ((1ULL << bits) - 1);
      double* o = out + (l0 + l) * n;
      size_t g = got[l];
      for (size_t i = 0; i + 8 <= len && g < n; i += 8) {   // a block holds 17 whole words
        uint64_t w;
        std::memcpy(&w, b + i, 8);
        w &= mask;
        o[g] = (double)w;
        g += w < ql;
      }
      return got[l] = g;
    });
  }
}

void sample_uniform(const uint8_t seed[32], const char* dom, uint64_t obj, uint32_t limb, uint64_t q,
                    size_t n, double* out) {
  sample_uniform_limbs(seed, dom, obj, limb, {q}, n, out);
}

void sample_ternary(const uint8_t seed[32], const char* dom, uint64_t obj, size_t n, int64_t* out) {
  ShakeStreams s(seed, 1);
  s.set(0, dom, obj, 0);
  std::vector<int8_t> v(n);
  int8_t* p[1] = {v.data()};
  ternary_streams(s, 1, n, p);
  std::copy(v.begin(), v.end(), out);
}

void sample_cbd21(const uint8_t seed[32], const char* dom, uint64_t obj, size_t n, int64_t* out) {
  ShakeStreams s(seed, 1);
  s.set(0, dom, obj, 0);
  const size_t blocks = blocks_of(6 * n);
  std::vector<uint8_t> b(blocks * kRate);
  uint8_t* p[1] = {b.data()};
  s.squeeze(p, blocks);
  for (size_t i = 0; i < n; ++i) {
    uint64_t w = 0;
    std::memcpy(&w, b.data() + 6 * i, 6);
    out[i] = __builtin_popcountll(w & ((1ULL << 21) - 1)) - __builtin_popcountll((w >> 21) & ((1ULL << 21) - 1));
  }
}

size_t encryption_noise_bytes(size_t n) { return n + 2 * blocks_of(6 * n) * kRate; }

void sample_encryption_many(const uint8_t seed[32], const uint64_t* objs, int count, size_t n, uint8_t* out) {
  const size_t stride = encryption_noise_bytes(n), blocks = blocks_of(6 * n);
  for (int p0 = 0; p0 < count; p0 += 8) {
    const int m = std::min(8, count - p0);
    ShakeStreams s(seed, m);
    int8_t* o[8];
    for (int l = 0; l < m; ++l) {
      s.set(l, "enc.u", objs[p0 + l], 0);
      o[l] = reinterpret_cast<int8_t*>(out + (size_t)(p0 + l) * stride);
    }
    ternary_streams(s, m, n, o);
  }
  for (int e0 = 0; e0 < 2 * count; e0 += 8) {   // error stream e: polynomial e % 2 of plaintext e / 2
    const int m = std::min(8, 2 * count - e0);
    ShakeStreams s(seed, m);
    uint8_t* o[8];
    for (int l = 0; l < m; ++l) {
      const int e = e0 + l;
      s.set(l, e % 2 ? "enc.e1" : "enc.e0", objs[e / 2], 0);
      o[l] = out + (size_t)(e / 2) * stride + n + (size_t)(e % 2) * blocks * kRate;
    }
    s.squeeze(o, blocks);
  }
}

// ------------------------------------------------------------------ pool
Pool::~Pool() {
  hipSetDevice(device_);
  for (auto& kv : cache_)
    for (void* p : kv.second) (void)hipFree(p);
  for (auto& kv : live_) (void)hipFree(kv.first);
}

static size_t round_size(size_t b) {
  if (b <= 4096) return 4096;
  size_t g = 1ULL << (63 - __builtin_clzll(b));
  size_t step = g / 8;   // 8 size classes per power of two
  return (b + step - 1) / step * step;
}

void* Pool::alloc(size_t bytes) {
  std::lock_guard<std::mutex> lk(mu_);
  size_t sz = round_size(bytes);
  auto it = cache_.find(sz);
  void* p = nullptr;
  if (it != cache_.end() && !it->second.empty()) {
    p = it->second.back();
    it->second.pop_back();
  } else {
    hipError_t e = hipMalloc(&p, sz);
    if (e != hipSuccess && !keep_cached_) {
      // release cached blocks and retry once
      for (auto& kv : cache_) {
        for (void* q : kv.second) { (void)hipFree(q); held_ -= kv.first; }
        kv.second.clear();
      }
      (void)hipGetLastError();
      e = hipMalloc(&p, sz);
    }
    if (e != hipSuccess) {
      (void)hipGetLastError();
      fail(COPSE_ENOMEM, "device allocation of " + std::to_string(sz) + " bytes failed");
    }
    held_ += sz;
  }
  live_[p] = sz;
  live_bytes_ += sz;
  peak_bytes_ = std::max(peak_bytes_, live_bytes_);
  return p;
}

void Pool::free(void* p) {
  if (!p) return;
  std::lock_guard<std::mutex> lk(mu_);
  auto it = live_.find(p);
  if (it == live_.end()) return;
  cache_[it->second].push_back(p);
  live_bytes_ -= it->second;
  live_.erase(it);
}

size_t Pool::live_bytes() {
  std::lock_guard<std::mutex> lk(mu_);
  return live_bytes_;
}

size_t Pool::peak_bytes() {
  std::lock_guard<std::mutex> lk(mu_);
  return peak_bytes_;
}

void Pool::reset_peak() {
  std::lock_guard<std::mutex> lk(mu_);
  peak_bytes_ = live_bytes_;
}

void Pool::trim() {
  std::lock_guard<std::mutex> lk(mu_);
  if (keep_cached_) return;
  for (auto& kv : cache_) {
    for (void* q : kv.second) { (void)hipFree(q); held_ -= kv.first; }
    kv.second.clear();
  }
}

}  // namespace copse
