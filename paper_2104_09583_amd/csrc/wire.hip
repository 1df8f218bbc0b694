// The data owner's and the wire's side of the boundary on the device: residues to and from 64-bit words
// (ciphertext import and export), slot vectors to plaintext polynomials and back (the transform modulo t, run
// by the ring transform's kernels with t as one more prime), and encryption of several plaintexts at once.
//
// All of it is bound by launches and by the copy to or from the caller's pageable memory, not by arithmetic,
// so the kernels are one pass each and fold in what the host did before: range checks, centering, the
// multiplication by t, the noise check.
#include <algorithm>

#include "internal.hpp"
#include "modarith.hpp"

namespace copse {

constexpr int kWireThreads = 256;
static dim3 wire_grid(const Context& c, int rows, int z = 1) {
  return dim3((unsigned)((c.N + kWireThreads - 1) / kWireThreads), rows, z);
}

// ------------------------------------------------------------------ residues <-> 64-bit words
// rows of nl limbs (row r: prime r % nl).  In place: a word and its residue share their eight bytes.
__global__ void words_to_residues_kernel(double* io, int nl, const DevPrime* P, int logN, int* bad) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (size_t)1 << logN) return;
  const size_t o = ((size_t)blockIdx.y << logN) + i;
  const uint64_t v = reinterpret_cast<const uint64_t*>(io)[o];
  const bool ok = v < (uint64_t)P[blockIdx.y % nl].q;
  if (!ok) *bad = 1;
  io[o] = ok ? (double)v : 0.0;
}
__global__ void residues_to_words_kernel(uint64_t* out, const double* in, int logN) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (size_t)1 << logN) return;
  const size_t o = ((size_t)blockIdx.y << logN) + i;
  out[o] = (uint64_t)in[o];
}

// The column pass with the conversion folded in, for the rings of the split transform (N = 2^13 .. 2^16): one
// thread keeps one column (2^S1 elements, C = N >> S1 apart) in registers.
//   forward (import): words from `words`, checked against the prime, then stages 0 .. S1 - 1; signed output for the row
//   pass to `io`
//   inverse (export): the row pass's signed output in `io` (< 32 q), the last stages, N^-1, canonical words to `words`
// words and io may be the same memory: a thread has read its column before it writes it.  Where words is pinned host
// memory, the loads and stores cross the bus and no copy stands before or after.
// Bound by the copy from or to the caller's memory.  A request of eight planes (42 MB) in, one evaluation, its result
// out: 5.50 ms with the conversion loops on the host, 3.14 ms here, of which the copy in takes 1.2 and the evaluation
// 1.4.
template <int S1, bool kInverse>
__global__ __launch_bounds__(64) void wire_cols_kernel(double* io, uint64_t* words, int nl,
                                                       const DevPrime* __restrict__ P, int logN, int* bad) {
  constexpr int R = 1 << S1;
  const size_t C = (size_t)1 << (logN - S1);
  const size_t col = (size_t)blockIdx.x * 64 + threadIdx.x;
  if (col >= C) return;
  const DevPrime pr = P[blockIdx.y % nl];
  double* a = io + ((size_t)blockIdx.y << logN) + col;
  uint64_t* w = words + ((size_t)blockIdx.y << logN) + col;
  double x[R];
  if (!kInverse) {
    const uint64_t q = (uint64_t)pr.q;
    bool ok = true;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const uint64_t v = w[r * C];
      ok = ok && v < q;
      x[r] = v < q ? (double)v : 0.0;
    }
    if (!ok) *bad = 1;
#pragma unroll
    for (int s = 0; s < S1; ++s) {
      const int half = R >> (s + 1);
#pragma unroll
      for (int g = 0; g < (1 << s); ++g) {
        const double w = pr.fwd[(1 << s) + g];
#pragma unroll
        for (int o = 0; o < half; ++o) bfly_ct(x[g * 2 * half + o], x[g * 2 * half + o + half], w, pr.q, pr.qinv);
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) a[r * C] = reduce_sym(x[r], pr.q, pr.qinv);
  } else {
#pragma unroll
    for (int r = 0; r < R; ++r) x[r] = a[r * C];
#pragma unroll
    for (int s = S1 - 1; s >= 0; --s) {
      const int half = R >> (s + 1);
#pragma unroll
      for (int g = 0; g < (1 << s); ++g) {
        const double w = pr.inv[(1 << s) + g];
#pragma unroll
        for (int o = 0; o < half; ++o) bfly_gs(x[g * 2 * half + o], x[g * 2 * half + o + half], w, pr.q, pr.qinv);
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const double v = canon(reduce_sym(mul_lazy(x[r], pr.ninv, pr.q, pr.qinv), pr.q, pr.qinv), pr.q);
      w[r * C] = (uint64_t)v;
    }
  }
}

template <bool kInverse>
static void launch_wire_cols(Context& c, double* io, uint64_t* out, int rows, int nl, int* bad) {
  const int logN = (int)c.log_n, S1 = logN - 12;
  const dim3 grid((unsigned)(((c.N >> S1) + 63) / 64), rows);
  switch (S1) {
    case 1: hipLaunchKernelGGL((wire_cols_kernel<1, kInverse>), grid, dim3(64), 0, c.stream, io, out, nl, c.d_primes, logN, bad); break;
    case 2: hipLaunchKernelGGL((wire_cols_kernel<2, kInverse>), grid, dim3(64), 0, c.stream, io, out, nl, c.d_primes, logN, bad); break;
    case 3: hipLaunchKernelGGL((wire_cols_kernel<3, kInverse>), grid, dim3(64), 0, c.stream, io, out, nl, c.d_primes, logN, bad); break;
    default: hipLaunchKernelGGL((wire_cols_kernel<4, kInverse>), grid, dim3(64), 0, c.stream, io, out, nl, c.d_primes, logN, bad); break;
  }
  COPSE_HIP(hipGetLastError());
}

// rows of an [np][nl][N] block with primes 0..nl-1
static const int2* limb_rows(Context& c, int np, int nl) {
  const std::string key = "ct:" + std::to_string(np) + ":" + std::to_string(nl);
  auto it = c.row_tables.find(key);
  if (it != c.row_tables.end()) return it->second;
  std::vector<int2> h;
  for (int k = 0; k < np; ++k)
    for (int i = 0; i < nl; ++i) h.push_back(make_int2(k * nl + i, i));
  return c.rows(key, h);
}

// A ciphertext's coefficient words to `out` (device-visible; tmp's own memory too), enqueued
static void ct_words(Context& c, const Ct& a, DBuf& tmp, uint64_t* out) {
  const int nl = a.level + 1, rows = a.npolys * nl;
  if (bridge_supported(c, 1)) {
    std::vector<const double*> polys;
    for (int k = 0; k < a.npolys; ++k) polys.push_back(a.poly(k, c.N));
    launch_ntt_inv_rows_gather(c, tmp.get(), polys, nl, c.N, 0, -1);
    launch_wire_cols<true>(c, tmp.get(), out, rows, nl, nullptr);
    return;
  }
  launch_copy(c, tmp.get(), a.data(), a.words());
  launch_ntt_inv(c, tmp.get(), limb_rows(c, a.npolys, nl), rows);
  hipLaunchKernelGGL(residues_to_words_kernel, wire_grid(c, rows), dim3(kWireThreads), 0, c.stream, out, tmp.get(),
                     (int)c.log_n);
  COPSE_HIP(hipGetLastError());
}

// Two pinned slots: a ciphertext's words are written into one by the kernel that makes them while the host copies the
// other out to the caller's buffer (the runtime's copy to pageable memory is a staging kernel and a wait of its own).
// Against copying from device memory: 16 results exported after a batched evaluation 16.68 -> 16.39 ms together, a fresh
// group of eight planes (42 MB, to fresh pages) encrypted and exported 5.41 -> 4.28 ms.  A ciphertext beyond a slot
// goes through device memory, in the one buffer that it needs in any case.
constexpr size_t kExportSlotMax = (size_t)8 << 20;

// slots of at least min(need, kExportSlotMax) bytes where the system has that much pinned memory left; where it has not,
// they stay as they are, and what does not fit them goes through device memory too
static void wire_slots(Context& c, size_t need) {
  need = std::min(need, kExportSlotMax);
  for (int k = 0; k < 2; ++k)
    if (!c.export_done[k]) COPSE_HIP(hipEventCreateWithFlags(&c.export_done[k], hipEventDisableTiming));
  if (need <= c.export_slot_bytes) return;
  COPSE_HIP(hipStreamSynchronize(c.stream));   // an import may still be read
  void* grown[2] = {nullptr, nullptr};
  for (int k = 0; k < 2; ++k)
    if (hipHostMalloc(&grown[k], need, hipHostMallocDefault) != hipSuccess) {
      (void)hipGetLastError();
      if (k == 1) (void)hipHostFree(grown[0]);
      return;
    }
  for (int k = 0; k < 2; ++k) {
    if (c.export_slot[k]) (void)hipHostFree(c.export_slot[k]);
    c.export_slot[k] = static_cast<char*>(grown[k]);
  }
  c.export_slot_bytes = need;
}

void export_cts(Context& c, const std::vector<const Ct*>& cts, uint64_t* buf) {
  size_t need = 0;
  for (const Ct* a : cts) need = std::max(need, a->words() * 8);
  wire_slots(c, need);
  struct Pending {
    uint64_t* to = nullptr;
    size_t bytes = 0;
  } pending[2];
  auto finish = [&](int slot) {
    if (!pending[slot].to) return;
    COPSE_HIP(hipEventSynchronize(c.export_done[slot]));
    std::memcpy(pending[slot].to, c.export_slot[slot], pending[slot].bytes);
    pending[slot].to = nullptr;
  };
  int slot = 0;
  for (const Ct* a : cts) {
    *buf++ = (uint64_t)a->npolys;
    *buf++ = (uint64_t)a->level;
    *buf++ = (uint64_t)c.N;
    *buf++ = 0;
    const size_t bytes = a->words() * 8;
    DBuf tmp(&c, a->words());
    if (bytes > c.export_slot_bytes) {
      ct_words(c, *a, tmp, reinterpret_cast<uint64_t*>(tmp.get()));
      COPSE_HIP(hipMemcpyAsync(buf, tmp.get(), bytes, hipMemcpyDeviceToHost, c.stream));
      COPSE_HIP(hipStreamSynchronize(c.stream));
    } else {
      finish(slot);
      ct_words(c, *a, tmp, reinterpret_cast<uint64_t*>(c.export_slot[slot]));
      COPSE_HIP(hipEventRecord(c.export_done[slot], c.stream));
      pending[slot].to = buf;
      pending[slot].bytes = bytes;
      slot ^= 1;
      finish(slot);   // the ciphertext before, while this one's words are written
    }
    buf += a->words();
  }
  finish(slot ^ 1);
}

// Words through a pinned slot up to this size: a result (0.5 MB) imported and decrypted takes 131 against 138 us with a
// copy from pageable memory, a small ring's request (eight planes of 2 MB) imported, evaluated and exported 0.80 against
// 0.85 ms; planes of 5 MB are copied by the host more slowly than by the runtime (3.13 against 3.00 ms).
constexpr size_t kImportSlotMax = (size_t)2 << 20;

// A ciphertext from coefficient words in caller memory, enqueued; *bad (device) becomes 1 when a word is not
// below its prime.  `words` must stay valid until the stream has been synchronized.
CtPtr ct_from_words(Context& c, const uint64_t* words, int level, int npolys, int* bad) {
  auto ct = ct_alloc(c, level, npolys);
  const int nl = level + 1, rows = npolys * nl;
  const size_t bytes = ct->words() * 8;
  const bool through_slot = bridge_supported(c, 1) && bytes <= kImportSlotMax;
  if (through_slot) wire_slots(c, bytes);
  if (through_slot && bytes <= c.export_slot_bytes) {
    const int slot = c.import_slot;
    c.import_slot ^= 1;
    COPSE_HIP(hipEventSynchronize(c.export_done[slot]));   // what last read or wrote the slot
    std::memcpy(c.export_slot[slot], words, bytes);
    launch_wire_cols<false>(c, ct->data(), reinterpret_cast<uint64_t*>(c.export_slot[slot]), rows, nl, bad);
    COPSE_HIP(hipEventRecord(c.export_done[slot], c.stream));
    launch_ntt_fwd_rows(c, ct->data(), limb_rows(c, npolys, nl), rows);
    return ct;
  }
  // a larger one as it is: the runtime pins the caller's pages and copies at the bus's rate
  COPSE_HIP(hipMemcpyAsync(ct->data(), words, bytes, hipMemcpyHostToDevice, c.stream));
  if (bridge_supported(c, 1)) {
    launch_wire_cols<false>(c, ct->data(), reinterpret_cast<uint64_t*>(ct->data()), rows, nl, bad);
    launch_ntt_fwd_rows(c, ct->data(), limb_rows(c, npolys, nl), rows);
    return ct;
  }
  hipLaunchKernelGGL(words_to_residues_kernel, wire_grid(c, rows), dim3(kWireThreads), 0, c.stream, ct->data(), nl,
                     c.d_primes, (int)c.log_n, bad);
  COPSE_HIP(hipGetLastError());
  launch_ntt_fwd(c, ct->data(), limb_rows(c, npolys, nl), rows);
  return ct;
}

// ------------------------------------------------------------------ slots <-> plaintext polynomials
// evaluation slot k of plaintext p: slots[p][inv[k]] mod t (inv: position of evaluation slot k among the
// slots; gathered, so that the writes are contiguous)
__global__ void slots_to_eval_kernel(double* ev, const uint64_t* slots, const uint32_t* inv, uint64_t t, int logN) {
  const size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= (size_t)1 << logN) return;
  const size_t base = (size_t)blockIdx.y << logN;
  const uint64_t v = slots[base + inv[k]];
  ev[base + k] = (double)(v < t ? v : v % t);
}
__device__ __forceinline__ double center_t(double m, double t) { return m > (t - 1.0) * 0.5 ? m - t : m; }

// limb rows of a plaintext: its coefficients centered mod t, reduced modulo every prime
__global__ void lift_plain_kernel(double* out, const double* m, double t, const DevPrime* P, int logN) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (size_t)1 << logN) return;
  const DevPrime& pr = P[blockIdx.y];
  out[((size_t)blockIdx.y << logN) + i] = mod_reduce(center_t(m[i], t), pr.q, pr.qinv);
}

// row (p, r) of the transform modulo t
static const int2* t_rows(Context& c, int count) {
  const std::string key = "tmod:" + std::to_string(count);
  auto it = c.row_tables.find(key);
  if (it != c.row_tables.end()) return it->second;
  std::vector<int2> h;
  for (int p = 0; p < count; ++p) h.push_back(make_int2(p, c.n_primes()));
  return c.rows(key, h);
}

// Coefficients in [0, t) of `count` slot vectors ([count][N] in caller memory), enqueued: the caller of this keeps them
// until the stream has been waited for
static DBuf encode_device(Context& c, const uint64_t* slots, int count) {
  DBuf up(&c, (size_t)count * c.N), m(&c, (size_t)count * c.N);
  COPSE_HIP(hipMemcpyAsync(up.get(), slots, (size_t)count * c.N * 8, hipMemcpyHostToDevice, c.stream));
  hipLaunchKernelGGL(slots_to_eval_kernel, wire_grid(c, count), dim3(kWireThreads), 0, c.stream, m.get(),
                     reinterpret_cast<const uint64_t*>(up.get()), c.d_slot_of_eval, c.t, (int)c.log_n);
  COPSE_HIP(hipGetLastError());
  launch_ntt_inv(c, m.get(), t_rows(c, count), count);
  return m;
}

std::unique_ptr<Plain> make_plain_slots(Context& c, const uint64_t* slots, int level) {
  auto p = std::make_unique<Plain>();
  p->level = level;
  p->buf = DBuf(&c, (size_t)(level + 1) * c.N);
  StreamWait wait{c.stream};   // slots is the caller's memory
  DBuf m = encode_device(c, slots, 1);
  hipLaunchKernelGGL(lift_plain_kernel, wire_grid(c, level + 1), dim3(kWireThreads), 0, c.stream, p->buf.get(), m.get(),
                     (double)c.t, c.d_primes, (int)c.log_n);
  COPSE_HIP(hipGetLastError());
  launch_ntt_fwd(c, p->buf.get(), limb_rows(c, 1, level + 1), level + 1);
  wait.finish();
  return p;
}

// ------------------------------------------------------------------ encryption
// z = 3 p + k, limb r: the coefficient rows of u (k = 0), t e0 + m (1) and t e1 (2) of plaintext p.  noise: per
// plaintext `stride` bytes, u as bytes, then the two error streams of which every six bytes are one centered binomial
// value (bits 0..20 against bits 21..41).
__global__ void enc_lift_kernel(double* out, const uint8_t* noise, size_t stride, const double* m, double t,
                                const DevPrime* P, int logN) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x, N = (size_t)1 << logN;
  if (i >= N) return;
  const int z = blockIdx.z, k = z % 3;
  const DevPrime& pr = P[blockIdx.y];
  const uint8_t* u = noise + (size_t)(z / 3) * stride;
  double v;
  if (k == 0) {
    v = (double)(int8_t)u[i];
  } else {
    // N and the streams' length are even, so every value starts on an even address
    const uint16_t* e = reinterpret_cast<const uint16_t*>(u + N + (size_t)(k - 1) * ((stride - N) / 2)) + 3 * i;
    const uint64_t w = (uint64_t)e[0] | (uint64_t)e[1] << 16 | (uint64_t)e[2] << 32;
    v = (double)((int)__popc((uint32_t)w & 0x1fffffu) - (int)__popc((uint32_t)(w >> 21) & 0x1fffffu)) * t;   // exact
  }
  if (k == 1) v += center_t(m[((size_t)(z / 3) << logN) + i], t);
  out[(((size_t)z * gridDim.y + blockIdx.y) << logN) + i] = mod_reduce(v, pr.q, pr.qinv);
}
// (pk_b u + d0, pk_a u + d1) per plaintext and limb
__global__ void enc_combine_kernel(MPack out, const double* rows, const double* pk_b, const double* pk_a,
                                   const DevPrime* P, int logN) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (size_t)1 << logN) return;
  const int r = blockIdx.y, nl = gridDim.y, p = blockIdx.z;
  const DevPrime& pr = P[r];
  const size_t o = ((size_t)r << logN) + i, ps = (size_t)nl << logN;
  const double* d = rows + (size_t)p * 3 * ps + o;
  const double u = d[0];
  out.p[p][o] = canon(reduce_sym(mul_lazy(pk_b[o], u, pr.q, pr.qinv) + d[ps], pr.q, pr.qinv), pr.q);
  out.p[p][ps + o] = canon(reduce_sym(mul_lazy(pk_a[o], u, pr.q, pr.qinv) + d[2 * ps], pr.q, pr.qinv), pr.q);
}

// Fresh encryptions at `level` of n plaintexts given by their coefficients in [0, t): (pk0 u + t e0 + m, pk1 u + t e1)
// A full group of eight planes encrypted and exported takes 4.2 ms (40.5 ms with encoding, sampling and layout on one
// host core): 0.7 the host's SHAKE-256, 0.3 the device, the rest the 42 MB copied out to fresh pages.
static void encrypt_many(Context& c, const Keys& k, const DBuf& m, int n, int level, const uint8_t seed[32],
                         const uint64_t* objs, std::vector<CtPtr>& out) {
  const size_t N = c.N, stride = encryption_noise_bytes(N);
  const int nl = level + 1;
  DBuf rows(&c, (size_t)3 * n * nl * N), dn(&c, (n * stride + 7) / 8);
  std::vector<CtPtr> cts;
  MPack po;
  for (int p = 0; p < n; ++p) {
    cts.push_back(ct_alloc(c, level, 2));
    po.p[p] = cts.back()->data();
  }
  std::vector<uint8_t> noise(n * stride);
  sample_encryption_many(seed, objs, n, N, noise.data());
  StreamWait wait{c.stream};
  COPSE_HIP(hipMemcpyAsync(dn.get(), noise.data(), noise.size(), hipMemcpyHostToDevice, c.stream));
  hipLaunchKernelGGL(enc_lift_kernel, wire_grid(c, nl, 3 * n), dim3(kWireThreads), 0, c.stream, rows.get(),
                     reinterpret_cast<const uint8_t*>(dn.get()), stride, m.get(), (double)c.t, c.d_primes,
                     (int)c.log_n);
  COPSE_HIP(hipGetLastError());
  launch_ntt_fwd(c, rows.get(), limb_rows(c, 3 * n, nl), 3 * n * nl);
  hipLaunchKernelGGL(enc_combine_kernel, wire_grid(c, nl, n), dim3(kWireThreads), 0, c.stream, po, rows.get(),
                     k.pk_b.get(), k.pk_a.get(), c.d_primes, (int)c.log_n);
  COPSE_HIP(hipGetLastError());
  wait.finish();
  for (auto& ct : cts) out.push_back(std::move(ct));
}

// Plaintexts travel eight at a time: the limb rows in flight stay below 80 MB (N = 32768, twelve limbs), and eight
// streams of randomness fill the host's vectors.  Where the device does not have that much left, fewer, down to one,
// whose three rows a limb any encryption needs.
constexpr int kEncryptMany = 8;
template <class Encrypt>
static void encrypt_batches(int count, Encrypt encrypt) {
  int many = kEncryptMany;
  for (int first = 0; first < count;) {
    const int n = std::min(many, count - first);
    try {
      encrypt(first, n);
      first += n;
    } catch (const Error& e) {
      if (e.code != COPSE_ENOMEM || n == 1) throw;
      many = (n + 1) / 2;
    }
  }
}

std::vector<CtPtr> encrypt_slots_many(Context& c, const Keys& k, const uint64_t* slots, int count, int level,
                                      const uint8_t seed[32], const uint64_t* objs) {
  std::vector<CtPtr> out;
  StreamWait wait{c.stream};   // slots is the caller's memory
  encrypt_batches(count, [&](int first, int n) {
    encrypt_many(c, k, encode_device(c, slots + (size_t)first * c.N, n), n, level, seed, objs + first, out);
  });
  wait.finish();
  return out;
}

// Evaluation slot k of bit plane first + y: the query layout (compile.cpp) read backwards, from the slot to the
// feature it holds, so that the features (n_queries x F words) are all that is copied to the device.
__global__ void query_eval_kernel(double* ev, const uint32_t* feats, const uint32_t* slot_of_eval, uint32_t n_queries,
                                  uint32_t n_features, uint32_t B, uint32_t q, uint32_t K, uint32_t block_w,
                                  uint32_t first, int server_rep, int logN) {
  const uint32_t k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= 1u << logN) return;
  const uint32_t half = 1u << (logN - 1), slot = slot_of_eval[k], col = slot & (half - 1);
  const uint32_t per_row = half / block_w, in_row = col / block_w, s = col % block_w;
  const uint32_t query = (slot >> (logN - 1)) * per_row + in_row;
  double v = 0.0;
  if (in_row < per_row && query < n_queries && s < B) {
    const uint32_t f = server_rep ? s % n_features : s % q / K;
    v = (double)((feats[query * n_features + f] >> (first + blockIdx.y)) & 1u);
  }
  ev[((size_t)blockIdx.y << logN) + k] = v;
}

// One query group: every bit plane encrypted at the top level (objects as copse_query_encrypt)
std::vector<CtPtr> encrypt_query(Context& c, const Keys& k, const copse_public_meta& M, const uint32_t* features,
                                 size_t n_queries, const uint8_t seed[32], uint32_t group) {
  // what the kernel divides by and indexes with (a compiled layout has it so)
  if (M.block_w == 0 || M.block_w > c.N / 2 || M.n_features == 0 || M.K == 0 || M.q == 0 ||
      (uint64_t)M.q > (uint64_t)M.K * M.n_features || n_queries > c.N / 2 / M.block_w * 2 || M.precision > 32)
    fail(COPSE_EINVAL, "layout made for another ring size");
  std::vector<CtPtr> out;
  if (M.precision == 0) return out;
  const size_t words = n_queries * M.n_features;
  DBuf feats(&c, (words + 1) / 2);
  StreamWait wait{c.stream};   // features is the caller's memory
  COPSE_HIP(hipMemcpyAsync(feats.get(), features, words * sizeof(uint32_t), hipMemcpyHostToDevice, c.stream));
  const uint32_t B = M.m + M.b + M.q - 2 + (M.server_rep ? M.n_features - 1 : 0);
  encrypt_batches((int)M.precision, [&](int first, int n) {
    DBuf m(&c, n * c.N);
    hipLaunchKernelGGL(query_eval_kernel, wire_grid(c, n), dim3(kWireThreads), 0, c.stream, m.get(),
                       reinterpret_cast<const uint32_t*>(feats.get()), c.d_slot_of_eval, (uint32_t)n_queries,
                       M.n_features, B, M.q, M.K, M.block_w, (uint32_t)first, M.server_rep ? 1 : 0, (int)c.log_n);
    COPSE_HIP(hipGetLastError());
    launch_ntt_inv(c, m.get(), t_rows(c, n), n);
    uint64_t objs[kEncryptMany];
    for (int p = 0; p < n; ++p) objs[p] = (1ULL << 56) | ((uint64_t)group << 32) | (first + (uint32_t)p);
    encrypt_many(c, k, m, n, c.L, seed, objs, out);
  });
  wait.finish();
  return out;
}

// ------------------------------------------------------------------ decryption of labels
// c0 + c1 s of a level-0 ciphertext
__global__ void phase0_kernel(double* out, const double* c0, const double* c1, const double* s, const DevPrime* P,
                              int logN) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (size_t)1 << logN) return;
  const DevPrime& pr = P[0];
  out[i] = canon(reduce_sym(mul_lazy(c1[i], s[i], pr.q, pr.qinv) + c0[i], pr.q, pr.qinv), pr.q);
}
// the phase's coefficients centered mod q_0, reduced mod t; the largest magnitude into *worst
__global__ void phase_mod_t_kernel(double* io, double q0, double t, double tinv, int logN, unsigned long long* worst) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  unsigned long long mag = 0;
  if (i < (size_t)1 << logN) {
    const double v = io[i];
    const bool neg = v > (q0 - 1.0) * 0.5;
    const double a = neg ? q0 - v : v;
    mag = (unsigned long long)a;
    const double r = mod_reduce(a, t, tinv);
    io[i] = neg && r != 0.0 ? t - r : r;
  }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) {
    const unsigned long long o = __shfl_xor(mag, d);
    mag = o > mag ? o : mag;
  }
  if ((threadIdx.x & 63) == 0) atomicMax(worst, mag);
}
// slot j < m of query k (block k of block_w slots): 0, 1, or 2 for any other value
__global__ void label_bits_kernel(uint8_t* bits, const double* ev, const uint32_t* eval_of_slot, uint32_t m, uint32_t total,
                                  uint32_t block_w, uint32_t blocks_per_row, int logN) {
  const uint32_t g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= total) return;
  const uint32_t k = g / m, j = g % m;
  const uint32_t slot = ((k / blocks_per_row) << (logN - 1)) + (k % blocks_per_row) * block_w + j;
  const double v = ev[eval_of_slot[slot]];
  bits[g] = v == 0.0 ? 0 : v == 1.0 ? 1 : 2;
}

// The label slots of a level-0 result: bits[n_queries * m] as label_bits_kernel; returns the largest centered
// phase coefficient.  Only these bytes leave the device (1.1 ms to 0.2 ms for the 16-tree forest's 32 queries
// together with the result's import: the transform modulo t took the host 0.8 ms).
uint64_t decrypt_label_slots(Context& c, const Keys& k, const copse_public_meta& meta, const Ct& ct, size_t n_queries,
                             std::vector<uint8_t>& bits) {
  if (!k.has_secret) fail(COPSE_EKEY, "secret key absent");
  const size_t N = c.N, total = n_queries * meta.m;
  const int logN = (int)c.log_n;
  DBuf ph(&c, N), back(&c, 1 + (total + 7) / 8);
  auto* worst = reinterpret_cast<unsigned long long*>(back.get());
  COPSE_HIP(hipMemsetAsync(worst, 0, 8, c.stream));
  hipLaunchKernelGGL(phase0_kernel, wire_grid(c, 1), dim3(kWireThreads), 0, c.stream, ph.get(), ct.poly(0, N),
                     ct.poly(1, N), k.s.get(), c.d_primes, logN);
  COPSE_HIP(hipGetLastError());
  launch_ntt_inv(c, ph.get(), limb_rows(c, 1, 1), 1);
  hipLaunchKernelGGL(phase_mod_t_kernel, wire_grid(c, 1), dim3(kWireThreads), 0, c.stream, ph.get(),
                     (double)c.primes[0], (double)c.t, 1.0 / (double)c.t, logN, worst);
  COPSE_HIP(hipGetLastError());
  launch_ntt_fwd(c, ph.get(), t_rows(c, 1), 1);
  if (total > 0) {
    hipLaunchKernelGGL(label_bits_kernel, dim3((unsigned)((total + kWireThreads - 1) / kWireThreads)),
                       dim3(kWireThreads), 0, c.stream, reinterpret_cast<uint8_t*>(worst + 1), ph.get(),
                       c.d_eval_of_slot, meta.m, (uint32_t)total, meta.block_w, (uint32_t)(N / 2 / meta.block_w), logN);
    COPSE_HIP(hipGetLastError());
  }
  std::vector<uint8_t> h(8 + total);
  COPSE_HIP(hipMemcpyAsync(h.data(), back.get(), h.size(), hipMemcpyDeviceToHost, c.stream));
  COPSE_HIP(hipStreamSynchronize(c.stream));
  bits.assign(h.begin() + 8, h.end());
  uint64_t w;
  std::memcpy(&w, h.data(), 8);
  return w;
}

}  // namespace copse
