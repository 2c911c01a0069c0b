// C ABI, context, table generation and kernel orchestration.
// Compiled as HIP for gfx950 (the product) or, with -DHCNN_HOSTEMU, as plain C++
// for the CPU checker of the kernel sources.
#include "../../include/hcnn.h"

#include <algorithm>
#include <cmath>
#include <mutex>
#include <new>
#include <vector>

#include "fv_kernels.h"
#include "ntt_kernels.h"
#include "rate_kernels.h"

using namespace hcnn;

namespace {

typedef unsigned __int128 u128;

// ---------------------------------------------------------------- host number theory
uint32_t h_mulmod(uint32_t a, uint32_t b, uint32_t m) { return (uint32_t)(((uint64_t)a * b) % m); }
uint32_t h_powmod(uint32_t a, uint64_t e, uint32_t m) {
  uint64_t r = 1, b = a % m;
  while (e) {
    if (e & 1) r = r * b % m;
    b = b * b % m;
    e >>= 1;
  }
  return (uint32_t)r;
}
uint32_t h_inv(uint32_t a, uint32_t prime) { return h_powmod(a % prime, (uint64_t)prime - 2, prime); }

bool h_is_prime(uint32_t x) {
  if (x < 2) return false;
  for (uint32_t sp : {2u, 3u, 5u, 7u, 11u, 13u}) {
    if (x % sp == 0) return x == sp;
  }
  uint32_t d = x - 1;
  int r = 0;
  while ((d & 1) == 0) { d >>= 1; ++r; }
  for (uint32_t a : {2u, 3u, 5u, 7u}) {          // decides every x < 3,215,031,751
    uint64_t y = h_powmod(a, d, x);
    if (y == 1 || y == x - 1) continue;
    bool comp = true;
    for (int i = 1; i < r; ++i) {
      y = y * y % x;
      if (y == x - 1) { comp = false; break; }
    }
    if (comp) return false;
  }
  return true;
}

// 64-bit variants for the plaintext modulus (up to 47 bits)
uint64_t h_mulmod64(uint64_t a, uint64_t b, uint64_t m) { return (uint64_t)((unsigned __int128)a * b % m); }
uint64_t h_powmod64(uint64_t b, uint64_t e, uint64_t m) {
  uint64_t r = 1 % m;
  b %= m;
  while (e) {
    if (e & 1) r = h_mulmod64(r, b, m);
    b = h_mulmod64(b, b, m);
    e >>= 1;
  }
  return r;
}
bool h_is_prime64(uint64_t x) {
  if (x < 2) return false;
  for (uint64_t sp : {2ull, 3ull, 5ull, 7ull, 11ull, 13ull, 17ull, 19ull, 23ull, 29ull, 31ull, 37ull}) {
    if (x % sp == 0) return x == sp;
  }
  uint64_t d = x - 1;
  int r = 0;
  while ((d & 1) == 0) { d >>= 1; ++r; }
  for (uint64_t a : {2ull, 3ull, 5ull, 7ull, 11ull, 13ull, 17ull, 19ull, 23ull, 29ull, 31ull, 37ull}) {   // decides every x < 2^64
    uint64_t y = h_powmod64(a, d, x);
    if (y == 1 || y == x - 1) continue;
    bool comp = true;
    for (int i = 1; i < r; ++i) {
      y = h_mulmod64(y, y, x);
      if (y == x - 1) { comp = false; break; }
    }
    if (comp) return false;
  }
  return true;
}
// product of all `ms` except index `skip` (skip < 0: all), modulo a 64-bit m
uint64_t h_prod_mod64(const std::vector<uint32_t>& ms, int skip, uint64_t m) {
  uint64_t r = 1 % m;
  for (int i = 0; i < (int)ms.size(); ++i)
    if (i != skip) r = h_mulmod64(r, ms[i] % m, m);
  return r;
}

// psi = x^((p-1)/2n) for the smallest x >= 2 giving order exactly 2n
uint32_t h_root_of_unity(uint32_t n, uint32_t p) {
  const uint64_t e = ((uint64_t)p - 1) / (2ull * n);
  for (uint32_t x = 2;; ++x) {
    uint32_t psi = h_powmod(x, e, p);
    if (h_powmod(psi, n, p) == p - 1) return psi;
  }
}

uint32_t h_brev(uint32_t v, int bits) {
  uint32_t r = 0;
  for (int i = 0; i < bits; ++i) { r = (r << 1) | (v & 1); v >>= 1; }
  return r;
}

// -p^-1 mod 2^32 for odd p (Newton iteration, doubling the number of correct bits each step)
uint32_t h_neg_inv32(uint32_t p) {
  uint32_t inv = 1;
  for (int it = 0; it < 5; ++it) inv *= 2u - p * inv;
  return 0u - inv;
}

ShoupConst h_shoup(uint32_t w, uint32_t p) {
  ShoupConst c;
  c.w = w;
  c.ws = (uint32_t)(((uint64_t)w << 32) / p);
  return c;
}

Mod h_mod(uint32_t p) {
  Mod m;
  m.p = p;
  m.c32 = (uint32_t)((1ull << 32) % p);
  m.c32s = (uint32_t)(((uint64_t)m.c32 << 32) / p);
  m.mu = (uint32_t)((1ull << 61) / p);
  return m;
}

// product of all `ms` except index `skip` (skip < 0: all), modulo m
uint32_t h_prod_mod(const std::vector<uint32_t>& ms, int skip, uint32_t m) {
  uint64_t r = 1 % m;
  for (int i = 0; i < (int)ms.size(); ++i)
    if (i != skip) r = r * (ms[i] % m) % m;
  return (uint32_t)r;
}

// little-endian multiword natural numbers, only for the size check of the auxiliary basis
typedef std::vector<uint32_t> Big;
void big_mul_small(Big& a, uint32_t f) {
  uint64_t carry = 0;
  for (auto& w : a) {
    uint64_t t = (uint64_t)w * f + carry;
    w = (uint32_t)t;
    carry = t >> 32;
  }
  if (carry) a.push_back((uint32_t)carry);
}
void big_add_small(Big& a, uint32_t v) {
  uint64_t carry = v;
  for (auto& w : a) {
    uint64_t t = (uint64_t)w + carry;
    w = (uint32_t)t;
    carry = t >> 32;
    if (!carry) break;
  }
  if (carry) a.push_back((uint32_t)carry);
}
int big_cmp(Big a, Big b) {
  while (!a.empty() && a.back() == 0) a.pop_back();
  while (!b.empty() && b.back() == 0) b.pop_back();
  if (a.size() != b.size()) return a.size() < b.size() ? -1 : 1;
  for (size_t i = a.size(); i-- > 0;)
    if (a[i] != b[i]) return a[i] < b[i] ? -1 : 1;
  return 0;
}

bool valid_n(uint32_t n) { return n >= 1024 && n <= 32768 && (n & (n - 1)) == 0; }
bool valid_rns_prime(uint32_t p, uint32_t n) {
  return p > (1u << 29) && p < (1u << 30) && (p - 1) % (2 * n) == 0 && h_is_prime(p);
}

int check_primes(uint32_t n, const uint32_t* q, uint32_t k, const uint32_t* p, uint32_t kp) {
  std::vector<uint32_t> all(q, q + k);
  if (kp) all.insert(all.end(), p, p + kp);
  for (uint32_t v : all)
    if (!valid_rns_prime(v, n)) return HCNN_ERR_PRIME;
  std::sort(all.begin(), all.end());
  if (std::adjacent_find(all.begin(), all.end()) != all.end()) return HCNN_ERR_PRIME;
  return HCNN_OK;
}

// is prod(p[0..kp)) > t*n*prod(q) + 1 ?
bool aux_sufficient(uint32_t n, const uint32_t* q, uint32_t k, uint64_t t, const uint32_t* p, uint32_t kp) {
  Big lhs{1}, rhs{1};
  for (uint32_t j = 0; j < kp; ++j) big_mul_small(lhs, p[j]);
  for (uint32_t i = 0; i < k; ++i) big_mul_small(rhs, q[i]);
  // t < 2^47 = (t >> 24) * 2^24 + (t & 0xffffff): two small factors and a sum
  {
    Big hi = rhs;
    big_mul_small(hi, (uint32_t)(t >> 24));
    big_mul_small(hi, 1u << 24);
    big_mul_small(rhs, (uint32_t)(t & 0xffffffu));
    if (rhs.size() < hi.size()) rhs.resize(hi.size(), 0);
    uint64_t carry = 0;
    for (size_t w = 0; w < rhs.size(); ++w) {
      const uint64_t sum = (uint64_t)rhs[w] + (w < hi.size() ? hi[w] : 0) + carry;
      rhs[w] = (uint32_t)sum;
      carry = sum >> 32;
    }
    if (carry) rhs.push_back((uint32_t)carry);
  }
  big_mul_small(rhs, n);
  big_add_small(rhs, 1);
  return big_cmp(lhs, rhs) > 0;
}

bool aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

}  // namespace

// ---------------------------------------------------------------- scratch of the entry point that allocates nothing
// hcnn_ct_square_relin_noalloc keeps the intermediate polynomials of its internal batch in this array instead of a
// buffer from hipMalloc.  Every device that loads the library holds its own copy (at its own address) until the
// process ends; every call on a device shares that copy.
constexpr size_t kStaticScratchBytes = (size_t)128 << 20;
#ifdef HCNN_HOSTEMU
alignas(256) static uint32_t scratch[kStaticScratchBytes / 4];
#else
static __device__ __align__(256) uint32_t scratch[kStaticScratchBytes / 4];
#endif

namespace {
#ifndef HCNN_HOSTEMU
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
uint32_t* g_scratch_addr[kMaxDevices] = {};
#endif

// Device address of `scratch` on the current device, looked up once per device.  (In host code the array's name is
// only a handle for the lookup: kernels and copies take the address returned here.)
int static_scratch_of_current_device(uint32_t** out) {
#ifdef HCNN_HOSTEMU
  *out = scratch;
  return 0;
#else
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return (int)e;
  if (dev < 0 || dev >= kMaxDevices) return HCNN_ERR_NODEVICE;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_addr[dev]) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return (int)e;
    if (!ptr) return HCNN_ERR_NODEVICE;
    g_scratch_addr[dev] = (uint32_t*)ptr;
  }
  *out = g_scratch_addr[dev];
  return 0;
#endif
}
}  // namespace

// ---------------------------------------------------------------- context
struct BConvHost {
  uint32_t ks = 0, kd = 0;
  std::vector<Mod> src_mod;
  std::vector<ShoupConst> zmul, xmul;
  std::vector<uint32_t> ginv, half;
  std::vector<BConvDst> dst;
  std::vector<BConvSrc> src;
  std::vector<int32_t> B, BT;
};

struct hcnn_ctx {
  uint32_t n = 0, logn = 0, k = 0, kp = 0;
  uint64_t t = 0;
  std::vector<uint32_t> q, p;
  hcnn_stream_t stream = nullptr;
  std::vector<void*> owned;

  Mod* d_mods = nullptr;            // [k + kp]
  NttLimb* d_limbs = nullptr;       // [k + kp]
  TwTable d_tw_fwd{}, d_tw_inv{};   // [k + kp][n/2]
  EncScale* d_delta = nullptr;      // [k]
  int32_t* d_tq_inv = nullptr;      // [kp] t * q^-1 mod p_j
  SplitRoot* d_scale_root = nullptr;   // [2][k + kp], n = 8192 and 32768: last inverse stage and the scaling's first factor in one
  BConvDev ext{}, to_p{}, to_q{}, dec{};
  uint32_t* d_gauss_t = nullptr;    // thresholds of the Gaussian sampler (uploaded on first use)
  uint32_t* d_dec_tab = nullptr;    // [k][3] constants of the decrypt rounding
  unsigned long long* d_counters = nullptr;   // [2]

  uint32_t* d_evk_hat = nullptr;
  uint32_t* d_evk_shared = nullptr;  // behind d_evk_hat in its allocation, or in one of its own: [4][n/64][k][outputs][64], where the shared-basis relinearisation is in use
  RelinPair* d_pair = nullptr;       // [outputs / 2]
  RelinCrt* d_crt = nullptr;         // [k]
  RelinCrtInv crt_inv{};
  bool has_key = false;

  uint32_t* work = nullptr;       // device work buffers of the entry points that may allocate (work_buffer)
  size_t work_bytes = 0;
  uint32_t* small_work = nullptr;
  size_t small_work_bytes = 0;
  uint32_t* static_scratch = nullptr;   // this device's copy of the file-scope array `scratch` (kStaticScratchBytes)

  uint32_t band = 128;
  uint64_t square_chunk = 0;
  uint64_t relin_order = 0;   // 0 = by key size, 1 = ciphertext-major, 2 = key-major
  uint64_t fusion = 0;   // one-kernel tensor / relinearisation: 0 = chosen per batch, 1 = never, 2 = always where available
  size_t max_lds = 0;
  uint32_t compute_units = 256;
  uint32_t relin_fused_wgs = 1, tensor_fused_wgs = 1;   // resident workgroups per compute unit of the one-kernel forms

  // optional per-kernel timing (HCNN_OPT_PROFILE): an event pair around every launch
  struct Pending { int cls; uint64_t blocks; hcnn_event_t start, stop; };
  bool profile = false;
  std::vector<Pending> pending;
  std::vector<hcnn_event_t> free_events;
  uint64_t prof_launches[HCNN_PROF_COUNT] = {};
  uint64_t prof_blocks[HCNN_PROF_COUNT] = {};
  double prof_ms[HCNN_PROF_COUNT] = {};
};

namespace {

template <class T>
int upload(hcnn_ctx* c, const std::vector<T>& h, T** d) {
  void* ptr = nullptr;
  int e = dev_malloc(&ptr, h.size() * sizeof(T));
  if (e) return e;
  c->owned.push_back(ptr);
  if (!h.empty()) {
    e = copy_h2d(ptr, h.data(), h.size() * sizeof(T), c->stream);
    if (e) return e;
  }
  *d = (T*)ptr;
  return 0;
}

template <class K> struct KernelClass { static constexpr int id = HCNN_PROF_OTHER; };
template <int A, int B, int C, int D> struct KernelClass<NttFwd<A, B, C, D>> { static constexpr int id = HCNN_PROF_NTT_FWD; };
template <int A, int B, int C, int D> struct KernelClass<NttInv<A, B, C, D>> { static constexpr int id = HCNN_PROF_NTT_INV; };
template <int A> struct KernelClass<ExtKernel<A>> { static constexpr int id = HCNN_PROF_BASE_EXT; };
template <int A, bool H> struct KernelClass<ScaleKernel<A, H>> { static constexpr int id = HCNN_PROF_SCALE; };
template <int O> struct KernelClass<RelinSharedMac<O>> { static constexpr int id = HCNN_PROF_RELIN_MAC; };
template <int A, int B> struct KernelClass<RelinBack<A, B>> { static constexpr int id = HCNN_PROF_NTT_INV; };
template <int A> struct KernelClass<RelinMacKernel<A>> { static constexpr int id = HCNN_PROF_RELIN_MAC; };
template <int A, int B, int C> struct KernelClass<RelinFused<A, B, C>> { static constexpr int id = HCNN_PROF_RELIN_FUSED; };
template <int A, int B, int C> struct KernelClass<TensorFused<A, B, C>> { static constexpr int id = HCNN_PROF_TENSOR; };
template <int F, bool S> struct KernelClass<MacKernel<F, S>> { static constexpr int id = HCNN_PROF_SCALAR_MAC; };
template <int B> struct KernelClass<MacMfma<B>> { static constexpr int id = HCNN_PROF_SCALAR_MAC; };
template <> struct KernelClass<MacPair> { static constexpr int id = HCNN_PROF_SCALAR_MAC; };
template <> struct KernelClass<MacPack> { static constexpr int id = HCNN_PROF_SCALAR_MAC; };
template <int F> struct KernelClass<MacKernelDirect<F>> { static constexpr int id = HCNN_PROF_SCALAR_MAC; };

int take_event(hcnn_ctx* c, hcnn_event_t* ev) {
  if (!c->free_events.empty()) {
    *ev = c->free_events.back();
    c->free_events.pop_back();
    return 0;
  }
  return event_create(ev);
}

// Launch on the context's stream; with profiling on, bracket the launch with two events.
// `units` (default: the grid) is what the profile counts: the rows of an NTT launch whose grid is padded.
template <class K, class Args>
int run(hcnn_ctx* c, size_t grid, size_t lds_bytes, const Args& a, size_t units = 0) {
  const hcnn_stream_t stream = c->stream;
  if (!c->profile || grid == 0) return launch<K>(stream, grid, lds_bytes, a);
  hcnn_ctx::Pending pd;
  pd.cls = KernelClass<K>::id;
  pd.blocks = units ? units : grid;
  int e;
  if ((e = take_event(c, &pd.start))) return e;
  if ((e = take_event(c, &pd.stop))) return e;
  if ((e = event_record(pd.start, stream))) return e;
  if ((e = launch<K>(stream, grid, lds_bytes, a))) return e;
  if ((e = event_record(pd.stop, stream))) return e;
  c->pending.push_back(pd);
  return 0;
}

int fold_profile(hcnn_ctx* c) {
  if (c->pending.empty()) return 0;
  int e = stream_sync(c->stream);
  if (e) return e;
  for (auto& pd : c->pending) {
    float ms = 0.f;
    if ((e = event_elapsed_ms(&ms, pd.start, pd.stop))) return e;
    c->prof_launches[pd.cls] += 1;
    c->prof_blocks[pd.cls] += pd.blocks;
    c->prof_ms[pd.cls] += ms;
    c->free_events.push_back(pd.start);
    c->free_events.push_back(pd.stop);
  }
  c->pending.clear();
  return 0;
}

// Tables of an exact centred base conversion src -> dst.
//   zfac[i]   extra factor folded into z_i (1 or t), also used as xmul
//   fold_inv  when true the tables give -(x * M^-1): B = -m_i^-1, V = 1
//             otherwise they give x:                 B = M/m_i,   V = -M   (all mod m'_j, centred, times 2^32)
int32_t h_centred(uint32_t x, uint32_t p) { return x > p / 2 ? (int32_t)x - (int32_t)p : (int32_t)x; }
int32_t h_mont(uint32_t x, uint32_t p) { return h_centred(h_mulmod(x, (uint32_t)((1ull << 32) % p), p), p); }

BConvHost make_bconv(const std::vector<uint32_t>& src, const std::vector<uint32_t>& dst, uint64_t zfac, bool fold_inv) {
  BConvHost h;
  h.ks = (uint32_t)src.size();
  h.kd = (uint32_t)dst.size();
  for (uint32_t i = 0; i < h.ks; ++i) {
    const uint32_t m = src[i];
    h.src_mod.push_back(h_mod(m));
    const uint32_t Mi_inv = h_inv(h_prod_mod(src, (int)i, m), m);        // (M/m_i)^-1 mod m_i
    const uint32_t zm = h_mulmod(Mi_inv, (uint32_t)(zfac % m), m);
    h.zmul.push_back(h_shoup(zm, m));
    h.xmul.push_back(h_shoup((uint32_t)(zfac % m), m));
    h.src.push_back(BConvSrc{m, h_neg_inv32(m), h_mont(1, m), h_mont(zm, m)});
  }
  h.ginv.assign((size_t)h.ks * h.ks, 0);
  for (uint32_t i = 0; i < h.ks; ++i)
    for (uint32_t l = 0; l < i; ++l) h.ginv[(size_t)i * h.ks + l] = h_inv(src[l] % src[i], src[i]);
  // mixed-radix digits of (M-1)/2, whose residue mod m_i is (m_i-1)/2
  h.half.assign(h.ks, 0);
  for (uint32_t i = 0; i < h.ks; ++i) {
    uint32_t tt = (src[i] - 1) / 2;
    for (uint32_t l = 0; l < i; ++l) {
      uint32_t al = h.half[l] % src[i];
      tt = (tt + src[i] - al) % src[i];
      tt = h_mulmod(tt, h.ginv[(size_t)i * h.ks + l], src[i]);
    }
    h.half[i] = tt;
  }
  h.B.assign((size_t)h.ks * h.kd, 0);
  h.BT.assign((size_t)h.ks * h.kd, 0);
  for (uint32_t j = 0; j < h.kd; ++j) {
    const uint32_t mj = dst[j];
    for (uint32_t i = 0; i < h.ks; ++i) {
      const uint32_t b = fold_inv ? mj - h_inv(src[i] % mj, mj) : h_prod_mod(src, (int)i, mj);
      h.B[(size_t)i * h.kd + j] = h.BT[(size_t)j * h.ks + i] = h_mont(b, mj);
    }
    h.dst.push_back(BConvDst{mj, h_neg_inv32(mj), h_mont(1, mj), fold_inv ? h_mont(1, mj) : -h_mont(h_prod_mod(src, -1, mj), mj)});
  }
  return h;
}

int upload_bconv(hcnn_ctx* c, const BConvHost& h, BConvDev* d) {
  int e;
  Mod* sm; ShoupConst* zm; ShoupConst* xm; uint32_t* gi; uint32_t* hf; BConvDst* dd; BConvSrc* ss; int32_t* B; int32_t* BT;
  if ((e = upload(c, h.src_mod, &sm))) return e;
  if ((e = upload(c, h.zmul, &zm))) return e;
  if ((e = upload(c, h.xmul, &xm))) return e;
  if ((e = upload(c, h.ginv, &gi))) return e;
  if ((e = upload(c, h.half, &hf))) return e;
  if ((e = upload(c, h.dst, &dd))) return e;
  if ((e = upload(c, h.src, &ss))) return e;
  if ((e = upload(c, h.B, &B))) return e;
  if ((e = upload(c, h.BT, &BT))) return e;
  d->ks = h.ks; d->kd = h.kd;
  d->src_mod = sm; d->zmul = zm; d->xmul = xm; d->ginv = gi; d->half = hf;
  d->dst = dd; d->src = ss; d->B = B; d->BT = BT;
  return 0;
}

int build_tables(hcnn_ctx* c) {
  const uint32_t n = c->n, L = c->k + c->kp;
  std::vector<uint32_t> all = c->q;
  all.insert(all.end(), c->p.begin(), c->p.end());

  std::vector<Mod> mods;
  std::vector<NttLimb> limbs;
  // radix-4 butterflies sit at the stages s, s + 1 with s = log2(n) mod 2; their constants carry 2^32 and are centred
  const uint32_t odd = c->logn & 1u;
  std::vector<R4Twiddle> quad[2];
  std::vector<int32_t> nuw[2];
  for (int d = 0; d < 2; ++d) {
    quad[d].assign((size_t)L * (n / 2), R4Twiddle{0, 0, 0, 0});
    nuw[d].assign((size_t)L * (n / 2), 0);
  }
  // every constant is +-psi^e * 2^32 (a product of twiddles adds exponents, a sign is psi^n): one table of powers per prime
  std::vector<int32_t> pw(2 * (size_t)n);
  for (uint32_t l = 0; l < L; ++l) {
    const uint32_t p = all[l];
    const uint32_t psi = h_root_of_unity(n, p), r32 = (uint32_t)((1ull << 32) % p);
    const uint32_t psi_s = h_shoup(psi, p).ws;
    auto centred = [&](uint32_t x) { return x > p / 2 ? (int32_t)x - (int32_t)p : (int32_t)x; };
    auto mont = [&](uint32_t x) { return centred(h_mulmod(x, r32, p)); };
    uint32_t v = r32;
    for (uint32_t e = 0; e < n; ++e) {
      pw[e] = centred(v);
      pw[e + n] = -pw[e];
      const uint32_t y = v * psi - (uint32_t)(((uint64_t)v * psi_s) >> 32) * p;
      v = y >= p ? y - p : y;
    }
    // exponent of a node's twiddle: brev(node) forward, its negative backward
    auto ex = [&](int dir, uint32_t node) {
      const uint32_t x = h_brev(node, (int)c->logn);
      return dir ? 2 * n - x : x;
    };
    for (int d = 0; d < 2; ++d) {
      R4Twiddle* q4 = quad[d].data() + (size_t)l * (n / 2);
      int32_t* q1 = nuw[d].data() + (size_t)l * (n / 2);
      for (uint32_t s = odd; s + 2 <= c->logn; s += 2)
        for (uint32_t node = 1u << s; node < 2u << s; ++node) {
          const uint32_t w = ex(d, node), ev = ex(d, 2 * node), u = ex(d, 2 * node + 1), m = 2 * n - 1;
          q4[node] = R4Twiddle{pw[w & m], pw[ev & m], pw[(ev + w) & m], pw[u & m]};
          q1[node] = pw[(u + w + n) & m];
        }
    }
    NttLimb nl{};
    nl.m = h_mod(p);
    nl.rc = centred(r32);
    nl.pinv = h_neg_inv32(p);
    nl.zero = 0;
    nl.w1 = pw[ex(0, 1)];
    nl.key_scale = mont(r32);
    for (int j = 0; j < 3; ++j) nl.byte_c[j] = mont(1u << (8 * (j + 1)));
    auto inv_root = [&](uint32_t scale) {
      auto sc = [&](uint32_t e) {           // psi^e * scale * 2^32
        const int32_t x = pw[e & (2 * n - 1)];
        return centred(h_mulmod(x < 0 ? (uint32_t)(x + (int32_t)p) : (uint32_t)x, scale, p));
      };
      const uint32_t w = ex(1, 1), v2 = ex(1, 2), u2 = ex(1, 3);
      return InvRoot{mont(scale), sc(w), sc(v2), sc(u2), sc(v2 + w), sc(u2 + w + n)};
    };
    const uint32_t ninv = h_inv(n % p, p);
    nl.inv = inv_root(ninv);
    nl.inv_r = inv_root(h_mulmod(ninv, r32, p));
    if (l >= c->k && l < c->k + kSharedPrimes && c->kp >= kSharedPrimes) {
      const std::vector<uint32_t> four(c->p.begin(), c->p.begin() + kSharedPrimes);
      nl.inv_z = inv_root(h_mulmod(ninv, h_inv(h_prod_mod(four, (int)(l - c->k), p), p), p));
    }
    mods.push_back(nl.m);
    limbs.push_back(nl);
  }
  int e;
  if ((e = upload(c, mods, &c->d_mods))) return e;
  if ((e = upload(c, limbs, &c->d_limbs))) return e;
  R4Twiddle* dq;
  int32_t* dn;
  for (int d = 0; d < 2; ++d) {
    if ((e = upload(c, quad[d], &dq))) return e;
    if ((e = upload(c, nuw[d], &dn))) return e;
    (d ? c->d_tw_inv : c->d_tw_fwd) = TwTable{dq, dn};
  }

  // floor(q/t) mod q_l = -(q mod t) * t^-1 mod q_l   (q = 0 mod q_l)
  const uint64_t q_mod_t = h_prod_mod64(c->q, -1, c->t);
  std::vector<EncScale> delta;
  for (uint32_t l = 0; l < c->k; ++l) {
    const uint32_t ql = c->q[l];
    const uint32_t v = h_mulmod((ql - (uint32_t)(q_mod_t % ql)) % ql, h_inv((uint32_t)(c->t % ql), ql), ql);
    const uint32_t r32 = (uint32_t)((1ull << 32) % ql), v2 = h_mulmod(v, r32, ql);
    const int32_t c32 = h_mont(h_mulmod(v, 1u << 31, ql), ql), c64 = h_mont(h_mulmod((v + v2) % ql, 1u << 31, ql), ql);
    delta.push_back(EncScale{h_mont(v, ql), h_mont(v2, ql), c32, c64});
  }
  if ((e = upload(c, delta, &c->d_delta))) return e;

  // decryption: r = [t*x]_q converted to the modulus t; the table carries the factor -q^-1 (DecRoundKernel)
  {
    BConvHost h = make_bconv(c->q, std::vector<uint32_t>{}, c->t, false);
    if ((e = upload_bconv(c, h, &c->dec))) return e;
    const uint64_t qinv_t = h_powmod64(q_mod_t, c->t - 2, c->t);
    std::vector<uint32_t> tab;
    for (uint32_t i = 0; i < c->k; ++i) {
      const uint64_t b = (c->t - h_mulmod64(h_prod_mod64(c->q, (int)i, c->t), qinv_t, c->t)) % c->t;
      for (int piece = 0; piece < 3; ++piece) tab.push_back((uint32_t)(b >> (16 * piece)) & 0xffffu);
    }
    if ((e = upload(c, tab, &c->d_dec_tab))) return e;
  }
  if (c->kp >= kSharedPrimes) {
    const std::vector<uint32_t> four(c->p.begin(), c->p.begin() + kSharedPrimes);
    std::vector<RelinCrt> crt;
    std::vector<RelinPair> pairs;
    for (uint32_t j = 0; j < c->k; ++j) {
      const uint32_t qj = c->q[j];
      RelinCrt kc;
      for (uint32_t r = 0; r < kSharedPrimes; ++r) kc.c[r] = h_mont(h_prod_mod(four, (int)r, qj), qj);
      kc.cv = -h_mont(h_prod_mod(four, -1, qj), qj);
      crt.push_back(kc);
      if (j % 2 == 0) {
        const bool alone = j + 1 == c->k;
        RelinPair pr;
        pr.inv = alone ? 0 : h_mont(h_inv(qj, c->q[j + 1]), c->q[j + 1]);
        for (uint32_t r = 0; r < kSharedPrimes; ++r) pr.q[r] = h_mont(qj % four[r], four[r]);
        pairs.push_back(pr);
      }
    }
    for (uint32_t r = 0; r < kSharedPrimes; ++r) c->crt_inv.f[r] = 1.0f / (float)four[r];
    if ((e = upload(c, crt, &c->d_crt))) return e;
    if ((e = upload(c, pairs, &c->d_pair))) return e;
  }
  if (c->kp) {
    BConvHost h_ext = make_bconv(c->q, c->p, 1, false);
    BConvHost h_to_p = make_bconv(c->q, c->p, c->t, true);
    BConvHost h_to_q = make_bconv(c->p, c->q, 1, false);
    if ((e = upload_bconv(c, h_ext, &c->ext))) return e;
    if ((e = upload_bconv(c, h_to_p, &c->to_p))) return e;
    if ((e = upload_bconv(c, h_to_q, &c->to_q))) return e;
    std::vector<int32_t> tq;
    for (uint32_t pj : c->p) tq.push_back(h_mont(h_mulmod((uint32_t)(c->t % pj), h_inv(h_prod_mod(c->q, -1, pj), pj), pj), pj));
    if ((e = upload(c, tq, &c->d_tq_inv))) return e;
    if (c->logn == 13 || c->logn == 15) {
      std::vector<SplitRoot> root;
      for (uint32_t half = 0; half < 2; ++half)
        for (uint32_t l = 0; l < L; ++l) {
          const uint32_t m = all[l];
          const uint32_t f = l < c->k ? h_to_p.zmul[l].w
                                      : h_mulmod((uint32_t)(c->t % m), h_inv(h_prod_mod(c->q, -1, m), m), m);
          const int32_t top = half ? limbs[l].inv_r.w : limbs[l].inv_r.c0;
          const int32_t x = h_centred(h_mulmod(top < 0 ? (uint32_t)(top + (int32_t)m) : (uint32_t)top, f, m), m);
          root.push_back(split_root_factors(x, x, half));
        }
      if ((e = upload(c, root, &c->d_scale_root))) return e;
    }
  }
  std::vector<unsigned long long> zeros(2, 0);
  if ((e = upload(c, zeros, &c->d_counters))) return e;
  return 0;
}

// Work buffer of a call that needs `bytes`: the small one, allocated on first use and kept as it is, or, for more, the
// large one, which grows on demand (it waits for the stream, frees and allocates) and is kept.  Which of the two a call
// takes depends on its size alone.
// The small one holds what key generation takes (2 + k polynomials), and 34 polynomials where that is at most 16 MiB (9 MiB at
// n = 8192, k = 8): every encryption, the decryption of up to 33 ciphertexts (a network's results) and the squaring of one or
// two.  None of them finds a buffer to grow that another one left (first decryption of 25 ciphertexts after key generation
// and encryption, n = 8192, k = 8, us: 335 with one buffer for all, 42 now).  A single growing buffer with a first size of
// 17 MiB made the first squaring slower instead (16 ciphertexts after key generation 186 -> 420 us, now 156: freeing takes
// up to 250 us, allocating 25 to 75).
constexpr size_t kSmallWorkPolys = 34, kSmallWorkBytes = (size_t)16 << 20;
int work_buffer(hcnn_ctx* c, size_t bytes, uint32_t** out) {
  const size_t poly = (size_t)c->k * c->n * 4;
  const size_t small = std::max((2 + c->k) * poly, std::min(kSmallWorkPolys * poly, kSmallWorkBytes));
  const bool large = bytes > small;
  uint32_t*& buf = large ? c->work : c->small_work;
  size_t& held = large ? c->work_bytes : c->small_work_bytes;
  if (bytes > held) {
    if (buf) {
      int e = stream_sync(c->stream);
      if (e) return e;
      dev_free(buf);
      buf = nullptr;
      held = 0;
    }
    const size_t want = large ? bytes : small;
    void* ptr = nullptr;
    int e = dev_malloc(&ptr, want);
    if (e) return e;
    buf = (uint32_t*)ptr;
    held = want;
  }
  *out = buf;
  return 0;
}

// Checker builds may send every ring and basis through the shared-basis relinearisation (the product takes it for n = 16384
// with 16 primes and n = 32768 with 12, and holds no kernels of it for others).
#ifdef HCNN_SHARED_ALL
constexpr bool kSharedAll = true;
#else
constexpr bool kSharedAll = false;
#endif

// ---------------------------------------------------------------- NTT dispatch
struct NttRows {
  const uint32_t* in;
  uint32_t* out;
  size_t rows;
  uint32_t cycle, limb_base;
  uint32_t in_group_rows, in_row0, out_group_rows, out_row0;
  const uint32_t* aux = nullptr;
  uint32_t own_limbs = 0;
  const int32_t* small = nullptr;
  uint32_t digits = 0, tile_words = 0;      // 0 digits: k
  const RelinPair* pair = nullptr;
};

// Do the squaring's forward transforms of `rows` rows (out of place) run as two workgroups per row?  n = 32768 always; n = 8192 while both
// halves of every row find a compute unit of their own: half as many waves share one then (us: one squaring of 8 primes 38.0 / 34.5, of 4
// 33.1 / 29.2, of 12 52.6 / 49.8, two of 8 42.4 / 38.6; n = 2048 gains nothing, four of 4 primes 26.9 / 28.3).
bool splits_rows(const hcnn_ctx* c, size_t rows) {
  return c->logn == 15 || (c->logn == 13 && (kSharedAll || 2 * rows <= c->compute_units));
}
// And the inverse transforms of the tensor's rows?  n = 32768 not while whole rows, but not all halves, find a compute unit of their own (two squarings
// of 16 primes 154 / 158 us).
bool splits_tensor_rows(const hcnn_ctx* c, size_t rows) {
  return splits_rows(c, rows) && (c->logn != 15 || 2 * rows <= c->compute_units || rows > c->compute_units);
}

template <int LOGN, int LOGR>
int ntt_launch(hcnn_ctx* c, const NttRows& r, bool inverse, int io) {
  NttArgs a{};
  a.in = r.in; a.out = r.out; a.aux = r.aux; a.small = r.small;
  a.tw = inverse ? c->d_tw_inv : c->d_tw_fwd;
  a.limbs = c->d_limbs;
  a.cycle = fast_div(r.cycle); a.limb_base = r.limb_base;
  a.in_group_rows = r.in_group_rows; a.in_row0 = r.in_row0;
  a.out_group_rows = r.out_group_rows; a.out_row0 = r.out_row0;
  a.n_rows = (uint32_t)r.rows;
  a.own_limbs = r.own_limbs;
  a.digits = fast_div(r.digits ? r.digits : c->k);
  a.tile_words = r.tile_words;
  a.pair = r.pair; a.k = c->k;
  const size_t lds = NttGeom<LOGN, LOGR>::kLdsBytes;
  if (inverse) {
    // Two workgroups per row where the reader takes the last stage: n = 32768 (4800 tensor rows 427 us with one, 348 with two; 3072
    // rows of the shared basis 250, 195), and launches that leave compute units idle otherwise
    constexpr int kCanSplit = LOGN == 13 || LOGN == 15;
    constexpr size_t lds_s = NttGeom<LOGN - kCanSplit, LOGR>::kLdsBytes;
    if (kCanSplit && (io == kNttLoadTensor || io == kNttLoadTensorMul) && splits_tensor_rows(c, r.rows)) {
      using Square = NttInv<LOGN, LOGR, kNttLoadTensor, kCanSplit>;
      using Product = NttInv<LOGN, LOGR, kNttLoadTensorMul, kCanSplit>;
      if (io == kNttLoadTensor) return run<Square>(c, Square::grid(r.rows), lds_s, a, r.rows);
      return run<Product>(c, Product::grid(r.rows), lds_s, a, r.rows);
    }
    using SquareRow = NttInv<LOGN, LOGR, kNttLoadTensor>;
    using ProductRow = NttInv<LOGN, LOGR, kNttLoadTensorMul>;
    if (io == kNttLoadTensor) return run<SquareRow>(c, SquareRow::grid(r.rows), lds, a, r.rows);
    if (io == kNttLoadTensorMul) return run<ProductRow>(c, ProductRow::grid(r.rows), lds, a, r.rows);
    if (io == kNttStoreAdd) return run<NttInv<LOGN, LOGR, kNttStoreAdd>>(c, r.rows, lds, a);
    if constexpr (LOGN == 15) {
      using Back = NttInv<LOGN, LOGR, kNttBackRow, 1>;
      if (io == kNttBackRow) return run<Back>(c, Back::grid(r.rows), lds_s, a, r.rows);
    }
    return run<NttInv<LOGN, LOGR>>(c, r.rows, lds, a);
  }
  // The largest ring runs its forward transforms as two workgroups per row (first stage folded into the load):
  // a whole row of it takes the LDS of a compute unit, half a row leaves room for two workgroups.  Each of the two
  // reads the whole row, so the form needs an output that is not its input.
  if constexpr (LOGN == 15) {
    if (r.in != r.out) {
      const size_t lds_h = NttGeom<LOGN - 1, LOGR>::kLdsBytes;
      if (io == kNttLoadDigit) {
        using K = NttFwd<LOGN, LOGR, kNttLoadDigit, 1>;
        return run<K>(c, K::grid(ntt_grouped_grid(r.rows, r.cycle)), lds_h, a, r.rows);
      }
      if (io == kNttDigitTile) {
        using K = NttFwd<LOGN, LOGR, kNttDigitTile, 1>;
        return run<K>(c, K::grid(ntt_grouped_grid(r.rows, r.cycle)), lds_h, a, r.rows);
      }
      if (io == kNttKeyTile) {
        using K = NttFwd<LOGN, LOGR, kNttKeyTile, 1>;
        return run<K>(c, K::grid(r.rows), lds_h, a, r.rows);
      }
      if (io == kNttStoreLazy) {
        using K = NttFwd<LOGN, LOGR, kNttStoreLazy, 1>;
        return run<K>(c, K::grid(r.rows), lds_h, a, r.rows);
      }
      if (io == kNttSmallKey) {
        using K = NttFwd<LOGN, LOGR, kNttSmallKey, 1>;
        return run<K>(c, K::grid(r.rows), lds_h, a, r.rows);
      }
      if (io == kNttStoreKey) {
        using K = NttFwd<LOGN, LOGR, kNttStoreKey, 1>;
        return run<K>(c, K::grid(r.rows), lds_h, a, r.rows);
      }
      using K = NttFwd<LOGN, LOGR, kNttPlain, 1>;
      return run<K>(c, K::grid(r.rows), lds_h, a, r.rows);
    }
    return io == kNttPlain ? run<NttFwd<LOGN, LOGR>>(c, r.rows, lds, a) : HCNN_ERR_ARG;
  } else {
    if constexpr (LOGN == 13) {
      if (r.in != r.out && splits_rows(c, r.rows)) {
        const size_t lds_h = NttGeom<LOGN - 1, LOGR>::kLdsBytes;
        if (io == kNttLoadDigit) {
          using K = NttFwd<LOGN, LOGR, kNttLoadDigit, 1>;
          return run<K>(c, K::grid(ntt_grouped_grid(r.rows, r.cycle)), lds_h, a, r.rows);
        }
        if (io == kNttStoreLazy) {
          using K = NttFwd<LOGN, LOGR, kNttStoreLazy, 1>;
          return run<K>(c, K::grid(r.rows), lds_h, a, r.rows);
        }
      }
    }
    if constexpr (LOGN == 14 || kSharedAll) {
      if (io == kNttDigitTile)
        return run<NttFwd<LOGN, LOGR, kNttDigitTile>>(c, ntt_grouped_grid(r.rows, r.cycle), lds, a, r.rows);
      if (io == kNttKeyTile) return run<NttFwd<LOGN, LOGR, kNttKeyTile>>(c, r.rows, lds, a);
    }
    if (io == kNttLoadDigit)
      return run<NttFwd<LOGN, LOGR, kNttLoadDigit>>(c, ntt_grouped_grid(r.rows, r.cycle), lds, a, r.rows);
    if (io == kNttStoreLazy) return run<NttFwd<LOGN, LOGR, kNttStoreLazy>>(c, r.rows, lds, a);
    if (io == kNttSmallKey) return run<NttFwd<LOGN, LOGR, kNttSmallKey>>(c, r.rows, lds, a);
    if (io == kNttStoreKey) return run<NttFwd<LOGN, LOGR, kNttStoreKey>>(c, r.rows, lds, a);
    if constexpr (LOGN == 11 || LOGN == 12) {        // (a pass less: latency, while a row finds a compute unit of its own)
      if (io == kNttPlain && r.rows <= c->compute_units) return run<NttFwd<LOGN, LOGR, kNttPlainFew>>(c, r.rows, lds, a);
    }
    return io == kNttPlain ? run<NttFwd<LOGN, LOGR>>(c, r.rows, lds, a) : HCNN_ERR_ARG;
  }
}

int ntt_rows(hcnn_ctx* c, const NttRows& r, bool inverse, int io = kNttPlain) {
  switch (c->logn) {
    case 10: return ntt_launch<10, 4>(c, r, inverse, io);
    case 11: return ntt_launch<11, 4>(c, r, inverse, io);
    case 12: return ntt_launch<12, 4>(c, r, inverse, io);
    // 16 residues per thread wherever 1024 threads hold the row: twice the waves of the 32-residue shapes (at n = 8192,
    // 1024 rows: forward 20.4 us with 32 residues and passes 5 + 4 + 2 + 2, 18.6 with 16 and 3 + 4 + 4 + 2; inverse
    // 20.4 and 16.8; n = 16384 8-10 % faster per row)
    case 13: return ntt_launch<13, 4>(c, r, inverse, io);
    case 14: return ntt_launch<14, 4>(c, r, inverse, io);
    case 15: return ntt_launch<15, 5>(c, r, inverse, io);
  }
  return HCNN_ERR_N;
}

// dense rows [rows][n], limb = base + r % cycle
int ntt_dense(hcnn_ctx* c, const uint32_t* in, uint32_t* out, size_t rows, uint32_t cycle, bool inverse,
              int io = kNttPlain, const uint32_t* aux = nullptr, uint32_t own_limbs = 0) {
  NttRows r{in, out, rows, cycle, 0, cycle, 0, cycle, 0, aux, own_limbs};
  return ntt_rows(c, r, inverse, io);
}

// Base-conversion kernels: one instance per number of ciphertext primes.
#define HCNN_EVERY_K(X)                                                                               \
  X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16) X(17) X(18)  \
  X(19) X(20) X(21) X(22) X(23) X(24) X(25) X(26) X(27) X(28) X(29) X(30) X(31) X(32)
static_assert(HCNN_MAX_LIMBS == 32, "HCNN_EVERY_K lists every number of primes");
int ext_dispatch(hcnn_ctx* c, size_t grid, const ExtArgs& a) {
  switch (c->k) {
#define HCNN_EXT_CASE(K) case K: return run<ExtKernel<K>>(c, grid, ExtKernel<K>::lds_bytes(), a);
    HCNN_EVERY_K(HCNN_EXT_CASE)
#undef HCNN_EXT_CASE
  }
  return HCNN_ERR_ARG;
}

int scale_dispatch(hcnn_ctx* c, size_t grid, const ScaleArgs& a) {
  switch (c->k) {
#define HCNN_SCALE_CASE(K) case K: return a.root ? run<ScaleKernel<K, true>>(c, grid, ScaleKernel<K, true>::lds_bytes(c->kp), a) \
                                                        : run<ScaleKernel<K, false>>(c, grid, ScaleKernel<K, false>::lds_bytes(c->kp), a);
    HCNN_EVERY_K(HCNN_SCALE_CASE)
#undef HCNN_SCALE_CASE
  }
  return HCNN_ERR_ARG;
}

template <int FT>
int mac_launch(hcnn_ctx* c, size_t grid, const MacArgs& a) {
  const size_t lds = MacKernel<FT>::lds_bytes(a.F, a.T);
  const size_t tiles = grid / a.G;
  const bool offsets_fit = (uint64_t)a.n_in * 2 * a.k * a.n / 4 <= 0xffffffffull;   // 16-byte offsets kept in 32 bits
  if (lds <= 64 * 1024 && lds <= c->max_lds && a.chunk >= kMacBatch && a.T >= kMacBatch && offsets_fit) {
    MacArgs b = a;
    b.chunk = a.chunk / kMacBatch * kMacBatch;      // the staged kernel reduces at batch boundaries
    // At most four workgroups per compute unit (requested through the LDS size): the inputs that the resident
    // workgroups of a die gather from then stay within its L2 (measured: 5-10 % faster on convolution shapes).
    const size_t lds_req = std::max<size_t>(lds, 36 * 1024);
    if (FT <= 8 && a.T % kMacBatch != 0)        // padded rows at few filters: skip the padding terms' multiply-adds
      return run<MacKernel<FT, true>>(c, MacKernel<FT>::grid(tiles, a.G), lds_req, b);
    return run<MacKernel<FT>>(c, MacKernel<FT>::grid(tiles, a.G), lds_req, b);
  }
  return run<MacKernelDirect<FT>>(c, grid, 0, a);
}

// Tiles per wave of a matrix form: up to K::max_steps, so that staging the tables is spread over many coefficients; fewer while the
// launch would not hold several rounds of workgroups (MacPack, whose unions take longest to stage: half as many; 4 filters x 18 terms, 16 groups, n =
// 8192, k = 6 at one / two tiles 18.9 / 15.6), or while half as many leave the fullest die a sixth less to do.  The dies take whole
// blocks of tiles: 1 to 4 blocks leave half of them idle, 9 to 12 are two rounds of which the second is half empty, 17 to 20 three (us, twice the
// tiles / these: 10 filters x 1601 terms, 130 groups, n = 1024, k = 2 1304 / 238; 16 x 1700, 130 groups, n = 8192, k = 3 2585 / 2015, k = 5 3773 /
// 3218; 16 x 1200, 256 groups, n = 2048, k = 3 861 / 752; 16 x 144, 361 groups 321 / 267; over unions 16 x 288, 196 groups, n = 4096, k = 3 491 /
// 398, k = 5 (144 groups) 533 / 490; 16 x 576, 256 groups, n = 2048, k = 3 548 / 449).  Less does not pay for staging twice: 25 to 28 blocks, an
// eighth, over unions 16 x 200, 400 groups, n = 1024, k = 13 538 / 575.
template <class K>
uint32_t mac_matrix_steps(const hcnn_ctx* c, const MacArgs& a) {
  MacArgs b = a;
  auto fullest_die = [&](uint32_t steps) {
    b.steps = steps;
    return (K::tile_blocks(b) + kXcds - 1) / kXcds * steps;
  };
  uint32_t steps = K::max_steps(a);
  while (steps > 1) {
    const uint32_t half = fullest_die(steps / 2), full = fullest_die(steps);       // (leaves b.steps = steps)
    if (K::grid(b) >= K::kLeastPerUnit * (size_t)c->compute_units && 6 * half > 5 * full) break;
    steps /= 2;
  }
  return steps;
}

template <class K>
int mac_matrix_launch(hcnn_ctx* c, const MacArgs& a, size_t lds_bytes) {
  MacArgs b = a;
  b.steps = mac_matrix_steps<K>(c, a);
  b.terms = fast_div(a.T); b.filters = fast_div(a.F);
  return run<K>(c, K::grid(b), lds_bytes, b);
}

// Neighbouring groups that a workgroup of the matrix form takes (2 or 1); 0: the call takes the vector form.
// Measured, vector / matrix form, us:
// - The matrix form, where the multiply-adds weigh more than the byte transposition (64 groups, n = 8192, k = 8: 14 filters x 25
//   terms 227 / 216, 16 x 25 259 / 237, 10 x 96 333 / 268, 16 x 144 731 / 372; 8 x 32, 135 / 174, is not taken).
// - The vector form, where the inputs are gathered less than 1.5 times and its workgroups (1024 coefficients of one group)
//   fill the chip: reading the inputs bounds the call (2 x 2 kernels without overlap, 32 channels, 16 groups x 16 filters, n =
//   8192, k = 10 310 / 325; gathered 1.65 times, 16 x 144, 9 groups, n = 16384, k = 16 513 / 462).  So does one group that fills it (8 x 64 at n = 32768, k = 24 64 / 68).
// - The matrix form, where one group's vector workgroups do not fill the chip (10 x 845, n = 8192, k = 8 127 / 58) and where the
//   vector form could not stage its row (16 x 1000, 9 groups, n = 8192, k = 10 6661 / 521).
// - Three to six groups go one at a time: half of a pair may be empty, and two pairs read their shared inputs twice (14 x 72,
//   4 groups, n = 32768, k = 12, pairs / single groups 205 / 181; 14 x 25, 3 groups, k = 24 156 / 136).
int mac_matrix_groups(const hcnn_ctx* c, size_t grid, const MacArgs& a) {
  const bool offsets_fit = (uint64_t)a.n_in * 2 * a.k * a.n / 4 <= 0xffffffffull;   // 16-byte offsets kept in 32 bits
  const size_t lds_max = std::min<size_t>(64 * 1024, c->max_lds);
  // (a row of weights bounded by zero counts its terms too: the tables are sized by them)
  const uint64_t w_max = a.w_abs_max > 0 ? (uint64_t)a.w_abs_max : 1;
  if (a.w_abs_max > 127 || a.T * w_max > kMfmaMaxSum || !offsets_fit) return 0;
  const bool many = (a.F >= 10 && a.T >= 96) || (a.F >= 14 && a.T >= 25), few_blocks = grid < 4 * (size_t)c->compute_units;
  const bool read_bound = !few_blocks && 2 * (uint64_t)a.G * a.T < 3 * (uint64_t)a.n_in;
  const bool long_row = MacKernel<1>::lds_bytes(a.F, a.T) > lds_max;
  if (!(a.G > 1 ? many && !read_bound : a.F >= 8 && a.T >= 64 && few_blocks) && !long_row) return 0;
  if (a.G >= 2 && !(a.G >= 3 && a.G <= 6) && MacMfma<2>::lds_bytes(a.T) <= lds_max) return 2;
  return MacMfma<1>::lds_bytes(a.T) <= lds_max ? 1 : 0;
}

// Tiles that a slot of the fullest die sums one after another: rounds of workgroups, two per compute unit, each with all its tiles.
template <class K>
double mac_matrix_serial_tiles(const hcnn_ctx* c, const MacArgs& a, uint32_t steps) {
  MacArgs b = a;
  b.steps = steps;
  const size_t slots = std::max<size_t>(2 * (size_t)c->compute_units / kXcds, 1);
  return (double)((K::grid(b) / kXcds + slots - 1) / slots) * steps * K::kStreams;
}

// Does a call that takes two groups per workgroup take MacPair?  Its inputs lie within 4 GiB (byte offsets in 32 bits), two workgroups'
// tables fit a compute unit, and it is done sooner: the serial tiles of the fullest die times what a tile of two groups costs, counted
// in terms of one group, staging spread over a wave's tiles.  The union has T (1 + 1 / sqrt(r)) terms where a convolution
// gathers every input r times (neighbours of an f x f kernel at stride s share f - s of f columns, r = (f / s)^2).  The other constants are fitted to
// 3000 convolutions in the sizes of all rings, both forms timed: the calls take 3.3 % less than with MacMfma<2> alone, 3.7 % less with the better
// form of every call.  The largest losses are 12 to 17 % of 80 to 130 us (108 terms, 289 groups, n = 1024, k = 3 78 / 91), stride 2 loses
// up to 8 %; rows that share nothing lose more (100 random terms, 288 groups, n = 2048, k = 4 295 / 343).  Staging and the ends of tiles weigh
// most on short rows and small launches, dies without tiles on small rings.  Us, MacMfma<2> / MacPair, 16 filters, refused: 48 terms, 576
// groups, n = 2048, k = 3 (6 blocks of tiles for 8 dies) 219 / 284; 25, 9 groups, n = 8192, k = 8 30 / 45; taken: 72, 289
// groups, n = 2048, k = 4 187 / 160; 850, 225 groups, n = 1024, k = 3 376 / 329; 576, 64 groups, n = 8192, k = 10 1502 / 1249.
bool mac_takes_pairs(const hcnn_ctx* c, const MacArgs& a) {
  if ((uint64_t)a.n_in * 2 * a.k * a.n * 4 > 0xffffffffull || MacPair::lds_bytes(a.T, a.n_in) > std::min<size_t>(80 * 1024, c->max_lds)) return false;
  const uint32_t sp = mac_matrix_steps<MacPair>(c, a), sm = mac_matrix_steps<MacMfma<2>>(c, a);
  const double T = a.T, gathered = std::max(1.0, (double)a.G * T / a.n_in);
  return mac_matrix_serial_tiles<MacPair>(c, a, sp) * (T * (1 + 1 / std::sqrt(gathered)) + 84 + 480.0 / sp) <
         mac_matrix_serial_tiles<MacMfma<2>>(c, a, sm) * (2 * T + 150 + T / sm);
}

// Groups of few filters that a call sums side by side in the sixteen rows of the matrix form (MacPack), over the union of their inputs; 0: it
// takes the vector form.  Both forms were timed on 3600 scalar MACs of up to 8 filters (all rings, 2 x 2 to 7 x 7, strides 1 and 2, up
// to 64 channels, maps up to 32 x 32; rows of random inputs), us, vector / pack:
// - Inputs gathered 3.5 times or more: geometric mean vector / pack 1.4 for convolutions.  5 x 25, stride 2, 144 groups, n = 8192, k = 8 224 / 174; 8 x 72, padded,
//   100 groups, k = 6 271 / 195; 8 x 288, 36 groups, n = 2048, k = 3 71 / 30; 1 x 72, padded 150 / 90.
// - Less often: the union saves little, and reading the inputs bounds either form (2 x 2 without overlap, 1 to 8 filters, n = 4096, k = 4 46-63 / 55-65;
//   3 x 3 at stride 2, gathered 1.7 times, n = 16384, k = 8, 4 filters 178 / 199, 8 filters 223 / 222; between 2.5 and 3.5 times as many gain as lose).
// - Little work: fewer than 150 multiply-adds a coefficient (F x T) times workgroups of the vector form for a compute unit of the fullest die.  Building the
//   union takes longer than the sums do: such calls take 10 % longer packed, 20 % where the rows are random (3 x 9, 25 groups, n = 2048, k = 4 4.9 / 7.3; 1 x 16, 36 groups, n =
//   4096, k = 3 5.3 / 8.2; 2 x 36, 31 groups of random rows, n = 2048, k = 2 5.1 / 9.9).
// - One filter and fewer than four of those workgroups, two filters and fewer than two: the sixteen or eight rows of a set share one long union, whose terms
//   run one after another in a launch that does not fill the chip (1 x 160, 16 groups, n = 2048, k = 3 10.1 / 22.4; 2 x 216, 25 groups, k = 4 21 / 27).
// - 5 or 6 filters and 200 terms or more over fewer than 64 groups at n >= 8192, gathered less than 6 times: half of these gain nothing or lose up to 10 %.
// - Fewer than 3/4 workgroups per compute unit with a tile per wave: the union's terms run one after another (1 x 125, 64 groups, n = 2048, k = 2 12 / 19).
// Of 2000 drawn convolutions whose inputs are gathered 3.5 times or more 56 take over 3 % longer than in the vector form, 27 over 10 %, nearly all of them less than
// 60 us (3 x 16, 9 groups, n = 8192, k = 7 7.7 / 10.4; 6 x 4, 961 groups, n = 1024, k = 3 43 / 58); 108 and 65 did without the lines on little work and on
// one and two filters and with eight tiles for every union.
uint32_t mac_pack_groups(const hcnn_ctx* c, const MacArgs& a) {
  const uint64_t w_max = a.w_abs_max > 0 ? (uint64_t)a.w_abs_max : 1;
  if (a.F > 8 || a.w_abs_max > 127 || a.T * w_max > kMfmaMaxSum || (uint64_t)a.n_in * 2 * a.k * a.n * 4 > 0xffffffffull) return 0;
  const uint64_t products = (uint64_t)a.G * a.T, units = c->compute_units;
  if (2 * products < 7 * (uint64_t)a.n_in) return 0;
  const uint64_t tiles = 2 * (uint64_t)a.k * a.n / (kEwThreads * kEwVec);
  const uint64_t vector_wgs = (tiles + kXcds - 1) / kXcds * a.G * kXcds;      // with every die as full as the fullest
  if (vector_wgs < 150 * units && (uint64_t)a.F * a.T * vector_wgs < 150 * units) return 0;
  if (a.F <= 2 && vector_wgs < (a.F == 1 ? 4 : 2) * units) return 0;
  if ((a.F == 5 || a.F == 6) && a.T >= 200 && a.G < 64 && a.n >= 8192 && products < 6 * (uint64_t)a.n_in) return 0;
  MacArgs b = a;
  b.pack = 16 / a.F;
  b.steps = 1;
  if (4 * MacPack::grid(b) < 3 * (size_t)c->compute_units) return 0;
  return MacPack::lds_bytes(b.pack, a.T, a.n_in) <= std::min<size_t>(64 * 1024, c->max_lds) ? b.pack : 0;
}

int mac_dispatch(hcnn_ctx* c, size_t grid, const MacArgs& a) {
  switch (mac_matrix_groups(c, grid, a)) {
    case 2:
      if (mac_takes_pairs(c, a)) return mac_matrix_launch<MacPair>(c, a, MacPair::lds_bytes(a.T, a.n_in));
      return mac_matrix_launch<MacMfma<2>>(c, a, MacMfma<2>::lds_bytes(a.T));
    case 1: return mac_matrix_launch<MacMfma<1>>(c, a, MacMfma<1>::lds_bytes(a.T));
  }
  if (const uint32_t pack = mac_pack_groups(c, a)) {
    MacArgs b = a;
    b.pack = pack;
    return mac_matrix_launch<MacPack>(c, b, MacPack::lds_bytes(b.pack, a.T, a.n_in));
  }
  switch (a.F) {
    case 1: return mac_launch<1>(c, grid, a);
    case 2: return mac_launch<2>(c, grid, a);
    case 3: return mac_launch<3>(c, grid, a);
    case 4: return mac_launch<4>(c, grid, a);
    case 5: return mac_launch<5>(c, grid, a);
    case 6: return mac_launch<6>(c, grid, a);
    case 7: return mac_launch<7>(c, grid, a);
    case 8: return mac_launch<8>(c, grid, a);
    case 9: return mac_launch<9>(c, grid, a);
    case 10: return mac_launch<10>(c, grid, a);
    case 11: return mac_launch<11>(c, grid, a);
    case 12: return mac_launch<12>(c, grid, a);
    case 13: return mac_launch<13>(c, grid, a);
    case 14: return mac_launch<14>(c, grid, a);
    case 15: return mac_launch<15>(c, grid, a);
    case 16: return mac_launch<16>(c, grid, a);
  }
  return HCNN_ERR_ARG;
}

// One-kernel relinearisation of more than 16 primes (n = 16384 takes it for up to 16)
template <int LOGN, int LOGR>
using RelinFusedLong = RelinFused<LOGN, LOGR, LOGN == 14 ? kNttFusedMac16 : kNttFusedMacAny>;

// Occupancy of the two long-running one-kernel forms for this ring and basis, asked of the runtime once.
int query_fused_occupancy(hcnn_ctx* c) {
  const uint32_t k = c->k;
  int e = 0, r = 1, t = 1;
#define HCNN_OCC(LOGN, LOGR)                                                                                          \
  {                                                                                                                   \
    const size_t lds = RelinFused<LOGN, LOGR>::kLdsBytes;                                                             \
    e = k <= 8    ? resident_workgroups_per_cu<RelinFused<LOGN, LOGR, kNttFusedMac>, RelinFusedArgs>(lds, &r)         \
        : k <= 16 ? resident_workgroups_per_cu<RelinFused<LOGN, LOGR, kNttFusedMac16>, RelinFusedArgs>(lds, &r)       \
                  : resident_workgroups_per_cu<RelinFusedLong<LOGN, LOGR>, RelinFusedArgs>(lds, &r);                  \
  }
  switch (c->logn) {
    case 10: HCNN_OCC(10, 4) break;
    case 11: HCNN_OCC(11, 4) break;
    case 12: HCNN_OCC(12, 4) break;
    case 13: HCNN_OCC(13, 4) break;
    case 14: HCNN_OCC(14, 4) break;                 // (the largest ring has no one-kernel relinearisation)
  }
#undef HCNN_OCC
  if (e) return e;
  switch (c->logn) {
    case 10: e = resident_workgroups_per_cu<TensorFused<10, 4>, TensorFusedArgs>(TensorFused<10, 4>::kLdsBytes, &t); break;
    case 11: e = resident_workgroups_per_cu<TensorFused<11, 4>, TensorFusedArgs>(TensorFused<11, 4>::kLdsBytes, &t); break;
    case 12: e = resident_workgroups_per_cu<TensorFused<12, 4>, TensorFusedArgs>(TensorFused<12, 4>::kLdsBytes, &t); break;
    case 13: e = resident_workgroups_per_cu<TensorFused<13, 4>, TensorFusedArgs>(TensorFused<13, 4>::kLdsBytes, &t); break;
    case 14: e = resident_workgroups_per_cu<TensorFused<14, 4>, TensorFusedArgs>(TensorFused<14, 4>::kLdsBytes, &t); break;
    case 15: e = resident_workgroups_per_cu<TensorFused<15, 5, 1>, TensorFusedArgs>(TensorFused<15, 5, 1>::kLdsBytes, &t); break;
  }
  if (e) return e;
  c->relin_fused_wgs = (uint32_t)r;
  c->tensor_fused_wgs = (uint32_t)t;
  return 0;
}

// Encryption and decryption rows: launches of CryptFused
constexpr size_t kCryptRows = (size_t)1 << 26;     // rows of one launch
template <class K>
int crypt_launch(hcnn_ctx* c, const CryptArgs& a) { return run<K>(c, K::grid(ntt_grouped_grid(a.n_rows, c->k)), K::kLdsBytes, a); }
template <int LOGN, int LOGR>
int crypt_fused(hcnn_ctx* c, const CryptArgs& a, bool enc, bool split) {
  if constexpr (LOGN == 13 || LOGN == 15) {
    if (split) {
      return crypt_launch<CryptFused<LOGN, LOGR, false, true, 1>>(c, a);
    }
  }
  if (enc) return crypt_launch<CryptFused<LOGN, LOGR, true>>(c, a);
  if (a.u) {
    // (the largest ring does not hold a second row in its registers)
    if constexpr (LOGN <= 14) return crypt_launch<CryptFused<LOGN, LOGR, false, true>>(c, a);
  }
  return crypt_launch<CryptFused<LOGN, LOGR, false>>(c, a);
}
int crypt_rows(hcnn_ctx* c, CryptArgs a, size_t n_ct, bool enc, bool split = false) {
  a.tw_fwd = c->d_tw_fwd; a.tw_inv = c->d_tw_inv; a.limbs = c->d_limbs; a.cycle = fast_div(c->k);
  a.n_rows = (uint32_t)(n_ct * c->k);
  switch (c->logn) {
    case 10: return crypt_fused<10, 4>(c, a, enc, split);
    case 11: return crypt_fused<11, 4>(c, a, enc, split);
    case 12: return crypt_fused<12, 4>(c, a, enc, split);
    case 13: return crypt_fused<13, 4>(c, a, enc, split);
    case 14: return crypt_fused<14, 4>(c, a, enc, split);
    case 15: return crypt_fused<15, 5>(c, a, enc, split);
  }
  return HCNN_ERR_N;
}
int secret_hat(hcnn_ctx* c, const int32_t* s, uint32_t* s_hat) {
  NttRows r{nullptr, s_hat, c->k, c->k, 0, c->k, 0, c->k, 0};
  r.small = s;
  return ntt_rows(c, r, false, kNttSmallKey);
}
// Does every (ciphertext, limb) row find a compute unit of its own?  Then a workgroup's own transform of s is shorter than
// a launch for it in front.
bool decrypts_with_own_key(const hcnn_ctx* c, size_t n_ct) { return c->logn <= 14 && n_ct * c->k <= c->compute_units; }
// Does a decryption take two workgroups per row, the rounding the last stage of their inverse transforms?  n = 8192 and 32768 while the fullest die, which has all
// rows of an eighth of the ciphertexts, has a compute unit for each half (us, whole rows / halves: n = 8192, 8 primes, 10 ciphertexts 17.5 / 14.1; n = 32768, 12
// primes, 4 49.9 / 40.8; 16 primes, 7 54.1 / 46.4).  Beyond, workgroups wait for each other: n = 8192, 10 primes, 12 ciphertexts (40 halves) 23.2 / 24.2, 26 primes, 2 (52)
// 23.5 / 25.4, n = 32768, 10 primes, 11 (40) 51.6 / 53.8, 12 primes, 10 51.6 / 54.8, 24 primes, 1 52.7 / 56.2; at n = 8192 17 to 24 primes gain as much from whole rows.
bool decrypts_by_halves(const hcnn_ctx* c, size_t n_ct) {
  const size_t fullest_die = 2 * ((n_ct + kXcds - 1) / kXcds) * c->k;
  return (c->logn == 13 || c->logn == 15) && (kSharedAll || fullest_die * kXcds <= c->compute_units);
}
// Work buffer of a decryption or a noise read-out: x [C][k][n] of up to 256 MiB (C ciphertexts a piece), then s_hat [k][n]
// unless the workgroups transform the secret themselves.
int decrypt_work(hcnn_ctx* c, size_t n_ct, bool own, size_t* C, uint32_t** x) {
  const size_t poly = (size_t)c->k * c->n;
  *C = std::min<size_t>(n_ct, std::max<size_t>(64, ((size_t)256 << 20) / (poly * 4)));
  return work_buffer(c, (*C + (own ? 0 : 1)) * poly * 4, x);
}
// x = c0 + c1*s mod q of cc ciphertexts
int decrypt_rows(hcnn_ctx* c, const int32_t* s, const uint32_t* cts, size_t cc, const uint32_t* s_hat, uint32_t* x, bool own, bool split = false) {
  CryptArgs a{};
  a.key = s_hat; a.cts = cts; a.out = x;
  a.u = own ? s : nullptr;
  return crypt_rows(c, a, cc, false, split);
}

// Median duration in milliseconds of `reps` launches of one kernel on the context's stream, one event pair each.
template <class K, class Args>
int timed_launches(hcnn_ctx* c, size_t grid, const Args& a, int reps, double* ms_out) {
  hcnn_event_t e0, e1;
  int e;
  if ((e = event_create(&e0))) return e;
  if ((e = event_create(&e1))) { event_destroy(e0); return e; }
  std::vector<float> ms;
  e = launch<K>(c->stream, grid, 0, a);                     // warm-up
  for (int r = 0; r < reps && !e; ++r) {
    float t = 0.f;
    if ((e = event_record(e0, c->stream))) break;
    if ((e = launch<K>(c->stream, grid, 0, a))) break;
    if ((e = event_record(e1, c->stream))) break;
    if ((e = stream_sync(c->stream))) break;
    if ((e = event_elapsed_ms(&t, e0, e1))) break;
    ms.push_back(t);
  }
  event_destroy(e0);
  event_destroy(e1);
  if (e) return e;
  std::sort(ms.begin(), ms.end());
  *ms_out = ms[ms.size() / 2];
  return 0;
}

}  // namespace

// ================================================================= C ABI
extern "C" {

int hcnn_gen_primes(uint32_t n, uint32_t count, uint32_t* primes_host) {
  if (!primes_host) return HCNN_ERR_NULL;
  if (!valid_n(n)) return HCNN_ERR_N;
  if (count == 0 || count > 2 * HCNN_MAX_LIMBS) return HCNN_ERR_ARG;
  const uint32_t step = 2 * n;
  uint32_t c = ((1u << 30) - 2) / step * step + 1;
  uint32_t found = 0;
  while (found < count) {
    if (c <= (1u << 29)) return HCNN_ERR_ARG;
    if (h_is_prime(c)) primes_host[found++] = c;
    c -= step;
  }
  return HCNN_OK;
}

int hcnn_min_aux_count(uint32_t n, uint32_t k, const uint32_t* q, uint64_t t, const uint32_t* cand,
                       uint32_t n_cand, uint32_t* k_aux_out) {
  if (!q || !cand || !k_aux_out) return HCNN_ERR_NULL;
  if (!valid_n(n)) return HCNN_ERR_N;
  if (k == 0 || k > HCNN_MAX_LIMBS || n_cand == 0 || n_cand > 2 * HCNN_MAX_LIMBS) return HCNN_ERR_ARG;
  int e = check_primes(n, q, k, cand, n_cand);
  if (e) return e;
  if (t < 2 || t >= (1ull << 47)) return HCNN_ERR_T;
  for (uint32_t kp = 1; kp <= n_cand && kp <= HCNN_MAX_LIMBS; ++kp) {
    if (aux_sufficient(n, q, k, t, cand, kp)) {
      *k_aux_out = kp;
      return HCNN_OK;
    }
  }
  return HCNN_ERR_AUX;
}

int hcnn_ctx_create(hcnn_ctx** out, uint32_t n, uint32_t k, const uint32_t* q, uint32_t k_aux,
                    const uint32_t* p, uint64_t t, void* hip_stream) {
  if (!out || !q || (k_aux && !p)) return HCNN_ERR_NULL;
  *out = nullptr;
  if (!valid_n(n)) return HCNN_ERR_N;
  if (k == 0 || k > HCNN_MAX_LIMBS || k_aux > HCNN_MAX_LIMBS) return HCNN_ERR_ARG;
  int e = check_primes(n, q, k, p, k_aux);
  if (e) return e;
  if (t < 2 || t >= (1ull << 47) || !h_is_prime64(t)) return HCNN_ERR_T;
  for (uint32_t i = 0; i < k; ++i)
    if (q[i] == t) return HCNN_ERR_T;
  for (uint32_t j = 0; j < k_aux; ++j)
    if (p[j] == t) return HCNN_ERR_T;
  if (k_aux && !aux_sufficient(n, q, k, t, p, k_aux)) return HCNN_ERR_AUX;

  hcnn_ctx* c = new (std::nothrow) hcnn_ctx();
  if (!c) return HCNN_ERR_ARG;
  c->n = n;
  while ((1u << c->logn) < n) ++c->logn;
  c->k = k; c->kp = k_aux; c->t = t;
  c->q.assign(q, q + k);
  if (k_aux) c->p.assign(p, p + k_aux);
  c->stream = (hcnn_stream_t)hip_stream;
  c->max_lds = max_lds_bytes();
  c->compute_units = compute_unit_count();
  if (c->max_lds < (size_t)(n + n / 32) * 4) {
    delete c;
    return HCNN_ERR_NODEVICE;
  }
  e = build_tables(c);
  if (!e) e = static_scratch_of_current_device(&c->static_scratch);
  if (!e) e = query_fused_occupancy(c);
  if (e) {
    hcnn_ctx_destroy(c);
    return e;
  }
  *out = c;
  return HCNN_OK;
}

int hcnn_ctx_destroy(hcnn_ctx* c) {
  if (!c) return HCNN_ERR_NULL;
  stream_sync(c->stream);
  fold_profile(c);
  for (auto ev : c->free_events) event_destroy(ev);
  for (void* p : c->owned) dev_free(p);
  if (c->d_evk_hat) dev_free(c->d_evk_hat);
  if (c->work) dev_free(c->work);
  if (c->small_work) dev_free(c->small_work);
  delete c;
  return HCNN_OK;
}

int hcnn_set_stream(hcnn_ctx* c, void* hip_stream) {
  if (!c) return HCNN_ERR_NULL;
  int e = stream_sync(c->stream);
  if (e) return e;
  c->stream = (hcnn_stream_t)hip_stream;
  return HCNN_OK;
}

// Smallest internal batch that takes the shared-basis relinearisation, 0: none does.  It saves k^2 - 6k transforms per
// ciphertext and pays with twice the key products and a base change.  Measured against the other forms with one q_j at a time (three
// primes, k^2 - 7k transforms, three times the products), us; two at a time the shared side takes 3 to 12 % of a squaring less, so that the lines lie on
// the safe side (n = 32768, k = 24, 4 ciphertexts 365 / 491, k = 16, 5 288 / 327, k = 12, 16 471 / 555; n = 16384, k = 16, 64 1037 / 1136):
// n = 32768  k = 24  32 ciphertexts 2255 / 3103, 6: 546 / 716, 4: 452 / 491, 1: 251 / 193;  k = 18  32: 1693 / 2017, 5: 354 / 386, 4: 303 / 305
//            k = 16  32: 1411 / 1677, 5: 295 / 327, 4: 272 / 264;  k = 13  32: 1185 / 1230, 8: 334 / 324, 5: 247 / 251, 4: 231 / 206
//            k = 12  32: 1033 / 1081, 16: 537 / 555, 8: 321 / 298, 4: 200 / 173
// n = 16384  k = 16  225: 3907 / 4110, 16: 334 / 333;  k = 11  225: 2547 / 2329;  n = 8192  k = 12  700: 3949 / 3592.
// Not measured: n = 16384 with 12 to 15 primes (left to the other forms) and with more than 16, where those forms have no
// one-kernel relinearisation and the minimum of 64 is likely too high.
static uint32_t shared_outputs(uint32_t k) { return 2 * ((k + 1) / 2); }       // (b, pair)
static size_t shared_basis_min(const hcnn_ctx* c) {
  if (c->kp < kSharedPrimes) return 0;
  if (kSharedAll) return 2;
  if (c->logn == 15) return c->k >= 18 ? 4 : c->k >= 13 ? 5 : c->k == 12 ? 16 : 0;
  return c->logn == 14 && c->k >= 16 ? 64 : 0;
}

// (Where the shared-basis relinearisation is in use the key is held a second time modulo its four primes, whatever forms the
// later calls take: 4 k^2 rows beside 2 k^2, once per key.)
int hcnn_set_relin_key(hcnn_ctx* c, const uint32_t* evk_dev) {
  if (!c || !evk_dev) return HCNN_ERR_NULL;
  if (!aligned16(evk_dev)) return HCNN_ERR_ALIGN;
  const size_t rows = (size_t)c->k * 2 * c->k;
  const size_t shared_rows = shared_basis_min(c) ? (size_t)c->k * shared_outputs(c->k) : 0;
  int e;
  const size_t own = rows * c->n, copy = shared_rows * kSharedPrimes * c->n;
  void* ptr = nullptr;
  if (!c->d_evk_hat) {
    // one allocation for both (a second one of exactly 64 MiB takes a millisecond to free; a device that cannot spare the copy, twice the
    // key's memory, keeps the other forms)
    if (copy && dev_malloc(&ptr, (own + copy) * 4) == 0) c->d_evk_shared = (uint32_t*)ptr + own;
    else if ((e = dev_malloc(&ptr, own * 4))) return e;
    c->d_evk_hat = (uint32_t*)ptr;
  } else if (copy && !c->d_evk_shared && dev_malloc(&ptr, copy * 4) == 0) {
    // (the key stays where it is: graphs that the caller recorded read it there)
    c->owned.push_back(ptr);
    c->d_evk_shared = (uint32_t*)ptr;
  }
  e = ntt_dense(c, evk_dev, c->d_evk_hat, rows, c->k, false, kNttStoreKey);
  if (e) return e;
  for (uint32_t r = 0; r < kSharedPrimes && c->d_evk_shared; ++r) {
    NttRows kr{evk_dev, c->d_evk_shared, shared_rows, 1, c->k + r, 1, 0, 1, r};
    kr.digits = shared_outputs(c->k);
    kr.tile_words = (uint32_t)(shared_rows * 64);
    kr.pair = c->d_pair;
    if ((e = ntt_rows(c, kr, false, kNttKeyTile))) return e;
  }
  c->has_key = true;
  return HCNN_OK;
}

int hcnn_ntt_fwd(hcnn_ctx* c, uint32_t* polys_dev, size_t n_polys) {
  if (!c) return HCNN_ERR_NULL;
  if (n_polys == 0) return HCNN_OK;
  if (!polys_dev) return HCNN_ERR_NULL;
  if (!aligned16(polys_dev)) return HCNN_ERR_ALIGN;
  if (n_polys > (size_t)0x7fffffff / c->k) return HCNN_ERR_ARG;
  return ntt_dense(c, polys_dev, polys_dev, n_polys * c->k, c->k, false);
}

int hcnn_ntt_inv(hcnn_ctx* c, uint32_t* polys_dev, size_t n_polys) {
  if (!c) return HCNN_ERR_NULL;
  if (n_polys == 0) return HCNN_OK;
  if (!polys_dev) return HCNN_ERR_NULL;
  if (!aligned16(polys_dev)) return HCNN_ERR_ALIGN;
  if (n_polys > (size_t)0x7fffffff / c->k) return HCNN_ERR_ARG;
  return ntt_dense(c, polys_dev, polys_dev, n_polys * c->k, c->k, true);
}

int hcnn_ct_scalar_mac(hcnn_ctx* c, const uint32_t* in, size_t n_in, const uint32_t* idx, const int32_t* w,
                       int32_t w_abs_max, size_t G, size_t F, size_t T, uint32_t* out) {
  if (!c) return HCNN_ERR_NULL;
  if (G == 0) return HCNN_OK;
  if (!in || !idx || !w || !out) return HCNN_ERR_NULL;
  if (!aligned16(in) || !aligned16(out)) return HCNN_ERR_ALIGN;
  if (n_in == 0 || n_in > 0xffffffffull || F == 0 || F > HCNN_MAX_FILTERS || T == 0 || T > 0xffffffffull ||
      w_abs_max < 0)
    return HCNN_ERR_ARG;
  if (G == 0) return HCNN_OK;
  const size_t ct_words = (size_t)2 * c->k * c->n;
  const size_t tiles = ct_words / (kEwThreads * kEwVec);
  if (G > (size_t)0x7fffffff / tiles) return HCNN_ERR_ARG;
  MacArgs a;
  a.in = in; a.idx = idx; a.w = w; a.out = out;
  a.mods = c->d_mods; a.limbs = c->d_limbs; a.k = c->k; a.n = c->n; a.steps = 0;
  a.n_in = (uint32_t)n_in; a.G = (uint32_t)G; a.F = (uint32_t)F; a.T = (uint32_t)T;
  a.w_abs_max = w_abs_max;
  // partial sums stay below 2^62 in magnitude: chunk * w_abs_max * 2^30 + 2^30 <= 2^62
  const uint64_t wm = w_abs_max > 0 ? (uint64_t)w_abs_max : 1;
  uint64_t chunk = ((1ull << 32) - 1) / wm;
  if (chunk > (1u << 30)) chunk = 1u << 30;          // a row shorter than the chunk is never folded midway
  a.chunk = (uint32_t)chunk;
  a.bad_counter = c->d_counters + 1;
  return mac_dispatch(c, G * tiles, a);
}

// Workgroups of the one-kernel relinearisation / of the one-kernel squaring tensor that the device holds at a time:
// compute units x the per-compute-unit figure that the runtime reported for the compiled kernel when the context
// was created (query_fused_occupancy).  The rounds of these long-running kernels are sized from it.
static size_t relin_fused_slots(const hcnn_ctx* c) { return (size_t)c->compute_units * c->relin_fused_wgs; }
static size_t tensor_fused_slots(const hcnn_ctx* c) { return (size_t)c->compute_units * c->tensor_fused_wgs; }

// Workgroups (ciphertext, prime) from which the one-kernel relinearisation takes `n_ct` ciphertexts that are not whole rounds of it, by
// themselves or (with_rounds) behind whole rounds.  4200 squarings of 1 to 700 ciphertexts timed with either form on 256 compute units (the lines are
// counts on that device, not shares of another one); time of a squaring with this form / with the separate kernels:
// - n = 1024 to 4096.  A workgroup transforms k + 2 rows one after another, the separate kernels all k^2 side by side, so that the line rises with k.  n = 1024, 16
//   workgroups 0.84-0.95 at up to 3 primes, but 1.2 at 5 and 6 until 24, 1.05 until 64; 7 and 8 primes 1.2 until 36, 1.05 until 160; n = 2048, 36 to 40 0.88-0.99 at up
//   to 4, 5 and 6 primes 1.05 until 64, 7 and 8 1.08 until 64, 9 to 11 1.22 at 40, 1.07 at 80, 1.05 at 350; n = 4096, 64 to 128 0.90-1.05 at up to 6, 9 to 11 1.08 at 110, 1.0
//   from 130 on, 12 to 14 1.14 at 110, 1.02 at 180, 0.96 at 300.  Ciphertexts in fours, which the separate inner product takes in one launch: n = 1024,
//   4 primes 1.05 at 48 and 64, 5 1.10 at 60 to 120, 7 1.13 at 56, 1.08 at 140, 6 1.06 at 360; n = 2048, 4 primes 1.07 at 48, 7 1.09 at 84, 6 1.03 at 312; n = 4096, 5 primes 1.08 at
//   80, 8 1.05 at 128, 0.99 at 192, 9 1.0 at 180, 12 0.92 at 384.
// - From n = 8192 on it matters whether the fullest die has a compute unit for each of its workgroups: n = 8192 190 0.99, 208 to 240 0.91-0.96 where it has, 198 to 260 1.01-1.17
//   where not, 297 to 340 0.89-0.97; n = 16384 128 1.0-1.04, 140 to 256 0.83-0.98 and 216 to 288 0.99-1.19, 320 0.97.  That die is counted with all primes of a
//   ciphertext on it, as they were when this was measured; where relin_share puts half of them there, some calls fill it less than the rule has it (17 to 20
//   ciphertexts of 12 primes: 36 workgroups counted, 30 there are) and stay with the separate kernels.
// - Behind whole rounds half as many do, whose workgroups end beside the last of those (1.0 or less; n = 16384: relin_fused_takes_rest).
constexpr uint32_t kRelinFusedMostSmall = 512, kRelinFusedMost = 288;      // the largest lines up to n = 4096 and beyond
constexpr uint32_t kRelinCts = 4;                                          // ciphertexts that share the inner product's loads of the key
static size_t relin_fused_least(const hcnn_ctx* c, size_t n_ct, bool with_rounds) {
  static constexpr uint32_t least[5] = {16, 40, 96, 192, 136};              // n = 1024 .. 16384
  const uint32_t l = least[c->logn - 10], k = c->k;
  if (with_rounds) return l / 2;
  if (c->logn <= 12) {
    const uint32_t by_primes = c->logn == 12 ? 2 * k * k : k * k * k / 2;
    const uint32_t fours = c->logn == 12 ? std::max(by_primes, std::min(24 * k, 192u)) : 4 * by_primes;
    return std::max(l, std::min(n_ct % kRelinCts == 0 ? fours : by_primes, kRelinFusedMostSmall));
  }
  return (n_ct + kXcds - 1) / kXcds * k > c->compute_units / kXcds ? kRelinFusedMost : l;
}
// Workgroups from which the one-kernel tensor is taken however its rounds are filled (the same measurements: with it / with two kernels, n =
// 1024 from 448 0.95-1.0, n = 2048 from 640 0.9-1.03, n = 4096 from 320 0.88-1.01, n = 8192 from 384 0.94-1.01, n = 32768 from 320 0.93-1.02; n = 16384, 0.95-1.05
// from 320 on, goes by its rounds alone: 0).
static size_t tensor_fused_least(const hcnn_ctx* c) {
  static constexpr size_t least[6] = {448, 640, 320, 384, 0, 320};
  return least[c->logn - 10];
}
// Workgroups of the one-kernel tensor of n_ct ciphertexts: one per (ciphertext, limb) pair, at n = 32768 two.
static size_t tensor_fused_wgs(const hcnn_ctx* c, size_t n_ct) { return n_ct * (c->k + c->kp) * (c->logn == 15 ? 2 : 1); }
// Does the default policy take it?  Its workgroups are long (five transforms), so it pays when they fill their rounds.  Measured at n = 8192, k = 8: 1.06 us
// per ciphertext in full rounds against 1.25 of the two separate kernels (64 to 512 ciphertexts), a ratio of 0.85; at n = 32768, k = 24 15.5 against
// 18.8 (32), 0.82.  A last round that is only partly filled is shorter too (workgroups with a compute unit to themselves run faster), so that from
// tensor_fused_least workgroups on it pays whatever their number.
static bool takes_tensor_fused(const hcnn_ctx* c, size_t n_ct) {
  const size_t wgs = tensor_fused_wgs(c, n_ct), least = tensor_fused_least(c);
  const size_t slots = tensor_fused_slots(c), rounds = (wgs + slots - 1) / slots;
  return (least && wgs >= least) || wgs * 8 >= rounds * slots * 7;
}

// Limbs of a ciphertext whose workgroups run side by side on one die in the one-kernel relinearisation.  All k read every digit row once, but bring the
// whole key (2 k^2 n words) into the die's L2 for the few ciphertexts that are there at a time; half of them read the digits on two dies
// and half of the key, for twice the ciphertexts.  Us, all / half / a quarter: n = 8192, k = 8, 64 squarings 185 / 182.5 / 182.7, 720 1987 / 1979 / 1990,
// k = 10, 64 266 / 263 / 266, k = 12, 512 2512 / 2475 / 2461; n = 16384, k = 12, 200 2123 / 2103 / 2108, k = 16, 40 726 / 717 / 717, k = 8, 64 411 / 407 / 406.
// A key that one L2 (4 MiB) holds gains nothing: n = 8192, k = 6, 400 795 / 799 / 799, n = 4096, k = 6, 1000 970 / 970 / 973.  (An odd k has no even halves.)
static uint32_t relin_share(const hcnn_ctx* c) {
  const bool outgrows_l2 = (size_t)2 * c->k * c->k * c->n * 4 >= ((size_t)4 << 20);
  return outgrows_l2 && c->k % 2 == 0 ? c->k / 2 : c->k;
}

// Does the one-kernel relinearisation take all n_ct ciphertexts of a batch, or the first `whole` of them, whole rounds by the count of ciphertexts?  At n =
// 16384, where a compute unit holds one workgroup, the rest joins if the fullest die, with its share of the limbs, goes through no more rounds for it (0.94-0.95
// of the time of the separate kernels for the rest) or fills the last one to half (0.93-0.96; less filled 1.02-1.09): 1060 squarings.  12 primes, 39 ciphertexts 473 /
// 529 us, 23 281 / 266; 11 primes, 55 598 / 656.
static bool relin_fused_takes_rest(const hcnn_ctx* c, size_t n_ct, size_t whole) {
  if (whole && c->logn == 14) {
    const size_t share = relin_share(c), slots = relin_fused_slots(c) / kXcds;
    auto on_die = [&](size_t cts) { return (cts * (c->k / share) + kXcds - 1) / kXcds * share; };
    const size_t last = (on_die(n_ct) - 1) % slots + 1;
    return (on_die(n_ct) - 1) / slots == (on_die(whole) - 1) / slots || 2 * last >= slots;
  }
  return (n_ct - whole) * c->k >= relin_fused_least(c, n_ct - whole, whole != 0);
}

// Ciphertexts of a batch that go to the separate kernels at most, where the one-kernel form is there: what the work buffer has room for.
static size_t relin_split_most(const hcnn_ctx* c, size_t fused_round) {
  return std::min(fused_round, (size_t)(c->logn <= 12 ? kRelinFusedMostSmall : kRelinFusedMost) / c->k + 1);
}

// Steps 6-8 through the shared basis (fv_kernels.h): y [n_ct][3][k][n] -> out; dig 4k, acc 4 and (largest ring only) z 4 rows an output
// per ciphertext.
static int relin_shared(hcnn_ctx* c, const uint32_t* y, size_t n_ct, uint32_t* dig, uint32_t* acc, uint32_t* z, uint32_t* out) {
  const uint32_t k = c->k, n = c->n, outs = shared_outputs(k);
  int e;
  NttRows r{y, dig, n_ct * k * kSharedPrimes, kSharedPrimes, k, kSharedPrimes, 0, kSharedPrimes, 0};
  r.tile_words = k * 64;
  if ((e = ntt_rows(c, r, false, kNttDigitTile))) return e;
  RelinSharedArgs sa{dig, c->d_evk_shared, acc, c->d_limbs + k, k, outs, n, (uint32_t)n_ct, (uint32_t)((n_ct + 7) / 8)};
  const size_t grid = (size_t)kSharedPrimes * (n / 64) * sa.n_grp;
  // (the profile's unit is three for a tile of 64 coefficients and eight ciphertexts, whose workgroups are kSharedPrimes: counted from the grid)
  const size_t units = grid * 3 / kSharedPrimes;
  switch ((outs + 7) / 8) {
#define HCNN_SHARED_MAC(O) case O: e = run<RelinSharedMac<O>>(c, grid, RelinSharedMac<O>::lds_bytes(k), sa, units); break;
#ifdef HCNN_SHARED_ALL
    HCNN_SHARED_MAC(1)
#endif
    HCNN_SHARED_MAC(2) HCNN_SHARED_MAC(3) HCNN_SHARED_MAC(4)
#undef HCNN_SHARED_MAC
    default: e = HCNN_ERR_ARG; break;
  }
  if (e) return e;
  const size_t rows = n_ct * outs;
  if (c->logn == 15) {
    NttRows b{acc, z, rows * kSharedPrimes, kSharedPrimes, k, kSharedPrimes, 0, kSharedPrimes, 0};
    b.digits = outs;
    b.tile_words = outs * 64;
    if ((e = ntt_rows(c, b, true, kNttBackRow))) return e;
    RelinCombineArgs ca{z, y, out, c->d_limbs, c->d_crt, c->crt_inv, fast_div(outs), k, n};
    return run<RelinCombine>(c, rows * (n / (kEwThreads * RelinCombine::kPer * 2)), 0, ca);
  }
  RelinBackArgs ba{acc, y, out, c->d_tw_inv, c->d_limbs, c->d_crt, c->crt_inv, k, fast_div(outs), k};
  switch (c->logn) {
#define HCNN_BACK(LOGN) case LOGN: return run<RelinBack<LOGN, 4>>(c, rows, RelinBack<LOGN, 4>::kLdsBytes, ba, kSharedPrimes * rows);
#ifdef HCNN_SHARED_ALL
    HCNN_BACK(10) HCNN_BACK(11) HCNN_BACK(12) HCNN_BACK(13)
#endif
    HCNN_BACK(14)
#undef HCNN_BACK
  }
  return HCNN_ERR_N;
}

// HMult of Sec. 2.1 on n_ct pairs (a_i, b_i); b == nullptr squares a (HSquare).
// static_ws: the intermediate polynomials go to this device's copy of the file-scope array `scratch` and nothing is
// allocated; a parameter set whose single ciphertext does not fit that array is refused.
static int mul_relin_impl(hcnn_ctx* c, const uint32_t* in, const uint32_t* in_b, size_t n_ct, uint32_t* out,
                          bool static_ws = false) {
  if (!c) return HCNN_ERR_NULL;
  if (n_ct == 0) return HCNN_OK;
  if (!in || !out) return HCNN_ERR_NULL;
  if (!aligned16(in) || !aligned16(out) || !aligned16(in_b)) return HCNN_ERR_ALIGN;
  if (c->kp == 0) return HCNN_ERR_AUX;
  const uint32_t k = c->k, kp = c->kp, L = k + kp, n = c->n;
  const size_t rn = n;
  const size_t ext_rows = in_b ? 4 * (size_t)L : 2 * (size_t)L;
  if (static_ws && (ext_rows + 3 * L + 3 * k + (size_t)k * k + 2 * k) * rn * 4 > kStaticScratchBytes)
    return HCNN_ERR_SCRATCH;
  if (!c->has_key) return HCNN_ERR_NOKEY;
  // n <= 16384: relinearisation runs as one kernel that needs no buffers for the transformed digits and the sums.
  // (At n = 16384 its 1024-thread workgroup fills a compute unit alone: measured +5..8 % up to 16 primes, no gain
  // with the in-loop folds of longer bases, which stay with the separate kernels; at n = 32768 a row and its sums
  // do not fit the registers of 1024 threads.)
  // Its workgroups are long (k + 2 transforms each): small batches go through the three separate kernels, which spread k^2
  // rows per ciphertext over the chip (relin_fused_least).
  const size_t shared_min = c->fusion == 0 && !static_ws && c->d_evk_shared ? shared_basis_min(c) : 0;
  const bool fused = c->fusion != 1 && (c->logn <= 13 || (c->logn == 14 && k <= 16));
  // (a round is counted in whole ciphertexts per die, also where half of a ciphertext's workgroups share one: relin_share)
  const size_t fused_round = fused ? relin_fused_slots(c) / kXcds / k * kXcds : 0;   // ciphertexts per round (0: never)
  const size_t words_main = (ext_rows + 3 * L + 3 * k) * rn;
  const size_t words_split = ((size_t)k * k + 2 * k) * rn, words_shared = (size_t)kSharedPrimes * (k + shared_outputs(k)) * rn;
  const size_t words_per_ct = words_main + (shared_min ? words_shared : words_split);
  size_t C = c->square_chunk;
  // 6 GiB of work buffer (of 288 GB): enough rows per launch at every n
  const size_t budget = static_ws ? kStaticScratchBytes : (size_t)6 << 30;
  if (static_ws && C > budget / (words_per_ct * 4)) C = 0;
  if (C == 0) {
    C = budget / (words_per_ct * 4);
    // measured: up to n = 8192 batches of 512 are 3-4 % faster than 256 (the long workgroups of the one-kernel
    // relinearisation leave a longer tail per launch), at n = 16384 128-256 is best; small rings need more
    // ciphertexts to fill the chip at all
    const size_t cap = std::max<size_t>(c->logn <= 13 ? 512 : 256, fused_round);
    if (C > cap) C = cap;
    if (!shared_min && fused_round && C > fused_round) C = C / fused_round * fused_round;   // whole rounds of the one-kernel relinearisation
    if (c->logn >= 14 && n_ct > C && !static_ws) {
      // batches of about the same size rather than a short last one, which would miss the shared basis (us: n = 16384, k = 16, 300 ciphertexts 4475 /
      // 4370, k = 8, 400 2503 / 2485; smaller rings lose up to 1 %)
      const size_t even = (n_ct + (n_ct + C - 1) / C - 1) / ((n_ct + C - 1) / C);
      C = !shared_min && fused_round ? std::min(C, (even + fused_round - 1) / fused_round * fused_round) : even;
    }
  }
  if (C < 1) C = 1;
  if (C > n_ct) C = n_ct;
  // ciphertexts of one internal batch that can take the separate kernels
  const size_t C_split = shared_min ? std::min(C, shared_min - 1) : (fused && fused_round) ? std::min(C, relin_split_most(c, fused_round)) : C;
  int e;
  uint32_t* ext = c->static_scratch;
  e = static_ws ? 0 : work_buffer(c, (C * words_main + std::max(C_split * words_split, shared_min ? C * words_shared : 0)) * 4, &ext);
  if (e) return e;
  uint32_t* ext_b = ext + C * 2 * L * rn;                 // used only by the two-operand product
  uint32_t* d = ext + C * ext_rows * rn;
  uint32_t* y = d + C * 3 * L * rn;
  uint32_t* dig = y + C * 3 * k * rn;
  const size_t ct_words = (size_t)2 * k * rn;
  const size_t bpp = n / kEwThreads;                 // blocks per polynomial, 1 coefficient / thread
  const size_t bpr = n / (kEwThreads * kEwVec);      // blocks per row, 4 coefficients / thread

  // How many ciphertexts of an internal batch of cc take the one-kernel relinearisation (steps 6-8 in one kernel: a row and its two
  // 64-bit sums stay in registers): all whole rounds of its workgroups, and what is left if that is enough by itself.
  auto fused_count = [&](size_t cc) -> size_t {
    if (!fused || !fused_round) return 0;
    if (c->fusion == 2) return cc;
    const size_t whole = cc / fused_round * fused_round;
    return relin_fused_takes_rest(c, cc, whole) ? cc : whole;
  };
  // One internal batch: ciphertexts [c0, c0 + cc) of the call, nf of
  // them through the one-kernel relinearisation.
  auto one_batch = [&](size_t c0, size_t cc, size_t nf) -> int {
    int e;
    uint32_t* const b_ext = ext;
    uint32_t* const b_ext_b = ext_b;
    uint32_t* const b_d = d;
    uint32_t* const b_y = y;
    const bool shared = shared_min && cc >= shared_min;
    uint32_t* const b_dig = dig;
    uint32_t* const b_acc = dig + (shared ? cc * kSharedPrimes : (cc - nf) * k) * k * rn;
    // 1. centred lift of c0, c1 extended to the auxiliary primes (only the new rows are written);
    // 2. forward NTT over all k + k' limbs, the first k read from the ciphertext itself
    // (forward rows by two workgroups: the new rows are staged in the array of the tensor, free until step 3, because that transform
    // cannot work in place)
    const bool tensor_fused = !in_b && c->fusion != 1 && (c->fusion == 2 || takes_tensor_fused(c, cc));      // steps 2 and 3 in one kernel
    const bool staged = !tensor_fused && splits_rows(c, cc * 2 * L);
    uint32_t* const b_new = staged ? b_d : b_ext;
    ExtArgs ea;
    ea.in = in + c0 * ct_words; ea.out = b_new; ea.bc = c->ext; ea.n = n; ea.band = c->band;
    ea.fallback_counter = c->d_counters;
    if ((e = ext_dispatch(c, cc * 2 * bpp, ea))) return e;
    if (tensor_fused) {
      TensorFusedArgs ta{in + c0 * ct_words, b_ext, b_d, c->d_tw_fwd, c->d_tw_inv, c->d_limbs, k, L, (uint32_t)(cc * L), fast_div(L), {0, 0}};
      // (up to one and a half rounds the order of the limbs gains nothing: n = 32768, k = 12, 8 ciphertexts 273 / 276 us)
      if (2 * tensor_fused_wgs(c, cc) > 3 * tensor_fused_slots(c)) ta.cts_div = fast_div((uint32_t)cc);
      const size_t rows = cc * L * 5;
      switch (c->logn) {
        case 10: e = run<TensorFused<10, 4>>(c, cc * L, TensorFused<10, 4>::kLdsBytes, ta, rows); break;
        case 11: e = run<TensorFused<11, 4>>(c, cc * L, TensorFused<11, 4>::kLdsBytes, ta, rows); break;
        case 12: e = run<TensorFused<12, 4>>(c, cc * L, TensorFused<12, 4>::kLdsBytes, ta, rows); break;
        case 13: e = run<TensorFused<13, 4>>(c, cc * L, TensorFused<13, 4>::kLdsBytes, ta, rows); break;
        // (1024 threads while every pair has a compute unit of its own, else two workgroups of 512 on each; both are counted in rounds of
        // one per compute unit.  Us, 1024 / 512 threads: 252 pairs 40 / 46, 504 77 / 71, 756 116 / 108, 7650 1140 / 1030)
        case 14:
          e = cc * L <= c->compute_units ? run<TensorFused<14, 4>>(c, cc * L, TensorFused<14, 4>::kLdsBytes, ta, rows)
                                         : run<TensorFused<14, 5>>(c, cc * L, TensorFused<14, 5>::kLdsBytes, ta, rows);
          break;
        case 15: e = run<TensorFused<15, 5, 1>>(c, TensorFused<15, 5, 1>::grid(cc * L), TensorFused<15, 5, 1>::kLdsBytes, ta, rows); break;
        default: e = HCNN_ERR_N; break;
      }
      if (e) return e;
    } else if ((e = ntt_dense(c, b_new, b_ext, cc * 2 * L, L, false, kNttStoreLazy, in + c0 * ct_words, k))) {
      return e;
    }
    if (in_b) {
      uint32_t* const b_new_b = staged ? b_d : b_ext_b;
      ea.in = in_b + c0 * ct_words; ea.out = b_new_b;
      if ((e = ext_dispatch(c, cc * 2 * bpp, ea))) return e;
      if ((e = ntt_dense(c, b_new_b, b_ext_b, cc * 2 * L, L, false, kNttStoreLazy, in_b + c0 * ct_words, k))) return e;
    }
    // 3+4. tensor formed while loading, then back to coefficients: the integer tensor, known mod q*p
    if (in_b) {
      if ((e = ntt_dense(c, b_ext, b_d, cc * 3 * L, L, true, kNttLoadTensorMul, b_ext_b))) return e;
    } else if (!tensor_fused) {
      if ((e = ntt_dense(c, b_ext, b_d, cc * 3 * L, L, true, kNttLoadTensor))) return e;
    }
    // 5. y = round(t/q * d) mod q
    const bool by_halves = tensor_fused ? c->logn == 15 : splits_tensor_rows(c, cc * 3 * L);
    ScaleArgs sa;
    sa.d = b_d; sa.y = b_y; sa.to_p = c->to_p; sa.to_q = c->to_q; sa.tq_inv = c->d_tq_inv; sa.limbs = c->d_limbs; sa.root = by_halves ? c->d_scale_root : nullptr; sa.n = n;
    sa.band = c->band; sa.fallback_counter = c->d_counters;
    if ((e = scale_dispatch(c, cc * 3 * bpp, sa))) return e;
    if (shared) return relin_shared(c, b_y, cc, b_dig, b_acc, b_d, out + c0 * ct_words);     // (the tensor's rows, 3L > 4k + 4, are free by now)
    // 6-8 in one kernel
    if (nf) {
      RelinFusedArgs fa{b_y, c->d_evk_hat, out + c0 * ct_words, c->d_tw_fwd, c->d_tw_inv, c->d_limbs, k, (uint32_t)(nf * k), fast_div(k), fast_div(relin_share(c))};
      const size_t grid = ntt_grouped_grid(nf * k, relin_share(c)), rows = nf * k * (k + 2);
#define HCNN_FUSED(LOGN, LOGR)                                                                                      \
  (k <= 8 ? run<RelinFused<LOGN, LOGR, kNttFusedMac>>(c, grid, RelinFused<LOGN, LOGR, kNttFusedMac>::kLdsBytes, fa, rows)             \
          : k <= 16 ? run<RelinFused<LOGN, LOGR, kNttFusedMac16>>(c, grid, RelinFused<LOGN, LOGR, kNttFusedMac16>::kLdsBytes, fa, rows) \
                    : run<RelinFusedLong<LOGN, LOGR>>(c, grid, RelinFusedLong<LOGN, LOGR>::kLdsBytes, fa, rows))
      switch (c->logn) {
        case 10: e = HCNN_FUSED(10, 4); break;
        case 11: e = HCNN_FUSED(11, 4); break;
        case 12: e = HCNN_FUSED(12, 4); break;
        case 13: e = HCNN_FUSED(13, 4); break;
        case 14: e = HCNN_FUSED(14, 4); break;
        default: e = HCNN_ERR_N; break;
      }
#undef HCNN_FUSED
      if (e) return e;
    }
    const size_t ns = cc - nf;                                // ciphertexts left for the separate kernels
    if (ns == 0) return 0;
    const uint32_t* y_s = b_y + nf * 3 * k * rn;
    uint32_t* out_s = out + (c0 + nf) * ct_words;
    // 6. RNS digits of y2, each reduced modulo every q_j while loading, transformed
    if ((e = ntt_dense(c, y_s, b_dig, ns * k * k, k, false, kNttLoadDigit))) return e;
    // 7. inner product with the evaluation key
    RelinMacArgs ra;
    ra.dig = b_dig; ra.evk = c->d_evk_hat; ra.acc = b_acc; ra.limbs = c->d_limbs; ra.k = k; ra.n = n;
    // in the plain (ciphertext-major) order every die touches the key tiles of all limbs: 2*k*k*(tiles/8) * 4 KiB
    ra.key_major = (bpr % kXcds == 0 && (size_t)2 * k * k * (bpr / kXcds) * 4096 > ((size_t)1 << 20)) ? 1u : 0u;
    if (c->relin_order == 1) ra.key_major = 0;
    if (c->relin_order == 2 && bpr % kXcds == 0) ra.key_major = 1;
    // groups of kRelinCts ciphertexts share their loads of the key; the remainder goes one by one
    const size_t full = ns / kRelinCts;
    if (full) {
      ra.n_grp = (uint32_t)full; ra.ct_base = 0;
      if ((e = run<RelinMacKernel<kRelinCts>>(c, full * k * bpr, 0, ra))) return e;
    }
    if (ns % kRelinCts) {
      ra.n_grp = (uint32_t)(ns % kRelinCts); ra.ct_base = (uint32_t)(full * kRelinCts);
      if ((e = run<RelinMacKernel<1>>(c, (ns % kRelinCts) * k * bpr, 0, ra))) return e;
    }
    // 8. c'_b = y_b + sum_i evk[i][b] * digit_i : inverse transform with the addition on the way out
    return ntt_dense(c, b_acc, out_s, ns * 2 * k, k, true, kNttStoreAdd, y_s);
  };

  for (size_t c0 = 0; c0 < n_ct; c0 += C) {
    const size_t cc = std::min(C, n_ct - c0);
    const size_t nf = fused_count(cc);
    if ((e = one_batch(c0, cc, nf))) return e;
  }
  return HCNN_OK;
}

int hcnn_ct_square_relin(hcnn_ctx* c, const uint32_t* in, size_t n_ct, uint32_t* out) {
  return mul_relin_impl(c, in, nullptr, n_ct, out);
}

int hcnn_ct_mul_relin(hcnn_ctx* c, const uint32_t* a, const uint32_t* b, size_t n_ct, uint32_t* out) {
  if (n_ct != 0 && c && !b) return HCNN_ERR_NULL;
  return mul_relin_impl(c, a, b, n_ct, out);
}

int hcnn_ct_square_relin_noalloc(hcnn_ctx* c, const uint32_t* in, size_t n_ct, uint32_t* out) {
  if (!c) return HCNN_ERR_NULL;
  // no event pair around the launches of this call: an event may have to be created
  const bool profile = c->profile;
  c->profile = false;
  const int e = mul_relin_impl(c, in, nullptr, n_ct, out, true);
  c->profile = profile;
  return e;
}

// ---------------------------------------------------------------- test helpers
int hcnn_keygen(hcnn_ctx* c, const int32_t* s, const uint32_t* a, const int32_t* e_small, const uint32_t* a_evk,
                const int32_t* e_evk, uint32_t* pk_out, uint32_t* evk_out) {
  if (!c || !s || !a || !e_small || !pk_out) return HCNN_ERR_NULL;
  if (evk_out && (!a_evk || !e_evk)) return HCNN_ERR_NULL;
  if (!aligned16(a) || !aligned16(pk_out) || !aligned16(a_evk) || !aligned16(evk_out)) return HCNN_ERR_ALIGN;
  const uint32_t k = c->k, n = c->n;
  const size_t rn = n, poly = (size_t)k * rn;
  const size_t bpp = n / kEwThreads;
  // scratch: s_hat [k][n] | s2 [k][n] | tmp [k*k][n]
  uint32_t* s_hat;
  int e = work_buffer(c, (2 * poly + (size_t)k * poly) * 4, &s_hat);
  if (e) return e;
  uint32_t* s2 = s_hat + poly;
  uint32_t* tmp = s2 + poly;

  SmallToRnsArgs sr{s, s_hat, c->d_mods, k, n};
  if ((e = run<SmallToRnsKernel>(c, bpp, 0, sr))) return e;
  if ((e = ntt_dense(c, s_hat, s_hat, k, k, false))) return e;

  // pk = (e - a*s, a)
  if ((e = ntt_dense(c, a, tmp, k, k, false))) return e;
  PointMulArgs pm{tmp, s_hat, tmp, c->d_mods, k, n, k, k, 1u};
  if ((e = run<PointMulKernel>(c, (size_t)k * bpp, 0, pm))) return e;
  if ((e = ntt_dense(c, tmp, tmp, k, k, true))) return e;
  AddSmallArgs as{tmp, e_small, pk_out, c->d_mods, k, n, 0u, 2 * k, 0u};
  if ((e = run<AddSmallKernel>(c, (size_t)k * bpp, 0, as))) return e;
  if ((e = copy_d2d(pk_out + poly, a, poly * 4, c->stream))) return e;
  if (!evk_out) return HCNN_OK;

  // s^2, coefficient domain
  PointMulArgs p2{s_hat, s_hat, s2, c->d_mods, k, n, k, k, 0u};
  if ((e = run<PointMulKernel>(c, (size_t)k * bpp, 0, p2))) return e;
  if ((e = ntt_dense(c, s2, s2, k, k, true))) return e;
  // evk[i][0] = g_i*s^2 - (a_i*s + e_i), evk[i][1] = a_i, all components at once
  if ((e = ntt_dense(c, a_evk, tmp, (size_t)k * k, k, false))) return e;
  PointMulArgs pe{tmp, s_hat, tmp, c->d_mods, k, n, k * k, k, 1u};
  if ((e = run<PointMulKernel>(c, (size_t)k * k * bpp, 0, pe))) return e;
  if ((e = ntt_dense(c, tmp, tmp, (size_t)k * k, k, true))) return e;
  AddSmallArgs ae{tmp, e_evk, evk_out, c->d_mods, k, n, 1u, 2 * k, 0u};
  if ((e = run<AddSmallKernel>(c, (size_t)k * k * bpp, 0, ae))) return e;
  AddDiagArgs ad{evk_out, s2, c->d_mods, k, n};
  if ((e = run<AddDiagKernel>(c, (size_t)k * bpp, 0, ad))) return e;
  for (uint32_t i = 0; i < k; ++i)
    if ((e = copy_d2d(evk_out + ((size_t)i * 2 + 1) * poly, a_evk + (size_t)i * poly, poly * 4, c->stream))) return e;
  return HCNN_OK;
}

static int encrypt_impl(hcnn_ctx* c, const uint32_t* pk, const uint32_t* m, const uint64_t* m64, const int32_t* u,
                        const int32_t* e1, const int32_t* e2, size_t n_ct, uint32_t* ct_out) {
  if (!c || !pk || (!m && !m64) || !u || !e1 || !e2 || !ct_out) return HCNN_ERR_NULL;
  if ((m != nullptr) != (c->t < (1ull << 32))) return HCNN_ERR_T;     // word size of the plaintext follows t
  if (!aligned16(pk) || !aligned16(ct_out)) return HCNN_ERR_ALIGN;
  if (n_ct == 0) return HCNN_OK;
  const uint32_t k = c->k, n = c->n;
  const size_t rn = n, poly = (size_t)k * rn;
  // scratch: pk_hat [2][k][n]
  uint32_t* pk_hat;
  int e = work_buffer(c, 2 * poly * 4, &pk_hat);
  if (e) return e;
  if ((e = ntt_dense(c, pk, pk_hat, 2 * (size_t)k, k, false, kNttStoreKey))) return e;
  const size_t C = kCryptRows / k;               // rows of a launch fit its 32-bit indices
  for (size_t c0 = 0; c0 < n_ct; c0 += C) {
    CryptArgs a{};
    a.key = pk_hat; a.u = u + c0 * rn; a.e1 = e1 + c0 * rn; a.e2 = e2 + c0 * rn;
    a.msg = m ? m + c0 * rn : nullptr; a.msg64 = m64 ? m64 + c0 * rn : nullptr; a.scale = c->d_delta;
    a.out = ct_out + c0 * 2 * poly;
    if ((e = crypt_rows(c, a, std::min(C, n_ct - c0), true))) return e;
  }
  return HCNN_OK;
}

int hcnn_encrypt(hcnn_ctx* c, const uint32_t* pk, const uint32_t* m, const int32_t* u, const int32_t* e1,
                 const int32_t* e2, size_t n_ct, uint32_t* ct_out) {
  if (!m) return HCNN_ERR_NULL;
  return encrypt_impl(c, pk, m, nullptr, u, e1, e2, n_ct, ct_out);
}

int hcnn_encrypt_wide(hcnn_ctx* c, const uint32_t* pk, const uint64_t* m, const int32_t* u, const int32_t* e1,
                      const int32_t* e2, size_t n_ct, uint32_t* ct_out) {
  if (!m) return HCNN_ERR_NULL;
  return encrypt_impl(c, pk, nullptr, m, u, e1, e2, n_ct, ct_out);
}

static int decrypt_impl(hcnn_ctx* c, const int32_t* sk, const uint32_t* ct, size_t n_ct, uint32_t* m_out,
                        uint64_t* m_out64) {
  if (!c || !sk || !ct || (!m_out && !m_out64)) return HCNN_ERR_NULL;
  if ((m_out != nullptr) != (c->t < (1ull << 32))) return HCNN_ERR_T;
  if (!aligned16(ct)) return HCNN_ERR_ALIGN;
  if (n_ct == 0) return HCNN_OK;
  const uint32_t k = c->k, n = c->n;
  const size_t rn = n, poly = (size_t)k * rn;
  const size_t bpp = n / kEwThreads;
  const bool split = decrypts_by_halves(c, n_ct), own = split || decrypts_with_own_key(c, n_ct);
  size_t C;
  uint32_t* x;
  int e = decrypt_work(c, n_ct, own, &C, &x);
  if (e) return e;
  uint32_t* s_hat = x + C * poly;                // (not there with its own key)
  if (!own && (e = secret_hat(c, sk, s_hat))) return e;
  for (size_t c0 = 0; c0 < n_ct; c0 += C) {
    const size_t cc = std::min(C, n_ct - c0);
    if ((e = decrypt_rows(c, sk, ct + c0 * 2 * poly, cc, s_hat, x, own, split))) return e;
    DecRoundArgs da;
    da.cts = ct + c0 * 2 * poly; da.limbs = c->d_limbs;
    da.x = x; da.m_out = m_out ? m_out + c0 * rn : nullptr; da.m_out64 = m_out64 ? m_out64 + c0 * rn : nullptr;
    da.bc = c->dec; da.tab = c->d_dec_tab; da.t = c->t; da.n = n;
    da.band = c->band; da.fallback_counter = c->d_counters;
    const size_t lds = DecRoundKernel<true, true>::lds_bytes(k);
    if ((e = split    ? run<DecRoundKernel<true, true>>(c, cc * bpp, lds, da)
             : k >= 4 ? run<DecRoundKernel<false, true>>(c, cc * bpp, lds, da)
                      : run<DecRoundKernel<false, false>>(c, cc * bpp, lds, da))) return e;
  }
  return HCNN_OK;
}

int hcnn_decrypt(hcnn_ctx* c, const int32_t* sk, const uint32_t* ct, size_t n_ct, uint32_t* m_out) {
  if (!m_out) return HCNN_ERR_NULL;
  return decrypt_impl(c, sk, ct, n_ct, m_out, nullptr);
}

int hcnn_decrypt_wide(hcnn_ctx* c, const int32_t* sk, const uint32_t* ct, size_t n_ct, uint64_t* m_out) {
  if (!m_out) return HCNN_ERR_NULL;
  return decrypt_impl(c, sk, ct, n_ct, nullptr, m_out);
}

int hcnn_noise_bits(hcnn_ctx* c, const int32_t* sk, const uint32_t* ct, size_t n_ct, uint32_t* bits_out) {
  if (!c || !sk || !ct || !bits_out) return HCNN_ERR_NULL;
  if (!aligned16(ct)) return HCNN_ERR_ALIGN;
  if (n_ct == 0) return HCNN_OK;
  const uint32_t k = c->k, n = c->n;
  const size_t rn = n, poly = (size_t)k * rn;
  const size_t bpp = n / kEwThreads;
  const bool own = decrypts_with_own_key(c, n_ct);
  size_t C;
  uint32_t* x;
  int e = decrypt_work(c, n_ct, own, &C, &x);
  if (e) return e;
  uint32_t* s_hat = x + C * poly;                // (not there with its own key)
  if ((e = dev_memset(bits_out, 0, n_ct * sizeof(uint32_t), c->stream))) return e;
  if (!own && (e = secret_hat(c, sk, s_hat))) return e;
  for (size_t c0 = 0; c0 < n_ct; c0 += C) {
    const size_t cc = std::min(C, n_ct - c0);
    if ((e = decrypt_rows(c, sk, ct + c0 * 2 * poly, cc, s_hat, x, own))) return e;
    NoiseArgs na;
    na.x = x; na.bits = bits_out + c0; na.bc = c->dec; na.n = n;
    if ((e = run<NoiseKernel>(c, cc * bpp, NoiseKernel::lds_bytes(k), na))) return e;
  }
  return HCNN_OK;
}

// ---------------------------------------------------------------- sampling
namespace {
// T[v] = floor(2^32 * P(|X| <= v)), X = round(N(0, 3.2^2)), v = 0..19: a format constant of the samplers
const uint32_t kGaussT[20] = {533280463u, 1549416568u, 2428136261u, 3117868636u, 3609276189u, 3927060812u, 4113592370u,
                              4212972233u, 4261030606u, 4282124752u, 4290528529u, 4293567340u, 4294564687u, 4294861785u,
                              4294942112u, 4294961823u, 4294966213u, 4294967101u, 4294967264u, 4294967291u};

int sample_impl(hcnn_ctx* c, uint32_t kind, uint64_t seed, uint64_t stream, void* out, size_t count) {
  if (!c) return HCNN_ERR_NULL;
  if (count == 0) return HCNN_OK;
  if (!out) return HCNN_ERR_NULL;
  int e;
  if (!c->d_gauss_t) {
    std::vector<uint32_t> tab(kGaussT, kGaussT + 20);
    if ((e = upload(c, tab, &c->d_gauss_t))) return e;
  }
  SampleArgs a;
  a.out = out; a.mods = c->d_mods; a.gauss_t = c->d_gauss_t; a.seed = seed;
  a.stream = (uint32_t)stream; a.kind = kind; a.k = c->k; a.n = c->n;
  a.total = (uint64_t)count * c->n * (kind == kSampleUniform ? c->k : 1u);
  const uint64_t blocks = (a.total + kEwThreads - 1) / kEwThreads;
  if (blocks > 0x7fffffffull) return HCNN_ERR_ARG;
  return run<SampleKernel>(c, (size_t)blocks, 0, a);
}
}  // namespace

int hcnn_sample_ternary(hcnn_ctx* c, uint64_t seed, uint64_t stream, int32_t* out, size_t n_polys) {
  return sample_impl(c, kSampleTernary, seed, stream, out, n_polys);
}
int hcnn_sample_gaussian(hcnn_ctx* c, uint64_t seed, uint64_t stream, int32_t* out, size_t n_polys) {
  return sample_impl(c, kSampleGaussian, seed, stream, out, n_polys);
}
int hcnn_sample_uniform(hcnn_ctx* c, uint64_t seed, uint64_t stream, uint32_t* out, size_t n_polys) {
  return sample_impl(c, kSampleUniform, seed, stream, out, n_polys);
}

// ---------------------------------------------------------------- diagnostics
int hcnn_get_stat(hcnn_ctx* c, int which, uint64_t* out) {
  if (!c || !out) return HCNN_ERR_NULL;
  if (which == HCNN_STAT_SCRATCH_BYTES) {
    *out = c->work_bytes + c->small_work_bytes;
    return HCNN_OK;
  }
  if (which == HCNN_STAT_RELIN_FUSED_WGS || which == HCNN_STAT_TENSOR_FUSED_WGS) {
    *out = which == HCNN_STAT_RELIN_FUSED_WGS ? relin_fused_slots(c) : tensor_fused_slots(c);
    return HCNN_OK;
  }
  if (which == HCNN_STAT_TENSOR_FUSED_LEAST) {
    *out = tensor_fused_least(c);
    return HCNN_OK;
  }
  if (which != HCNN_STAT_EXACT_FALLBACKS && which != HCNN_STAT_BAD_INPUT) return HCNN_ERR_ARG;
  unsigned long long v[2] = {0, 0};
  int e = copy_d2h(v, c->d_counters, sizeof(v), c->stream);
  if (e) return e;
  *out = v[which];
  return HCNN_OK;
}

int hcnn_measure_ceiling(hcnn_ctx* c, int which, double* value_out) {
  if (!c || !value_out) return HCNN_ERR_NULL;
  if (which < 0 || which >= HCNN_CEIL_COUNT) return HCNN_ERR_ARG;
  int e;
  double ms = 0.0;
  if (which <= HCNN_CEIL_WRITE) {
    const size_t bytes = (size_t)512 << 20;                                       // per buffer
    const size_t grid = bytes / ((size_t)kRateThreads * kStreamUnroll * 16);
    void* src = nullptr;
    void* dst = nullptr;
    if ((e = dev_malloc(&src, bytes))) return e;
    if ((e = dev_malloc(&dst, bytes))) { dev_free(src); return e; }
    StreamArgs a;
    a.src = (const U4*)src; a.dst = (U4*)dst; a.fill = 0x01010101u;
    a.mode = 2;                                                                  // defined contents for both buffers
    e = launch<StreamKernel>(c->stream, grid, 0, a);
    if (!e) { a.dst = (U4*)src; e = launch<StreamKernel>(c->stream, grid, 0, a); a.dst = (U4*)dst; }
    a.mode = which == HCNN_CEIL_COPY ? 0u : (which == HCNN_CEIL_READ ? 1u : 2u);
    a.fill = 0x5a5a5a5au;                              // read mode: the xor of equal words is 0, never this
    if (!e) e = timed_launches<StreamKernel>(c, grid, a, 9, &ms);
    const int es = stream_sync(c->stream);
    dev_free(src);
    dev_free(dst);
    if (e || es) return e ? e : es;
    // (a build that does not time its launches -- the host emulation -- reports 0)
    *value_out = ms > 0.0 ? (which == HCNN_CEIL_COPY ? 2.0 : 1.0) * (double)bytes / (ms * 1e-3) / 1e9 : 0.0;
    return HCNN_OK;
  }
  void* out = nullptr;
  if ((e = dev_malloc(&out, kRateThreads * 4))) return e;
  RateArgs a;
  a.out = (uint32_t*)out; a.seed = 12345u;
  const size_t grid = (size_t)c->compute_units * 8;          // 8 workgroups of 256 per compute unit: full occupancy
  switch (which) {
    case HCNN_CEIL_MUL_LO: e = timed_launches<RateKernel<kRateMulLo>>(c, grid, a, 5, &ms); break;
    case HCNN_CEIL_MUL_HI: e = timed_launches<RateKernel<kRateMulHi>>(c, grid, a, 5, &ms); break;
    case HCNN_CEIL_MAD_U64: e = timed_launches<RateKernel<kRateMadU64>>(c, grid, a, 5, &ms); break;
    case HCNN_CEIL_MAD_I64: e = timed_launches<RateKernel<kRateMadI64>>(c, grid, a, 5, &ms); break;
    default: e = timed_launches<RateKernel<kRateAdd>>(c, grid, a, 5, &ms); break;
  }
  dev_free(out);
  if (e) return e;
  *value_out = ms > 0.0 ? (double)grid * kRateThreads * kRateIters * kRateChains / (ms * 1e-3) / 1e12 : 0.0;
  return HCNN_OK;
}

int hcnn_profile_read(hcnn_ctx* c, int cls, uint64_t* launches, uint64_t* blocks, double* total_ms) {
  if (!c || !launches || !blocks || !total_ms) return HCNN_ERR_NULL;
  if (cls < 0 || cls >= HCNN_PROF_COUNT) return HCNN_ERR_ARG;
  int e = fold_profile(c);
  if (e) return e;
  *launches = c->prof_launches[cls];
  *blocks = c->prof_blocks[cls];
  *total_ms = c->prof_ms[cls];
  return HCNN_OK;
}

int hcnn_reset_stats(hcnn_ctx* c) {
  if (!c) return HCNN_ERR_NULL;
  int pe = fold_profile(c);
  if (pe) return pe;
  for (int i = 0; i < HCNN_PROF_COUNT; ++i) { c->prof_launches[i] = 0; c->prof_blocks[i] = 0; c->prof_ms[i] = 0.0; }
  return dev_memset(c->d_counters, 0, 2 * sizeof(unsigned long long), c->stream);
}

int hcnn_set_option(hcnn_ctx* c, int which, uint64_t value) {
  if (!c) return HCNN_ERR_NULL;
  switch (which) {
    case HCNN_OPT_AMBIGUITY_BAND:
      // never below the error bound 2*ks of the estimate, at most "always ask the exact comparison"
      if (value < 4ull * HCNN_MAX_LIMBS || value > (1ull << 26)) return HCNN_ERR_ARG;
      c->band = (uint32_t)value;
      return HCNN_OK;
    case HCNN_OPT_SQUARE_CHUNK:
      c->square_chunk = value;
      return HCNN_OK;
    case HCNN_OPT_PROFILE:
      c->profile = value != 0;
      return HCNN_OK;
    case HCNN_OPT_RELIN_ORDER:
      if (value > 2) return HCNN_ERR_ARG;
      c->relin_order = value;
      return HCNN_OK;
    case HCNN_OPT_FUSION:
      if (value > 2) return HCNN_ERR_ARG;
      c->fusion = value;
      return HCNN_OK;
  }
  return HCNN_ERR_ARG;
}

const char* hcnn_strerror(int code) {
  switch (code) {
    case HCNN_OK: return "ok";
    case HCNN_ERR_NULL: return "null pointer";
    case HCNN_ERR_N: return "n must be a power of two in [1024, 32768]";
    case HCNN_ERR_PRIME: return "modulus is not a distinct prime in (2^29, 2^30) congruent to 1 mod 2n";
    case HCNN_ERR_T: return "t must be a prime below 2^47 other than the ciphertext primes (and the plaintext word size must match it)";
    case HCNN_ERR_AUX: return "auxiliary basis missing or too small (need prod p > t*n*q + 1)";
    case HCNN_ERR_ARG: return "invalid count, size or option";
    case HCNN_ERR_NOKEY: return "relinearisation key not set";
    case HCNN_ERR_ALIGN: return "device pointer not 16-byte aligned";
    case HCNN_ERR_NODEVICE: return "no usable device or LDS too small";
    case HCNN_ERR_SCRATCH: return "one ciphertext's intermediate polynomials exceed the 128 MiB static scratch array";
  }
#ifndef HCNN_HOSTEMU
  if (code > 0) return hipGetErrorString((hipError_t)code);
#endif
  return "unknown error";
}

#ifdef HCNN_HOSTEMU
void hcnn_emu_device(uint32_t units, size_t largest_allocation) { emu_units = units; emu_largest = largest_allocation; }
#endif

}  // extern "C"
