// Element-wise and base-conversion kernels of the FV hot path.
//
// All of them are streaming kernels: a thread owns one coefficient position (or
// four consecutive ones) and walks over limbs / terms, so every global access is
// unit-stride across the lanes of a wavefront.
#pragma once
#include "modarith.h"
#include "ntt_kernels.h"

namespace hcnn {

constexpr int kEwThreads = 256;   // threads per workgroup of the element-wise kernels
constexpr int kEwVec = 4;         // coefficients per thread where 16-byte accesses are used
constexpr uint32_t kXcds = 8;     // accelerator dies (each with its own L2); workgroup i runs on die i % 8

// ===================================================================================
// Exact centred base conversion.
//
// Source basis m_0..m_{ks-1} (product M), destination moduli m'_0..m'_{kd-1}.
// For an integer x given by residues x_i, |x| <= (M-1)/2:
//     z_i = [x_i * (M/m_i)^-1]_{m_i},   sum_i z_i * (M/m_i) = x + v*M,
//     v   = round(sum_i z_i / m_i)                      (because |x|/M < 1/2),
//     x mod m'_j = sum_i z_i * [(M/m_i)]_{m'_j} - v * [M]_{m'_j}.
// The tables hold the destination constants centred and with the factor 2^32 of the signed Montgomery reduction, so that
//     out_j = ( sum_i z_i * B[i][j] + v * V[j] (+ caller's extra term) ) * 2^-32 mod m'_j
// is one 64-bit accumulation and one reduction (V = -[M]_{m'}; callers may fold further constant factors into zmul, B
// and V).  A product is below 2^30 * 2^29 in magnitude; the reduction takes 12 of them, a fold (sfold) leaves room for 9 more.
//
// sum_i z_i/m_i is estimated in fixed point with 26 fractional bits: every term
// floor(4 z_i * floor(2^56/m_i) / 2^32) is low by less than 2 units, so the estimate S
// satisfies S <= exact*2^26 < S + 2*ks.  When frac(S/2^31 + 1/2) is within `band`
// units of wrapping the estimate cannot decide the rounding; the decision is then taken
// exactly by comparing the mixed-radix (Garner) digits of the non-negative lift of x
// with those of (M-1)/2.  With the default band (128) that happens for about one
// coefficient in 2^19.
// ===================================================================================
struct alignas(16) BConvDst {
  uint32_t p, pinv;          // m'_j, -m'_j^-1 mod 2^32
  int32_t rc, v;             // 2^32 mod m'_j centred, V[j]
};
struct alignas(16) BConvSrc {
  uint32_t p, pinv;
  int32_t rc, zm;            // zm: zmul_i * 2^32 centred, sredc(x * zm) = x * zmul_i
};
struct BConvDev {
  uint32_t ks, kd;
  const Mod* src_mod;        // [ks]
  const ShoupConst* zmul;    // [ks]   z_i = in_i * zmul_i mod m_i
  const ShoupConst* xmul;    // [ks]   residue of the converted integer = in_i * xmul_i mod m_i
  const uint32_t* ginv;      // [ks][ks] ginv[i*ks + l] = m_l^-1 mod m_i, l < i
  const uint32_t* half;      // [ks]   mixed-radix digits of (M-1)/2
  const BConvDst* dst;       // [kd]
  const int32_t* B;          // [ks][kd]
  const int32_t* BT;         // [kd][ks]  the same constants, transposed
  const BConvSrc* src;       // [ks]   signed form of the source side (intermediate residues of the scaling step)
};
constexpr int kSumRoom = 12, kSumAfterFold = 9;

constexpr uint32_t kFracBits = 26;
constexpr uint32_t kFracOne = 1u << kFracBits;

// Fixed-point estimate of z/m with 26 fractional bits (low by less than 2 units).  The sum of up
// to 32 such terms plus one half stays below 2^32.
HCNN_HD uint32_t frac_est(uint32_t z, const Mod& m) { return mulhi32(z << 2, m.mu >> 5); }

// col[i*stride] holds the residues x_i of a non-negative integer X < M on entry; they are replaced
// by its mixed-radix digits.  Returns 1 when X > (M-1)/2.
HCNN_HD uint32_t garner_gt_half(const BConvDev& bc, uint32_t* col, int stride) {
  for (uint32_t i = 1; i < bc.ks; ++i) {
    const Mod m = ldc(bc.src_mod, i);
    uint32_t t = col[i * stride];
    for (uint32_t l = 0; l < i; ++l) {
      const uint32_t al = reduce32(col[l * stride], m);
      t = sub_mod(t, al, m.p);
      t = mul_mod(t, ldc(bc.ginv, i * bc.ks + l), m);
    }
    col[i * stride] = t;
  }
  for (int i = (int)bc.ks - 1; i >= 0; --i) {
    const uint32_t a = col[i * stride], h = ldc(bc.half, i);
    if (a > h) return 1;
    if (a < h) return 0;
  }
  return 0;
}

// Rounding decision from the estimate S (sum of frac_est terms).  `exact` is called only when the
// estimate is not trustworthy AND the true fraction is near 1/2; it must return 1 when the
// non-negative lift exceeds (M-1)/2.
template <class Exact>
HCNN_HD uint32_t bconv_round(uint32_t S, uint32_t band, Exact exact, unsigned long long* fallback_counter) {
  const uint32_t w = S + (kFracOne >> 1);
  uint32_t v = w >> kFracBits;
  const uint32_t wf = w & (kFracOne - 1);
  if (wf >= kFracOne - band) {
    const uint32_t sf = S & (kFracOne - 1);
    if (sf >= (kFracOne >> 2) && sf < 3u * (kFracOne >> 2)) {   // only then can the estimate be off
      v = (S >> kFracBits) + exact();
      atomic_inc64(fallback_counter);
    }
  }
  return v;
}

// ---- generic (run-time ks, kd) helpers: per-thread columns in LDS -----------------------------
// step(0 .. count - 1); FOURS: four at a time, so that their loads are in flight together (decryptions, us: 10 of 8 primes by halves, n = 8192
// 16.0 / 14.1, 300 of 12 136 / 131, 60 of 16, n = 32768 210 / 200; up to three primes pay for the longer code: 900 of 3, n = 2048 37.4 / 39.4).
template <bool FOURS, class Step>
HCNN_HD void each_prime(uint32_t count, Step step) {
  uint32_t i = 0;
  if constexpr (FOURS) {
    for (; i + 4 <= count; i += 4) {
#pragma unroll
      for (uint32_t j = 0; j < 4; ++j) step(i + j);
    }
  }
  for (; i < count; ++i) step(i);
}
// Computes z_i (stored to zcol) and returns v.  gcol is a second private column for the exact path.
template <bool FOURS = false, class In>
HCNN_HD uint32_t bconv_prepare(const BConvDev& bc, In in, uint32_t* zcol, uint32_t* gcol, int stride,
                               uint32_t band, unsigned long long* fallback_counter) {
  uint32_t S = 0;
  each_prime<FOURS>(bc.ks, [&](uint32_t i) {
    const Mod m = ldc(bc.src_mod, i);
    const uint32_t z = shoup_mul(in(i), ldc(bc.zmul, i), m.p);
    zcol[i * stride] = z;
    S += frac_est(z, m);
  });
  auto exact = [&]() {
    for (uint32_t i = 0; i < bc.ks; ++i) gcol[i * stride] = shoup_mul(in(i), ldc(bc.xmul, i), ldc(bc.src_mod, i).p);
    return garner_gt_half(bc, gcol, stride);
  };
  return bconv_round(S, band, exact, fallback_counter);
}

// Canonical residue of a sum in the form of the tables.
HCNN_HD uint32_t bconv_reduce(int64_t acc, const BConvDst& d) { return canon_p(sredc(sfold(acc, d.rc), d.p, d.pinv), d.p); }
// acc + sum_i z[i] * b[i], folded where the room ends; `used`: products' worth of room that acc takes
// (z: untraced, here and below -- a factor that the compiler knows to be non-negative it extends with zeros, and the signed
// 32 x 32 product is lost to a 64-bit one: three instructions instead of one)
template <int K>
HCNN_HD int64_t bconv_sum(int64_t acc, const int32_t (&z)[K], const int32_t* b, int used, int32_t rc) {
#pragma unroll
  for (int i = 0; i < K; ++i) {
    if (used == kSumRoom) { acc = sfold(acc, rc); used = kSumRoom - kSumAfterFold; }
    acc += (int64_t)z[i] * ldc(b, i);
    ++used;
  }
  return acc;
}

// ---------------------------------------------------------------- q -> q u p extension
// in  [n_ct][2][k][n]  ->  out [n_ct][2][k+kd][n]; rows 0..k-1 are copies, rows k.. are
// the residues of the centred lift modulo the auxiliary primes.
struct ExtArgs {
  const uint32_t* in;
  uint32_t* out;
  BConvDev bc;
  uint32_t n;
  uint32_t band;
  unsigned long long* fallback_counter;
};
// The number of source primes is a compile-time constant (every k is instantiated): z_i stay in VGPRs, every table index is a
// compile-time constant (scalar loads), the LDS column is touched only by the exact path.
template <int K>
struct ExtKernel {
  static constexpr int kThreads = kEwThreads;
  static constexpr int kPhases = 1;
  struct Regs {};
  static size_t lds_bytes() { return (size_t)K * kThreads * 4; }
  template <int PH>
  HCNN_HD static void phase(const ExtArgs& a, unsigned bid, int tid, uint32_t* lds, Regs&) {
    const uint32_t n = a.n;
    const uint32_t blocks_per_poly = n / kThreads;
    const size_t poly = bid / blocks_per_poly;
    const uint32_t c = (bid % blocks_per_poly) * kThreads + tid;
    const uint32_t* src = a.in + poly * K * n + c;
    const uint32_t kp = a.bc.kd;
    uint32_t* dst = a.out + poly * (size_t)(K + kp) * n + c;
    uint32_t x[K];
    int32_t z[K];
    uint32_t S = 0;
#pragma unroll
    for (int i = 0; i < K; ++i) x[i] = src[(size_t)i * n];
#pragma unroll
    for (int i = 0; i < K; ++i) {
      const Mod m = ldc(a.bc.src_mod, i);
      const uint32_t zi = shoup_mul(x[i], ldc(a.bc.zmul, i), m.p);
      S += frac_est(zi, m);
      z[i] = untraced((int32_t)zi);
    }
    auto exact = [&]() {
      uint32_t* col = lds + tid;
#pragma unroll
      for (int i = 0; i < K; ++i) col[i * kThreads] = shoup_mul(x[i], ldc(a.bc.xmul, i), ldc(a.bc.src_mod, i).p);
      return garner_gt_half(a.bc, col, kThreads);
    };
    const int32_t v = untraced((int32_t)bconv_round(S, a.band, exact, a.fallback_counter));
    // (rows 0..K-1 of `out` are not written: the forward transform reads those limbs from the ciphertext itself)
    // rolled loop over the destination primes (three at a time for short bases, whose small launches wait for the tables: one squaring of 8 primes
    // at n = 8192 34.4 / 34.1 us; the compiler does not unroll the like of it in the scaling): row j of the transposed table is one contiguous scalar load
#pragma unroll K <= 8 ? 3 : 1
    for (uint32_t j = 0; j < kp; ++j) {
      const BConvDst d = ldc_at(a.bc.dst + j, 0u);
      dst[(size_t)(K + j) * n] = bconv_reduce(bconv_sum<K>((int64_t)v * d.v, z, a.bc.BT + (size_t)j * K, 1, d.rc), d);
    }
  }
};

// ---------------------------------------------------------------- scale-and-round (HMult step 2)
// d [n_ct][3][k+kp][n] (coefficient domain, integer tensor known mod q and mod p)
//   -> y [n_ct][3][k][n],  y = round(t*d/q) mod q.
// With r = [t*d]_q (centred): y = (t*d - r)/q exactly.  Modulo p_j:
//     y = d'_j * (t q^-1) - sum_i z_i * q_i^-1 + v          (z_i = [t d_i (q/q_i)^-1]_{q_i})
// (table to_p: B = -q_i^-1, V = 1, extra term d'_j * tq_inv_j), then y, which satisfies
// |y| < p/2 by the choice of the auxiliary basis, is converted p -> q (table to_q).
struct ScaleArgs {
  const uint32_t* d;
  uint32_t* y;
  BConvDev to_p;              // src q (zmul = t*(q/q_i)^-1, xmul = t), dst p
  BConvDev to_q;              // src p (zmul = (p/p_j)^-1, xmul = 1), dst q
  const int32_t* tq_inv;      // [kp]  t * q^-1 mod p_j, in the form of the tables
  const NttLimb* limbs;       // [k + kp]
  const SplitRoot* root;      // HALVES: [2][k + kp]
  uint32_t n;
  uint32_t band;
  unsigned long long* fallback_counter;
};
// The number of ciphertext primes is a compile-time constant (see ExtKernel), the loop over the auxiliary primes is rolled:
// y_j is produced, used at once for the p -> q conversion (k running 64-bit sums) and parked in the LDS column for the exact
// path, so the register footprint is 3k + O(1) and the code size does not grow with k*k'.
// Bound: up to k = 8 4.7 TB/s (3 L rows read, 3 k written) at 0.61 of the issue slots, 0.525 us per ciphertext at 64, whose rows still lie in the memory-side cache, and 0.51
// at 1024: neither by itself (one auxiliary row of a thread is in flight); the multiply-adds and reductions beyond.
// HALVES (n = 8192, 32768): d holds rows without the last stage of their inverse transforms (n = 32768, and calls of one or two ciphertexts; n = 8192 keeps
// whole rows otherwise: 720 squarings 1977 us, 1993 by halves; 30 of 16 primes 271, 277).  The stage is one more product of every residue: its
// constants carry the factor that the residue is multiplied with here (z_i directly, or the sum's term of p_j), so that it needs no
// reduction of its own.  A wave takes the same 32 positions of both halves: its two loads of a row are a cache line each.  (The same words read by
// waves of the two halves instead, and the stage by itself with constants picked per lane: 32 ciphertexts, k = 24 530 and 426 us; without the stage 313.)
template <int K, bool HALVES>
struct ScaleKernel {
  static constexpr int kThreads = kEwThreads;
  static constexpr int kPhases = HALVES ? 2 : 1;
  struct Regs {};
  // a column per thread for the exact path, then (HALVES) the constants of both halves
  HCNN_HOSTDEV static uint32_t col_words(uint32_t kp) { return ((uint32_t)K > kp ? (uint32_t)K : kp) * kThreads; }
  static size_t lds_bytes(uint32_t kp) { return (col_words(kp) + (HALVES ? 4 * (K + kp) : 0)) * 4; }
  template <int PH>
  HCNN_HD static void phase(const ScaleArgs& a, unsigned bid, int tid, uint32_t* lds, Regs&) {
    const uint32_t n = a.n, kp = a.to_p.kd;
    const uint32_t L = K + kp;
    uint32_t* const l_root = lds + col_words(kp);
    if constexpr (HALVES && PH == 0) {
      for (uint32_t x = tid; x < 4 * L; x += kThreads) l_root[x] = ld_at(reinterpret_cast<const uint32_t*>(a.root), x * 4);
      return;
    }
    const uint32_t blocks_per_poly = n / kThreads;
    const size_t poly = bid / blocks_per_poly;             // (ct, component)
    const uint32_t half = HALVES ? ((uint32_t)tid >> 5) & 1u : 0;
    const uint32_t c = HALVES ? (bid % blocks_per_poly) * (kThreads / 2) + ((uint32_t)tid >> 6) * 32 + ((uint32_t)tid & 31u)
                              : (bid % blocks_per_poly) * kThreads + tid;
    const uint32_t* src = a.d + poly * (size_t)L * n + c;
    uint32_t* dst = a.y + poly * (size_t)K * n + half * (n / 2) + c;
    uint32_t* col = lds + tid;
    // what lies at this coefficient in row l, and its product with the last stage's constants
    struct Words { uint32_t lo, hi; };
    auto load = [&](uint32_t l) { return Words{src[(size_t)l * n], HALVES ? src[(size_t)l * n + n / 2] : 0u}; };
    auto rooted = [&](const Words& w, uint32_t l) {
      const uint32_t* f = l_root + (half * L + l) * 2;
      return untraced((int64_t)(int32_t)w.lo * (int32_t)f[0]) + (int64_t)(int32_t)w.hi * (int32_t)f[1];
    };
    // the residue itself, canonical up to one prime (the exact path needs it)
    auto residue = [&](uint32_t i) -> uint32_t {
      const Words w = load(i);
      if constexpr (!HALVES) return w.lo;
      const NttLimb m = ldc(a.limbs, i);
      return (uint32_t)split_root((int32_t)w.lo, (int32_t)w.hi, split_root_factors(m.inv_r.c0, m.inv_r.w, half), m.m.p, m.pinv) + m.m.p;
    };

    int32_t z[K];
    uint32_t S = 0;
    {
      Words dq[K];
#pragma unroll
      for (int i = 0; i < K; ++i) dq[i] = load(i);
#pragma unroll
      for (int i = 0; i < K; ++i) {
        const Mod m = ldc(a.to_p.src_mod, i);
        uint32_t zi;
        if constexpr (HALVES) zi = canon_p(sredc(rooted(dq[i], i), m.p, ldc(&a.limbs[i].pinv, 0)), m.p);
        else zi = shoup_mul(dq[i].lo, ldc(a.to_p.zmul, i), m.p);
        S += frac_est(zi, m);
        z[i] = untraced((int32_t)zi);
      }
    }
    auto exact_q = [&]() {
      for (uint32_t i = 0; i < (uint32_t)K; ++i)
        col[i * kThreads] = shoup_mul(residue(i), ldc(a.to_p.xmul, i), ldc(a.to_p.src_mod, i).p);
      return garner_gt_half(a.to_p, col, kThreads);
    };
    const int32_t v = untraced((int32_t)bconv_round(S, a.band, exact_q, a.fallback_counter));

    int64_t out_acc[K];
#pragma unroll
    for (int i = 0; i < K; ++i) out_acc[i] = 0;
    uint32_t S2 = 0, room = kSumRoom;
    Words dp_next = load(K);
#pragma unroll 1
    for (uint32_t j = 0; j < kp; ++j) {
      const Words dpj = dp_next;
      if (j + 1 < kp) dp_next = load(K + j + 1);
      const BConvDst d = ldc_at(a.to_p.dst + j, 0u);
      int64_t first;
      if constexpr (HALVES) first = rooted(dpj, K + j);
      else first = (int64_t)untraced((int32_t)csub(dpj.lo, d.p)) * ldc(a.tq_inv, j);                // arrives in [0, 2p)
      first += (int64_t)v * d.v;
      const int32_t yj = sredc(bconv_sum<K>(first, z, a.to_p.BT + (size_t)j * K, HALVES ? 3 : 2, d.rc), d.p, d.pinv);
      col[j * kThreads] = (uint32_t)yj;                           // made canonical by the exact path if it runs
      const BConvSrc q = ldc_at(a.to_q.src + j, 0u);
      const uint32_t z2 = canon_p(sredc((int64_t)yj * q.zm, q.p, q.pinv), q.p);
      S2 += frac_est(z2, ldc(a.to_q.src_mod, j));
      const int32_t* b2 = a.to_q.B + (size_t)j * K;
      const int32_t zs = untraced((int32_t)z2);
      if (room == 0) {
        room = kSumAfterFold;
#pragma unroll
        for (int i = 0; i < K; ++i) out_acc[i] = sfold(out_acc[i], ldc(a.to_q.dst, i).rc);
      }
      --room;
#pragma unroll
      for (int i = 0; i < K; ++i) out_acc[i] += (int64_t)zs * ldc(b2, i);
    }
    auto exact_p = [&]() {
      for (uint32_t j = 0; j < kp; ++j) {
        const BConvSrc q = ldc_at(a.to_q.src + j, 0u);
        col[j * kThreads] = canon_p(sredc((int64_t)(int32_t)col[j * kThreads] * q.rc, q.p, q.pinv), q.p);
      }
      return garner_gt_half(a.to_q, col, kThreads);
    };
    const int32_t v2 = untraced((int32_t)bconv_round(S2, a.band, exact_p, a.fallback_counter));
#pragma unroll
    for (int i = 0; i < K; ++i) {
      const BConvDst d = ldc_at(a.to_q.dst + i, 0u);
      dst[(size_t)i * n] = bconv_reduce(out_acc[i] + (int64_t)v2 * d.v, d);      // v2 * V < 2^36
    }
  }
};

// ---------------------------------------------------------------- relinearisation inner product
// (the digit reduction and the final addition are fused into the transforms, see ntt_kernels.h)
// acc[ct][b][j] = sum_i evk_hat[i][b][j] * dig_hat[ct][i][j]   (all NTT domain)
struct RelinMacArgs {
  const uint32_t* dig;   // [n_ct][k][k][n]
  const uint32_t* evk;   // [k][2][k][n]
  uint32_t* acc;         // [n_ct][2][k][n]
  const NttLimb* limbs;
  uint32_t k, n;
  uint32_t n_grp;        // groups of CT ciphertexts in this launch
  uint32_t ct_base;      // first ciphertext of the launch
  uint32_t key_major;    // workgroup order, see the kernel
};
// A workgroup takes one (limb j, coefficient tile) for CT consecutive ciphertexts: every evaluation-key tile
// is loaded once and multiplied with the digits of all CT ciphertexts from registers.  (The key is read from
// L2; with one ciphertext per workgroup it makes up two thirds of what flows from L2 into the compute units,
// and that flow, not HBM, then bounds the kernel.)
HCNN_HD int64_t mul_s32(uint32_t a, uint32_t b) { return (int64_t)(int32_t)a * (int32_t)b; }
template <int CT>
struct RelinMacKernel {
  static constexpr int kThreads = kEwThreads;
  static constexpr int kPhases = 1;
  struct Regs {};
  template <int PH>
  HCNN_HD static void phase(const RelinMacArgs& a, unsigned bid, int tid, uint32_t*, Regs&) {
    const uint32_t per_row = a.n / (kThreads * kEwVec);
    size_t grp;
    uint32_t j, tile;
    if (a.key_major) {
      // (chosen by the host when the evaluation key outgrows an L2 in the plain order)
      // die x takes the coefficient tiles x, x+8, ... ; for one (limb, tile) it sweeps the ciphertexts of
      // the batch back to back, so the 2k evaluation-key tiles they all multiply with stay in that die's L2
      const uint32_t xcd = bid % kXcds, local = bid / kXcds;
      grp = local % a.n_grp;
      const uint32_t rest = local / a.n_grp;
      tile = (rest % (per_row / kXcds)) * kXcds + xcd;
      j = rest / (per_row / kXcds);
    } else {
      const size_t row = bid / per_row;                     // (group, j)
      tile = bid % per_row;
      grp = row / a.k;
      j = (uint32_t)(row % a.k);
    }
    const size_t ct0 = a.ct_base + grp * CT;
    const uint32_t c = (tile * kThreads + tid) * kEwVec;
    const NttLimb L = ldc(a.limbs, j);
    const size_t rn = a.n;
    // signed digits in [-p, p), centred key values: 16 products stay below 8 p^2 < 2^63, 13 after a fold (whose result takes
    // the room of two).  The loads of two digits are issued before the first product: left to the scheduler, which saves
    // registers, every load was waited for by itself (squaring of 4 ciphertexts at n = 8192, k = 8 57.6 / 49.8 us, of 16 at n = 2048,
    // k = 4 36.2 / 33.1)
    int64_t s0[CT][4], s1[CT][4];
#pragma unroll
    for (int t = 0; t < CT; ++t)
      for (int q = 0; q < 4; ++q) { s0[t][q] = 0; s1[t][q] = 0; }
    for (uint32_t i0 = 0, run = 16; i0 < a.k; i0 += run, run = 13) {
      if (i0 > 0) {
#pragma unroll
        for (int t = 0; t < CT; ++t)
          for (int q = 0; q < 4; ++q) { s0[t][q] = sfold(s0[t][q], L.rc); s1[t][q] = sfold(s1[t][q], L.rc); }
      }
      const uint32_t i1 = i0 + run < a.k ? i0 + run : a.k;
      auto load = [&](uint32_t i, U4& e0, U4& e1, U4 (&d)[CT]) {
        e0 = *reinterpret_cast<const U4*>(a.evk + (((size_t)i * 2 + 0) * a.k + j) * rn + c);
        e1 = *reinterpret_cast<const U4*>(a.evk + (((size_t)i * 2 + 1) * a.k + j) * rn + c);
#pragma unroll
        for (int t = 0; t < CT; ++t)
          d[t] = *reinterpret_cast<const U4*>(a.dig + (((ct0 + t) * a.k + i) * a.k + j) * rn + c);
      };
      auto multiply = [&](const U4& E0, const U4& E1, const U4 (&D)[CT]) {
#pragma unroll
        for (int t = 0; t < CT; ++t) {
          s0[t][0] += mul_s32(D[t].x, E0.x); s0[t][1] += mul_s32(D[t].y, E0.y);
          s0[t][2] += mul_s32(D[t].z, E0.z); s0[t][3] += mul_s32(D[t].w, E0.w);
          s1[t][0] += mul_s32(D[t].x, E1.x); s1[t][1] += mul_s32(D[t].y, E1.y);
          s1[t][2] += mul_s32(D[t].z, E1.z); s1[t][3] += mul_s32(D[t].w, E1.w);
        }
      };
      U4 e[2][2], d[2][CT];
      uint32_t i = i0;
      for (; i + 2 <= i1; i += 2) {
        load(i, e[0][0], e[0][1], d[0]);
        load(i + 1, e[1][0], e[1][1], d[1]);
        sched_fence();
        multiply(e[0][0], e[0][1], d[0]);
        multiply(e[1][0], e[1][1], d[1]);
      }
      if (i < i1) {
        load(i, e[0][0], e[0][1], d[0]);
        sched_fence();
        multiply(e[0][0], e[0][1], d[0]);
      }
    }
    // (the sums are left signed in (-p, p): the inverse transform that reads them takes them as they are)
    auto out = [&](int64_t s) { return (uint32_t)sredc(sfold(s, L.rc), L.m.p, L.pinv); };
#pragma unroll
    for (int t = 0; t < CT; ++t) {
      U4 r0, r1;
      r0.x = out(s0[t][0]); r0.y = out(s0[t][1]); r0.z = out(s0[t][2]); r0.w = out(s0[t][3]);
      r1.x = out(s1[t][0]); r1.y = out(s1[t][1]); r1.z = out(s1[t][2]); r1.w = out(s1[t][3]);
      *reinterpret_cast<U4*>(a.acc + (((ct0 + t) * 2 + 0) * a.k + j) * rn + c) = r0;
      *reinterpret_cast<U4*>(a.acc + (((ct0 + t) * 2 + 1) * a.k + j) * rn + c) = r1;
    }
  }
};

// ---------------------------------------------------------------- shared-basis relinearisation
// The inner product over the integers instead of modulo every q_j, for two primes of the ciphertext at a time: digits are below 2^30
// and key coefficients modulo q_j q_j' within 0.63 * 2^60 of zero (RelinPair), so sum_i D_i * key[i] is below k n 0.63 * 2^90 <= 2^109.4 in magnitude
// and four auxiliary primes (product above 2^116) hold it.  4k digit transforms and 4k inverse ones replace k^2 and 2k; the
// inner product has twice the terms:
//   acc[ct][o][r] = sum_i dig[ct][i][r] * key[i][o][r],   o = (b, pair) of 2 ceil(k/2), r < 4      (NTT domain, modulo p_r)
// (Every q_j by itself takes three primes, 3k and 6k transforms and three times the terms; three at a time five, 5k + 10k/3 and 5/3.  Us, one q_j / two
// at a time: n = 16384, k = 16, 225 squarings 3430 / 3195, of it digits 280 / 385, key product 714 / 502, back 818 / 648; n = 32768, k = 24,
// 32 2107 / 1912: 150 / 200, 361 / 215, back rows and combination 559 / 385.)
// A workgroup takes 64 coefficients of one r for CT ciphertexts: their digits go to LDS once, its eight waves share out
// the outputs (O each) and load every key word once for the CT ciphertexts.
struct RelinSharedArgs {
  const uint32_t* dig;   // [n_ct][4][n/64][k][64], signed in [-p, p)
  const uint32_t* key;   // [4][n/64][k][outs][64], as kNttStoreKey leaves it
  uint32_t* acc;         // [n_ct][4][n/64][outs][64], signed in (-p, p)
  const NttLimb* limbs;  // of the four primes
  uint32_t k, outs, n, n_ct, n_grp;
};
template <int O>
struct RelinSharedMac {
  static constexpr int kThreads = 512;
  static constexpr int kPhases = 2;
  static constexpr int kMinWavesPerSimd = 4;
  // The key words of the next digit are on their way while one is multiplied: left to the compiler, the loop waits for its loads (measured with
  // three primes, us: n = 32768, k = 24, 32 ciphertexts 395 / 347; n = 16384, k = 16, 225 704 / 683; more digits ahead were slower).
  // Bound: digits read and sums written (n = 16384, k = 16, 225 ciphertexts 502 us, 397 by bytes; 16 ciphertexts a workgroup 600).
  static constexpr int CT = 8;
  struct Regs {};
  static size_t lds_bytes(uint32_t k) { return (size_t)CT * k * 64 * 4; }
  template <int PH>
  HCNN_HD static void phase(const RelinSharedArgs& a, unsigned bid, int tid, uint32_t* lds, Regs&) {
    // the ciphertext groups of one (r, tile) follow each other on one die: its key words stay in that L2
    const uint32_t xcd = bid % kXcds, local = bid / kXcds;
    const uint32_t grp = local % a.n_grp, unit = local / a.n_grp * kXcds + xcd;
    const uint32_t tiles = a.n / 64, r = unit / tiles, tile = unit % tiles;
    const uint32_t wave = wave_uniform((uint32_t)tid / 64), lane = (uint32_t)tid % 64;
    const uint32_t ct0 = grp * CT;
    if constexpr (PH == 0) {
      const uint32_t words = a.k * 16;                // 16-byte words of one ciphertext's tile
      for (uint32_t x = tid; x < CT * words; x += kThreads) {
        const uint32_t t = x / words, ct = ct0 + t < a.n_ct ? ct0 + t : a.n_ct - 1;
        reinterpret_cast<U4*>(lds)[x] =
            *reinterpret_cast<const U4*>(a.dig + (((size_t)ct * kSharedPrimes + r) * tiles + tile) * a.k * 64 + (x - t * words) * 4);
      }
    } else {
      const uint32_t o0 = wave * O, outs = a.outs;
      if (o0 >= outs) return;
      const NttLimb L = ldc(a.limbs, r);
      const uint32_t* key = a.key + ((size_t)r * tiles + tile) * a.k * outs * 64;
      int64_t s[CT][O];
#pragma unroll
      for (int t = 0; t < CT; ++t)
#pragma unroll
        for (int o = 0; o < O; ++o) s[t][o] = 0;
      // (fold rule of RelinMacKernel)
      for (uint32_t i0 = 0, run = 16; i0 < a.k; i0 += run, run = 13) {
        if (i0 > 0) {
#pragma unroll
          for (int t = 0; t < CT; ++t)
#pragma unroll
            for (int o = 0; o < O; ++o) s[t][o] = sfold(s[t][o], L.rc);
        }
        const uint32_t i1 = i0 + run < a.k ? i0 + run : a.k;
        auto load = [&](uint32_t i, int32_t (&e)[O]) {
          const uint32_t ii = i < i1 ? i : i1 - 1;
#pragma unroll
          for (int o = 0; o < O; ++o) {
            const uint32_t oo = o0 + o < outs ? o0 + o : outs - 1;
            e[o] = (int32_t)ld_at(key + ((size_t)ii * outs + oo) * 64, lane * 4);
          }
        };
        auto multiply = [&](uint32_t i, const int32_t (&e)[O]) {
#pragma unroll
          for (int t = 0; t < CT; ++t) {
            const int32_t d = (int32_t)lds[(t * a.k + i) * 64 + lane];
#pragma unroll
            for (int o = 0; o < O; ++o) s[t][o] += (int64_t)d * e[o];
          }
        };
        int32_t e[2][O];
        load(i0, e[0]);
        sched_fence();
        for (uint32_t i = i0; i < i1; i += 2) {
          load(i + 1, e[1]);
          sched_fence();
          multiply(i, e[0]);
          if (i + 1 >= i1) break;
          load(i + 2, e[0]);
          sched_fence();
          multiply(i + 1, e[1]);
        }
      }
#pragma unroll
      for (int t = 0; t < CT; ++t) {
        if (ct0 + t >= a.n_ct) break;
#pragma unroll
        for (int o = 0; o < O; ++o)
          if (o0 + o < outs)
            st_at(a.acc + ((((size_t)(ct0 + t) * kSharedPrimes + r) * tiles + tile) * outs + o0 + o) * 64, lane * 4,
                  (uint32_t)sredc(sfold(s[t][o], L.rc), L.m.p, L.pinv));
      }
    }
  }
};

// Largest ring: the four rows of an output, left at the last stage of their inverse transforms (kNttBackRow), through that stage, to modulo
// the pair's primes, plus y_b.  A thread takes four coefficients of each half.
struct RelinCombineArgs {
  const uint32_t* z;     // [n_ct][outs][4][n], dense rows
  const uint32_t* y;     // [n_ct][3][k][n]
  uint32_t* out;         // [n_ct][2][k][n]
  const NttLimb* limbs;
  const RelinCrt* crt;   // [k]
  RelinCrtInv crt_inv;
  FastDiv outputs;       // (b, pair)
  uint32_t k, n;
};
struct RelinCombine {
  static constexpr int kPer = 4;                 // coefficients of each half
  static constexpr int kThreads = kEwThreads;
  static constexpr int kPhases = 1;
  struct Regs {};
  template <int PH>
  HCNN_HD static void phase(const RelinCombineArgs& a, unsigned bid, int tid, uint32_t*, Regs&) {
    const uint32_t per_row = a.n / (kThreads * kPer * 2);
    const uint32_t row = bid / per_row, c = (bid % per_row * kThreads + tid) * kPer, h2 = a.n / 2;
    const uint32_t ct = quot(row, a.outputs), o = row - ct * a.outputs.d;
    const uint32_t b = o >= a.outputs.d / 2 ? 1u : 0u, j0 = 2 * (o - b * (a.outputs.d / 2));
    const uint32_t* zp = a.z + (size_t)row * kSharedPrimes * a.n;
    U4 lo[kSharedPrimes], hi[kSharedPrimes];
#pragma unroll
    for (uint32_t r = 0; r < kSharedPrimes; ++r) {
      lo[r] = ld4_at(zp + (size_t)r * a.n, c * 4);
      hi[r] = ld4_at(zp + (size_t)r * a.n + h2, c * 4);
    }
    int32_t z[2][kPer][kSharedPrimes];
#pragma unroll
    for (uint32_t r = 0; r < kSharedPrimes; ++r) {
      const NttLimb* lb = a.limbs + a.k + r;
      const InvRoot top = ldc(&lb->inv_z, 0);
      const uint32_t p = ldc(&lb->m.p, 0), pinv = ldc(&lb->pinv, 0);
      const int32_t x[kPer] = {(int32_t)lo[r].x, (int32_t)lo[r].y, (int32_t)lo[r].z, (int32_t)lo[r].w};
      const int32_t y[kPer] = {(int32_t)hi[r].x, (int32_t)hi[r].y, (int32_t)hi[r].z, (int32_t)hi[r].w};
#pragma unroll
      for (uint32_t h = 0; h < 2; ++h)
#pragma unroll
        for (int e = 0; e < kPer; ++e) z[h][e][r] = split_root(x[e], y[e], split_root_factors(top.c0, top.w, h), p, pinv);
    }
#pragma unroll
    for (uint32_t h = 0; h < 2; ++h) {
      int32_t v[kPer];
#pragma unroll
      for (int e = 0; e < kPer; ++e) v[e] = relin_crt_round(z[h][e], a.crt_inv);
#pragma unroll
      for (uint32_t s = 0; s < 2; ++s) {
        const uint32_t j = j0 + s;
        if (j >= a.k) break;
        const NttLimb L = ldc(a.limbs, j);
        const RelinCrt kc = ldc(a.crt, j);
        const U4 y = ld4_at(a.y + ((size_t)(ct * 3 + b) * a.k + j) * a.n + h * h2, c * 4);
        auto one = [&](int e, uint32_t add) { return add_mod(relin_crt(z[h][e], v[e], kc, L.m.p, L.pinv), add, L.m.p); };
        U4 r;
        r.x = one(0, y.x); r.y = one(1, y.y); r.z = one(2, y.z); r.w = one(3, y.w);
        st4_at(a.out + ((size_t)(ct * 2 + b) * a.k + j) * a.n + h * h2, c * 4, r);
      }
    }
  }
};

// ---------------------------------------------------------------- scalar multiply-accumulate
// out[f][g] = sum_tau w[g][f][tau] * in[idx[g][tau]]  per residue (HMultPlain by an integer + HAdd).
struct MacArgs {
  const uint32_t* in;     // [n_in][2][k][n]
  const uint32_t* idx;    // [G][T]
  const int32_t* w;       // [G][F][T]
  uint32_t* out;          // [F][G][2][k][n]
  const Mod* mods;        // [k]
  const NttLimb* limbs;   // [k]
  uint32_t k, n;
  uint32_t n_in, G, F, T;
  int32_t w_abs_max;
  uint32_t chunk;         // terms between reductions of the signed 64-bit accumulators
  uint32_t steps;         // matrix forms: tiles per wave
  uint32_t pack;          // MacPack: groups that share the sixteen rows
  FastDiv terms, filters; // unions: T, F
  unsigned long long* bad_counter;
};
// Fallback for gather rows too long to stage in LDS: indices and weights are read from global
// memory inside the term loop.
template <int FT>
struct MacKernelDirect {
  static constexpr int kThreads = kEwThreads;
  static constexpr int kPhases = 1;
  struct Regs {};
  HCNN_HD static int64_t fold(int64_t s, const Mod& m) {
    const uint64_t mag = s < 0 ? (uint64_t)(-s) : (uint64_t)s;
    const uint32_t r = reduce64(mag, m);
    return (s < 0 && r != 0) ? (int64_t)(m.p - r) : (int64_t)r;
  }
  template <int PH>
  HCNN_HD static void phase(const MacArgs& a, unsigned bid, int tid, uint32_t*, Regs&) {
    const uint32_t ct_words32 = 2u * a.k * a.n;                       // at most 2^22
    const size_t ct_words = ct_words32;
    const uint32_t tiles = ct_words32 / (kThreads * kEwVec);
    const uint32_t g = bid / tiles;
    const uint32_t tile = bid % tiles;
    const uint32_t pos = (tile * kThreads + tid) * kEwVec;            // word offset inside a ciphertext
    const uint32_t row = tile / (a.n / (kThreads * kEwVec));          // (poly, limb) row; uniform in the block
    const uint32_t limb = row % a.k;
    const Mod m = ldc(a.mods, limb);
    const uint32_t* idx = a.idx + (size_t)g * a.T;
    const int32_t* w = a.w + (size_t)g * a.F * a.T;
    int64_t s[FT][4];
#pragma unroll
    for (int f = 0; f < FT; ++f) { s[f][0] = 0; s[f][1] = 0; s[f][2] = 0; s[f][3] = 0; }
    uint32_t since = 0;
    for (uint32_t tau = 0; tau < a.T; ++tau) {
      const uint32_t src = idx[tau];
      if (src >= a.n_in) {
        if (tid == 0 && tile == 0) atomic_inc64(a.bad_counter);
        continue;
      }
      const U4 x = *reinterpret_cast<const U4*>(a.in + (size_t)src * ct_words + pos);
#pragma unroll
      for (int f = 0; f < FT; ++f) {
        int32_t wf = w[(size_t)f * a.T + tau];
        if (wf > a.w_abs_max || wf < -a.w_abs_max) {
          if (tid == 0 && tile == 0) atomic_inc64(a.bad_counter);
          wf = 0;
        }
        // residues are below 2^30, so they are valid signed 32-bit operands: one 32x32+64 multiply-add each
        s[f][0] += (int64_t)wf * (int64_t)(int32_t)x.x;
        s[f][1] += (int64_t)wf * (int64_t)(int32_t)x.y;
        s[f][2] += (int64_t)wf * (int64_t)(int32_t)x.z;
        s[f][3] += (int64_t)wf * (int64_t)(int32_t)x.w;
      }
      if (++since == a.chunk) {
        since = 0;
#pragma unroll
        for (int f = 0; f < FT; ++f)
          for (int q = 0; q < 4; ++q) s[f][q] = fold(s[f][q], m);
      }
    }
#pragma unroll
    for (int f = 0; f < FT; ++f) {
      U4 r;
      r.x = (uint32_t)fold(s[f][0], m); r.y = (uint32_t)fold(s[f][1], m);
      r.z = (uint32_t)fold(s[f][2], m); r.w = (uint32_t)fold(s[f][3], m);
      *reinterpret_cast<U4*>(a.out + ((size_t)f * a.G + g) * ct_words + pos) = r;
    }
  }
};

// Main variant: the gather row and the F*T weights of the group are staged in LDS once per
// workgroup (validated while staging: a bad index or weight becomes a zero-weight term on input 0;
// the row is padded to a multiple of kMacBatch with zero-weight terms on its last input), so the
// term loop reads them with broadcast LDS reads and carries no data-dependent branches.  Inputs are fetched kMacBatch terms
// ahead of their use (double buffering in registers) to keep HBM requests in flight during the
// multiply-adds.  Requires chunk % kMacBatch == 0.
// SKIP: the multiply-adds of the padding terms are skipped (a branch in the term loop, uniform over the workgroup).
// Measured: 6 % faster at 8 filters x 27 terms, nothing at 5 x 25, 14 % slower at 16 filters and hundreds of
// terms (where nothing is padded); the host picks the form by filter count and row length.
constexpr uint32_t kMacBatch = 4;
template <int FT, bool SKIP = false>
struct MacKernel {
  static constexpr int kThreads = kEwThreads;
  static constexpr int kPhases = 2;
  struct Regs {};
  static size_t padded_terms(size_t T) { return (T + kMacBatch - 1) / kMacBatch * kMacBatch; }
  static size_t lds_bytes(size_t F, size_t T) { return ((1 + F) * padded_terms(T) + 2 * kMacBatch) * 4; }
  static size_t grid(size_t tiles, size_t G) { return kXcds * ((tiles + kXcds - 1) / kXcds) * G; }
  template <int PH>
  HCNN_HD static void phase(const MacArgs& a, unsigned bid, int tid, uint32_t* lds, Regs&) {
    const uint32_t ct_words32 = 2u * a.k * a.n;                       // at most 2^22
    const size_t ct_words = ct_words32;
    const uint32_t tiles = ct_words32 / (kThreads * kEwVec);
    // Workgroups go to the 8 XCDs round-robin by index, and each XCD has its own L2.  XCD x sweeps
    // the coefficient tiles x, x+8, ... and, inside a tile, the groups in order: the blocks that are
    // resident on one XCD at a time then share their gather rows' inputs (neighbouring filter
    // placements overlap), so every input tile is fetched from HBM about once.
    const uint32_t xcd = bid % kXcds, local = bid / kXcds;
    const uint32_t tile = (local / a.G) * kXcds + xcd;
    const uint32_t g = local % a.G;
    if (tile >= tiles) return;                                        // padding blocks (whole block)
    const uint32_t Tpad = (a.T + kMacBatch - 1) / kMacBatch * kMacBatch;
    uint32_t* l_idx = lds;                                            // [Tpad + 2*kMacBatch]
    int32_t* l_w = reinterpret_cast<int32_t*>(lds + Tpad + 2 * kMacBatch);   // [F][Tpad]
    if constexpr (PH == 0) {
      const uint32_t* idx = a.idx + (size_t)g * a.T;
      const int32_t* w = a.w + (size_t)g * a.F * a.T;
      for (uint32_t tau = tid; tau < Tpad + 2 * kMacBatch; tau += kThreads) {
        // the padding terms and the read-ahead slots of the last batches fetch the row's last input once more
        // (the compute unit's cache has just seen it); padding terms carry weight zero, read-ahead slots are never
        // consumed
        const bool pad = tau >= a.T;
        uint32_t src = idx[pad ? a.T - 1 : tau];
        const bool bad_src = src >= a.n_in;
        if (bad_src) {
          src = 0;
          if (tile == 0 && !pad) atomic_inc64(a.bad_counter);
        }
        l_idx[tau] = src * (ct_words32 / 4);   // offset of the input in 16-byte units (the host checked that it fits)
        if (tau >= Tpad) continue;
#pragma unroll
        for (int f = 0; f < FT; ++f) {
          int32_t wf = pad ? 0 : w[(size_t)f * a.T + tau];
          if (wf > a.w_abs_max || wf < -a.w_abs_max) {
            wf = 0;
            if (tile == 0) atomic_inc64(a.bad_counter);
          }
          l_w[(size_t)f * Tpad + tau] = bad_src ? 0 : wf;
        }
      }
    } else {
      const uint32_t pos = (tile * kThreads + tid) * kEwVec;          // word offset inside a ciphertext
      const uint32_t row = tile / (a.n / (kThreads * kEwVec));        // (poly, limb) row; uniform in the block
      const Mod m = ldc(a.mods, row % a.k);
      const U4* in = reinterpret_cast<const U4*>(a.in + pos);
      // accumulators carry the bias p*2^33 (a multiple of p above 2^62), so they stay positive while
      // the signed partial sums stay inside (-2^62, 2^62) and one unsigned reduction folds them
      const uint64_t bias = (uint64_t)m.p << 33;
      uint64_t s[FT][4];
#pragma unroll
      for (int f = 0; f < FT; ++f) { s[f][0] = bias; s[f][1] = bias; s[f][2] = bias; s[f][3] = bias; }
      auto fetch = [&](U4 (&buf)[kMacBatch], uint32_t t) {
#pragma unroll
        for (uint32_t b = 0; b < kMacBatch; ++b)
          buf[b] = in[(size_t)l_idx[t + b]];
      };
      auto consume = [&](const U4 (&buf)[kMacBatch], uint32_t t) {
#pragma unroll
        for (uint32_t b = 0; b < kMacBatch; ++b) {
          if constexpr (SKIP) {
            if (t + b >= a.T) break;            // padding terms of the last batch
          }
#pragma unroll
          for (int f = 0; f < FT; ++f) {
            const int64_t wf = l_w[(size_t)f * Tpad + t + b];
            // residues are below 2^30, so they are valid signed 32-bit operands: one 32x32+64 multiply-add each
            s[f][0] += (uint64_t)(wf * (int64_t)(int32_t)buf[b].x);
            s[f][1] += (uint64_t)(wf * (int64_t)(int32_t)buf[b].y);
            s[f][2] += (uint64_t)(wf * (int64_t)(int32_t)buf[b].z);
            s[f][3] += (uint64_t)(wf * (int64_t)(int32_t)buf[b].w);
          }
        }
      };
      auto refold = [&]() {
#pragma unroll
        for (int f = 0; f < FT; ++f)
          for (int q = 0; q < 4; ++q) s[f][q] = bias + reduce64(s[f][q], m);
      };
      // two register buffers used alternately: the loads of the next batch are in flight while the
      // current one is consumed.  Every fetch is unconditional (the gather row is followed by 2*kMacBatch
      // entries that name its last input again) so that the number of loads in flight is the same on every path
      // and the compiler can wait for exactly the older batch.
      U4 buf_a[kMacBatch], buf_b[kMacBatch];
      fetch(buf_a, 0);
      uint32_t since = 0;
      for (uint32_t tau = 0; tau < Tpad; tau += 2 * kMacBatch) {
        fetch(buf_b, tau + kMacBatch);
        if (since >= a.chunk) { since = 0; refold(); }
        since += kMacBatch;
        consume(buf_a, tau);
        fetch(buf_a, tau + 2 * kMacBatch);
        if (tau + kMacBatch < Tpad) {
          if (since >= a.chunk) { since = 0; refold(); }
          since += kMacBatch;
          consume(buf_b, tau + kMacBatch);
        }
      }
#pragma unroll
      for (int f = 0; f < FT; ++f) {
        U4 r;
        r.x = reduce64(s[f][0], m); r.y = reduce64(s[f][1], m);
        r.z = reduce64(s[f][2], m); r.w = reduce64(s[f][3], m);
        *reinterpret_cast<U4*>(a.out + ((size_t)f * a.G + g) * ct_words + pos) = r;
      }
    }
  }
};

// Many filters: the sums as matrix products on the byte planes of the residues (v_mfma_i32_16x16x64_i8).
// With F filters every gathered residue feeds F multiply-adds; at 16 filters the kernel above is bound by their rate (576 terms:
// 28 T multiply-adds/s of 34).  Here a residue is split into four bytes; a matrix instruction multiplies 16 filters x 64 terms
// of 8-bit weights with 64 terms x 16 coefficients of one byte plane, and the vector unit is left with the 4 x 4 byte
// transposition that brings four terms of a coefficient into one operand word (8 v_perm_b32 per four residues) and with
// the recombination of the four 32-bit sums of an output.
//   wave            one group g, tiles of 64 consecutive coefficients; a lane holds 4 of them (one 16-byte load per term)
//   lane            lg = lane / 16, ln = lane % 16: coefficients 4 ln .. 4 ln + 3; of every 16 terms those 4 lg .. 4 lg + 3
//   operand word    quad step q of a chunk of 64 terms: terms 16 q + 4 lg .. + 3 of filter ln (weights) or of coefficient
//                   4 ln + s (data, s = 0..3); weights and data use the same order of terms
//   result          sums of filters 4 lg .. 4 lg + 3 at coefficient 4 ln + s
// Bytes 0..2 of a residue are taken less 128 (byte 3 is below 64); the sums start at 128 * (sum of the weights) instead of 0.
// The GB groups of a workgroup are neighbours (kernel placements that share most of their inputs): their waves run through
// the terms together and find each other's inputs in the compute unit's cache.  The XCD order of the tiles is that of MacKernel.
// A term row is padded to a multiple of 16 with zero-weight terms on its last input.
// Two groups, not four: a last workgroup of 4 is up to three quarters empty, and a launch of few groups stages twice the tables per
// tile (us, four / two groups per workgroup: 16 filters x 576 terms, 64 groups, n = 8192, k = 10 1676 / 1548; 10 x 576, 9 groups
// 395 / 347; 10 x 96, 8 groups, n = 4096, k = 4 21 / 15).  Where its workgroups have enough to do, MacPair takes the pairs.
// Bound: the gather.  576 terms x 16 filters over 64 groups at n = 8192, k = 10: vector form 3.40 ms, this one 1.50, 24 GB gathered at
// 32 bytes per clock and compute unit (18 GB of it from L2), vector unit 55 % used, matrix unit 12 %.  Measured and left out: a second register
// buffer of inputs (spills: a third slower); the waves kept in step by a barrier per chunk (L2 requests halved, no faster: the
// waits it adds cost what it saves); eight groups on eight waves.
constexpr uint32_t kMfmaMaxSum = 1u << 20;     // T * |w| <= 2^20: sums of weight * byte stay below 2^28, and 4 * 2^28 * p/2
                                               // leaves the Montgomery step within (-p, p)
// What the two kernels below share: the sums of one tile for NG groups over one list of terms.
struct MacMatrix {
  static constexpr uint32_t kTile = 64;
  static constexpr uint32_t kLeastPerUnit = 4;     // workgroups per compute unit below which waves take fewer tiles (mac_matrix_steps)
  HCNN_HOSTDEV static uint32_t chunks(uint32_t T) { return (T + 63) / 64; }
  // workgroups of a launch: every die takes the same number of tile blocks (the last ones may be empty), each for all blocks of groups
  static size_t grid(uint32_t tile_blocks, size_t group_blocks) { return (size_t)kXcds * ((tile_blocks + kXcds - 1) / kXcds) * group_blocks; }

#if defined(HCNN_HOSTEMU)
  // The checker runs lane by lane: every lane forms its own 4 filters x 4 coefficients from the staged tables.
  struct Sums { int32_t v[4] = {0, 0, 0, 0}; };
  static int32_t weight(const uint32_t* l_w, uint32_t f, uint32_t t) {          // term t of a chunk
    return (int8_t)(l_w[((t / 4 % 4 * 16 + f) * 4) + t / 16] >> (8 * (t % 4)));
  }
  static void weight_sums(const uint32_t* l_w, uint32_t n_chunks, uint32_t lane, Sums& out) {
    for (int r = 0; r < 4; ++r)
      for (uint32_t t = 0; t < n_chunks * 64; ++t) out.v[r] += 128 * weight(l_w + t / 64 * 256, lane / 16 * 4 + r, t % 64);
  }
  template <int Q> struct Inputs { const uint32_t *in, *l_off; uint32_t unit; };
  template <bool WIDE, int Q>
  static void load(const uint32_t* in, const uint32_t* l_off, uint32_t lane, Inputs<Q>& x, uint32_t) { x = Inputs<Q>{in + lane % 16 * 4, l_off, WIDE ? 16u : 1u}; }
  static void multiply_half(const Inputs<2>& half, const uint32_t* l_w, uint32_t h, uint32_t lane, Sums (&acc)[4][4]) {
    for (uint32_t t = 0; t < 32; ++t)
      for (int s = 0; s < 4; ++s) {
        const uint32_t x = half.in[(size_t)half.l_off[t] * half.unit / 4 + s];
        for (int r = 0; r < 4; ++r)
          for (int j = 0; j < 4; ++j)
            acc[s][j].v[r] += weight(l_w, lane / 16 * 4 + r, 32 * h + t) * ((int32_t)(x >> (8 * j) & 0xff) - (j < 3 ? 128 : 0));
      }
  }
  template <int Q, int NG>
  static void multiply(const Inputs<Q>& chunk, const uint32_t* l_w, uint32_t w_stride, uint32_t lane, Sums (&acc)[NG][4][4]) {
    const uint32_t *in = chunk.in, *l_off = chunk.l_off;
    for (uint32_t t = 0; t < 16 * Q; ++t)
      for (int s = 0; s < 4; ++s) {
        const uint32_t x = in[(size_t)l_off[t] * chunk.unit / 4 + s];
        for (int g = 0; g < NG; ++g)
          for (int r = 0; r < 4; ++r)
            for (int j = 0; j < 4; ++j)
              acc[g][s][j].v[r] += weight(l_w + g * w_stride, lane / 16 * 4 + r, t) * ((int32_t)(x >> (8 * j) & 0xff) - (j < 3 ? 128 : 0));
      }
  }
#elif !defined(__HIP_DEVICE_COMPILE__)
  // (the host pass of the device build only parses the callers)
  struct Sums { int32_t v[4] = {0, 0, 0, 0}; };
  __device__ static void weight_sums(const uint32_t*, uint32_t, uint32_t, Sums&);
  template <int Q> struct Inputs {};
  template <bool WIDE, int Q> __device__ static void load(const uint32_t*, const uint32_t*, uint32_t, Inputs<Q>&, uint32_t);
  template <int Q, int NG> __device__ static void multiply(const Inputs<Q>&, const uint32_t*, uint32_t, uint32_t, Sums (&)[NG][4][4]);
  __device__ static void multiply_half(const Inputs<2>&, const uint32_t*, uint32_t, uint32_t, Sums (&)[4][4]);
#else
  typedef int32_t Vec __attribute__((ext_vector_type(4)));
  struct Sums { Vec v = {0, 0, 0, 0}; };
  __device__ __forceinline__ static void weight_sums(const uint32_t* l_w, uint32_t n_chunks, uint32_t lane, Sums& out) {
    const Vec ones = {0x01010101, 0x01010101, 0x01010101, 0x01010101};
    for (uint32_t c = 0; c < n_chunks; ++c)
      out.v = __builtin_amdgcn_mfma_i32_16x16x64_i8(reinterpret_cast<const Vec*>(l_w + c * 256)[lane], ones, out.v, 0, 0, 0);
    out.v *= 128;
  }
  // The inputs of Q quad steps of 16 terms, four coefficients per lane
  template <int Q> struct Inputs { hcnn_word4 x[Q][4]; };
  // in: the tile's first coefficient of input 0; offsets count 16 bytes (WIDE) or bytes.  terms (a multiple of 16): what is left
  template <bool WIDE, int Q>
  __device__ __forceinline__ static void load(const uint32_t* in, const uint32_t* l_off, uint32_t lane, Inputs<Q>& to, uint32_t terms) {
    typedef const hcnn_word4 __attribute__((address_space(1))) * gptr;
    const uint32_t ln = lane % 16;
    const gptr src = (gptr)(const hcnn_word4*)in + ln;
    auto one = [&](uint32_t off) -> hcnn_word4 {
      if constexpr (WIDE) return src[off];
      else {
        const U4 t = ld4_at(in, off + ln * 16);
        return hcnn_word4{t.x, t.y, t.z, t.w};
      }
    };
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      if (!WIDE && q * 16u >= terms) break;
      const hcnn_word4 off = *reinterpret_cast<const hcnn_word4*>(l_off + q * 16 + lane / 16 * 4);
      to.x[q][0] = one(off.x); to.x[q][1] = one(off.y); to.x[q][2] = one(off.z); to.x[q][3] = one(off.w);
      if (!WIDE) sched_fence();
    }
  }
  // the bytes of four terms' words s as operand words, one per byte plane
  template <class Planes>
  __device__ __forceinline__ static void planes(const hcnn_word4 (&x)[4], int s, int q, Planes& b) {
    const uint32_t lo01 = __builtin_amdgcn_perm(x[1][s], x[0][s], 0x05010400u);    // a0 b0 a1 b1
    const uint32_t hi01 = __builtin_amdgcn_perm(x[1][s], x[0][s], 0x07030602u);    // a2 b2 a3 b3
    const uint32_t lo23 = __builtin_amdgcn_perm(x[3][s], x[2][s], 0x05010400u);
    const uint32_t hi23 = __builtin_amdgcn_perm(x[3][s], x[2][s], 0x07030602u);
    b[0][q] = (int32_t)(__builtin_amdgcn_perm(lo23, lo01, 0x05040100u) ^ 0x80808080u);
    b[1][q] = (int32_t)(__builtin_amdgcn_perm(lo23, lo01, 0x07060302u) ^ 0x80808080u);
    b[2][q] = (int32_t)(__builtin_amdgcn_perm(hi23, hi01, 0x05040100u) ^ 0x80808080u);
    b[3][q] = (int32_t)__builtin_amdgcn_perm(hi23, hi01, 0x07060302u);
  }
  // Two quad steps (half h of a chunk) times the weights of one set: half as many inputs in registers, half as long products
  __device__ __forceinline__ static void multiply_half(const Inputs<2>& in, const uint32_t* l_w, uint32_t h, uint32_t lane, Sums (&acc)[4][4]) {
    typedef int32_t Vec2 __attribute__((ext_vector_type(2)));
    const int64_t w = __builtin_bit_cast(int64_t, *reinterpret_cast<const Vec2*>(l_w + lane * 4 + h * 2));
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      Vec2 b[4];
#pragma unroll
      for (int q = 0; q < 2; ++q) planes(in.x[q], s, q, b);
#pragma unroll
      for (int j = 0; j < 4; ++j)
        acc[s][j].v = __builtin_amdgcn_mfma_i32_16x16x32_i8(w, __builtin_bit_cast(int64_t, b[j]), acc[s][j].v, 0, 0, 0);
    }
  }
  // ... and their products with the weights of NG groups, w_stride words apart; operand words beyond the Q steps are zero
  template <int Q, int NG>
  __device__ __forceinline__ static void multiply(const Inputs<Q>& in, const uint32_t* l_w, uint32_t w_stride, uint32_t lane, Sums (&acc)[NG][4][4]) {
    Vec w[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) w[g] = reinterpret_cast<const Vec*>(l_w + g * w_stride)[lane];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      Vec b[4] = {};
#pragma unroll
      for (int q = 0; q < Q; ++q) planes(in.x[q], s, q, b);
#pragma unroll
      for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[g][s][j].v = __builtin_amdgcn_mfma_i32_16x16x64_i8(w[g], b[j], acc[g][s][j].v, 0, 0, 0);
      if (NG > 1) sched_fence();
    }
  }
#endif

  // Sums of the 64 coefficients of tile t for NG groups, as residues in [0, p): word s of out[group][r] belongs to filter
  // 4 (lane / 16) + r and coefficient 4 (lane % 16) + s.  l_off: `terms` offsets (a multiple of 16; WIDE: in 16-byte units, else
  // bytes), l_w the groups' weight words, w_stride apart, zero beyond the last term, wsum 128 times the sums of their weights.
  template <int NG, bool WIDE>
  HCNN_HD static void tile(const MacArgs& a, uint32_t t, const uint32_t* l_off, const uint32_t* l_w, uint32_t w_stride, uint32_t terms,
                           uint32_t lane, const Sums (&wsum)[NG], U4 (&out)[NG][4]) {
    const NttLimb L = ldc(a.limbs, t / (a.n / kTile) % a.k);
    const uint32_t* in = a.in + t * kTile;
    Sums acc[NG][4][4];                                               // [group][s][byte]
#pragma unroll
    for (int gi = 0; gi < NG; ++gi)
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[gi][s][j] = j < 3 ? wsum[gi] : Sums{};
    if constexpr (NG == 1 && !WIDE) {
      // half a chunk at a time: four waves per SIMD
      Inputs<2> x{};
      for (uint32_t c = 0; c * 32 < terms; ++c) {
        load<WIDE>(in, l_off + c * 32, lane, x, terms - c * 32);
        multiply_half(x, l_w + c / 2 * 256, c % 2, lane, acc[0]);
      }
    } else if constexpr (NG > 1) {
      // one loop body (a second one does not hold the sums in registers): a quad step beyond the last is not loaded, what its
      // operand words hold meets weights of zero
      Inputs<4> x{};
      for (uint32_t c = 0; c * 64 < terms; ++c) {
        load<WIDE>(in, l_off + c * 64, lane, x, terms - c * 64);
        multiply(x, l_w + c * 256, w_stride, lane, acc);
      }
    } else {
      auto step = [&](auto q, uint32_t c) {
        Inputs<decltype(q)::value> x;
        load<WIDE>(in, l_off + c * 64, lane, x, 64);
        multiply(x, l_w + c * 256, w_stride, lane, acc);
      };
      for (uint32_t c = 0; c * 64 < terms; ++c) {
        if (c * 64 + 64 <= terms) step(std::integral_constant<int, 4>{}, c);
        else if (c * 64 + 48 <= terms) step(std::integral_constant<int, 3>{}, c);
        else if (c * 64 + 32 <= terms) step(std::integral_constant<int, 2>{}, c);
        else step(std::integral_constant<int, 1>{}, c);
      }
    }
#pragma unroll
    for (int gi = 0; gi < NG; ++gi) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        uint32_t o[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          int64_t x = (int64_t)acc[gi][s][0].v[r] * L.rc;
          x += (int64_t)acc[gi][s][1].v[r] * L.byte_c[0];
          x += (int64_t)acc[gi][s][2].v[r] * L.byte_c[1];
          x += (int64_t)acc[gi][s][3].v[r] * L.byte_c[2];
          o[s] = canon_p(sredc(x, L.m.p, L.pinv), L.m.p);
        }
        out[gi][r].x = o[0]; out[gi][r].y = o[1]; out[gi][r].z = o[2]; out[gi][r].w = o[3];
      }
    }
  }
  HCNN_HD static void store(const MacArgs& a, uint32_t f, uint32_t g, uint32_t t, uint32_t lane, const U4& u) {
    if (f < a.F && g < a.G) *reinterpret_cast<U4*>(a.out + ((size_t)f * a.G + g) * ((size_t)2 * a.k * a.n) + t * kTile + lane % 16 * 4) = u;
  }
};

template <int GB>
struct MacMfma : MacMatrix {
  // (one group: the workgroup's waves take tiles, and eight of them share the staged tables)
  static constexpr int kThreads = GB == 1 ? 512 : 256;
  static constexpr int kPhases = 2;
  static constexpr int kMinWavesPerSimd = 2;     // 64 registers of inputs in flight, 64 of sums
  struct Regs {};
  static constexpr uint32_t kStreams = kThreads / 64 / GB;      // waves on one group
  static uint32_t max_steps(const MacArgs&) { return 8; }
  HCNN_HOSTDEV static uint32_t terms(uint32_t T) { return (T + 15) / 16 * 16; }
  // offsets and weights of one group (32 bits hold it for every row that lds_bytes lets through)
  HCNN_HOSTDEV static uint32_t group_words(uint32_t T) { return chunks(T) * (64 + 256); }
  static size_t lds_bytes(size_t T) { return (size_t)GB * ((T + 63) / 64 * (64 + 256)) * 4; }
  static uint32_t tile_blocks(const MacArgs& a) {
    const uint32_t per = a.steps * kStreams, tiles = 2 * a.k * a.n / kTile;
    return (tiles + per - 1) / per;
  }
  static size_t grid(const MacArgs& a) { return MacMatrix::grid(tile_blocks(a), (a.G + GB - 1) / GB); }

  template <int PH>
  HCNN_HD static void phase(const MacArgs& a, unsigned bid, int tid, uint32_t* lds, Regs&) {
    const uint32_t g_blocks = (a.G + GB - 1) / GB;
    const uint32_t xcd = bid % kXcds, local = bid / kXcds;
    const uint32_t tb = (local / g_blocks) * kXcds + xcd, g0 = local % g_blocks * GB;
    const uint32_t tiles = 2 * a.k * a.n / kTile;
    const uint32_t tile0 = tb * a.steps * kStreams;
    if (tile0 >= tiles) return;                                       // padding blocks (whole block)
    const uint32_t words = group_words(a.T), T16 = terms(a.T);
    if constexpr (PH == 0) {
      // Every load is unconditional (clamped to the row's last term, the last filter, the last group) and the groups' loads
      // are issued together: with a branch per load the eight loads of a word waited for one another, and a launch that
      // runs few tiles per workgroup spent most of its time here (us, branches / now, four groups per workgroup: 14 filters x 25
      // terms, 4 groups, n = 8192, k = 8 22.1 / 17.2; 10 x 96 36.6 / 30.0)
      const uint32_t* idx[GB];
      const int32_t* w[GB];
#pragma unroll
      for (uint32_t gi = 0; gi < GB; ++gi) {
        const size_t g = g0 + gi < a.G ? g0 + gi : a.G - 1;
        idx[gi] = a.idx + g * a.T;
        w[gi] = a.w + g * a.F * a.T;
      }
      uint32_t bad = 0;
      for (uint32_t t = tid; t < T16; t += kThreads) {
        uint32_t src[GB];
#pragma unroll
        for (uint32_t gi = 0; gi < GB; ++gi) src[gi] = idx[gi][t < a.T ? t : a.T - 1];
#pragma unroll
        for (uint32_t gi = 0; gi < GB; ++gi) {
          const bool out = src[gi] >= a.n_in;
          bad += out && t < a.T && g0 + gi < a.G;
          lds[gi * words + t] = (out ? 0 : src[gi]) * (2u * a.k * a.n / 4);       // in 16-byte units (the host checked that it fits)
        }
      }
      for (uint32_t x = tid; x < chunks(a.T) * 256; x += kThreads) {
        // four terms of a filter per thread; the 64 bytes of a quad step lie with four neighbours, so that a wave's load
        // touches 16 short runs and not 64 words (rows of a multiple of 32 terms suffered most: 128 bytes apart)
        const uint32_t lg = x % 4, f = x / 4 % 16, q = x / 64 % 4, t0 = x / 256 * 64 + q * 16 + lg * 4;
        const uint32_t word = x / 256 * 256 + (lg * 16 + f) * 4 + q;
        int32_t wf[GB][4];
        uint32_t src[GB][4];
#pragma unroll
        for (uint32_t gi = 0; gi < GB; ++gi)
#pragma unroll
          for (uint32_t b = 0; b < 4; ++b) {
            const uint32_t t = t0 + b < a.T ? t0 + b : a.T - 1;
            wf[gi][b] = w[gi][(size_t)(f < a.F ? f : a.F - 1) * a.T + t];
            src[gi][b] = idx[gi][t];
          }
#pragma unroll
        for (uint32_t gi = 0; gi < GB; ++gi) {
          uint32_t packed = 0;
#pragma unroll
          for (uint32_t b = 0; b < 4; ++b) {
            const bool term = (t0 + b < a.T) & (f < a.F), beyond = (wf[gi][b] > a.w_abs_max) | (wf[gi][b] < -a.w_abs_max);
            bad += term & beyond & (g0 + gi < a.G);
            packed |= (term & !beyond & (src[gi][b] < a.n_in)) ? (uint32_t)(wf[gi][b] & 0xff) << (8 * b) : 0u;
          }
          lds[gi * words + chunks(a.T) * 64 + word] = packed;
        }
      }
      if (tb == 0)
        for (; bad != 0; --bad) atomic_inc64(a.bad_counter);
    } else {
      const uint32_t wave = wave_uniform((uint32_t)tid / 64), lane = (uint32_t)tid % 64;
      const uint32_t gi = wave % GB, g = g0 + gi;
      if (g >= a.G) return;
      const uint32_t* l_off = lds + gi * words;
      const uint32_t* l_w = l_off + chunks(a.T) * 64;
      Sums wsum[1];                                                      // 128 * sum of the weights, per filter
      weight_sums(l_w, chunks(a.T), lane, wsum[0]);
      for (uint32_t st = 0; st < a.steps; ++st) {
        const uint32_t t = tile0 + st * kStreams + wave / GB;
        if (t >= tiles) break;
        U4 u[1][4];
        tile<1, true>(a, t, l_off, l_w, 0, T16, lane, wsum, u);
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) store(a, lane / 16 * 4 + r, g, t, lane, u[0][r]);
      }
    }
  }
};

// Neighbouring groups as one, over the union of their rows.  Neighbouring placements of a 3 x 3 kernel share two thirds of their
// inputs, and the kernel above is bound by the gather; a term that only some of the groups have meets zero weights of the others in the
// matrix unit, which has room.
//   MacPair: two groups of up to 16 filters, a set of sums each (12 loads for every 18 of the kernel above)
//   MacPack: 16 / F groups of F <= 8 filters side by side in the sixteen rows of one set.  Half a chunk of terms at a time, so that four waves
//   fit a SIMD (121 registers; whole chunks take 180: 5 x 25, stride 2, 144 groups, n = 8192, k = 8 192 us, 174 with halves, vector form
//   224; its inputs and outputs take 166 at the copy rate)
// The tables are built from the rows as they are, in any order: phases
//   0  clear         1  a bit per group and input that a term of non-zero weight names      2-4  prefix sums of the union's bits: a slot
//   per input        5  offsets and weight bytes to their slots; a term that names an input a second time in its row gets a slot of
//   its own behind them (the slots hold at most the terms of both rows)
//   6  sums: every wave its own tiles of 64 coefficients, as above
template <int SETS>
struct MacUnion : MacMatrix {
  static constexpr int kThreads = 256;
  static constexpr int kPhases = 7;
  static constexpr int kMinWavesPerSimd = SETS == 1 ? 4 : 2;     // 64 registers of sums per set, 32 or 64 of inputs in flight
  static constexpr uint32_t kStreams = kThreads / 64;
  static constexpr uint32_t kRows = SETS == 1 ? 8 : 16;              // filters at most
  struct Regs {};
  HCNN_HOSTDEV static uint32_t groups(const MacArgs& a) { return SETS == 1 ? a.pack : (uint32_t)SETS; }
  // LDS: offsets, weights of every set; a bit per input that a group names, each group's claimed ones, the first slot of every 32 inputs,
  // counts of the threads' and of sixteen threads' slots and their sum, slots of repeated terms
  HCNN_HOSTDEV static uint32_t bit_words(uint32_t n_in) { return (n_in + 31) / 32; }
  static size_t lds_bytes(size_t groups, size_t T, size_t n_in) {
    return ((groups * T + 63) / 64 * (64 + SETS * 256) + (n_in + 31) / 32 * (2 + groups) + kThreads + 16 + 4) * 4;
  }
  static uint32_t tile_blocks(const MacArgs& a) {
    const uint32_t per = a.steps * kStreams, tiles = 2 * a.k * a.n / kTile;
    return (tiles + per - 1) / per;
  }
  static size_t grid(const MacArgs& a) { return MacMatrix::grid(tile_blocks(a), (a.G + groups(a) - 1) / groups(a)); }

  template <int PH>
  HCNN_HD static void phase(const MacArgs& a, unsigned bid, int tid, uint32_t* lds, Regs&) {
    const uint32_t n_grp = groups(a), g_blocks = (a.G + n_grp - 1) / n_grp;
    const uint32_t xcd = bid % kXcds, local = bid / kXcds;
    const uint32_t tb = (local / g_blocks) * kXcds + xcd, g0 = local % g_blocks * n_grp;
    const uint32_t tiles = 2 * a.k * a.n / kTile, tile0 = tb * a.steps * kStreams;
    if (tile0 >= tiles) return;                                       // padding blocks (whole block)
    const uint32_t cap = chunks(n_grp * a.T), bw = bit_words(a.n_in);
    uint32_t* l_off = lds;
    uint32_t* l_w = lds + cap * 64;                                   // [SETS][cap][256]
    uint32_t* bits = l_w + cap * SETS * 256;
    uint32_t* claim = bits + bw;                                      // [n_grp][bw]
    uint32_t* first = claim + n_grp * bw;                             // slots in front of a word's
    uint32_t* part = first + bw;                                      // [256 + 16]
    uint32_t* total = part + kThreads + 16;                           // slots without the repeated terms'
    uint32_t* count = total + 1;                                      // slots of repeated terms
    const uint32_t per = (bw + kThreads - 1) / kThreads, w0 = (uint32_t)tid * per, w1 = w0 + per < bw ? w0 + per : bw;     // words of this thread
    const uint32_t wave = wave_uniform((uint32_t)tid / 64), lane = (uint32_t)tid % 64;
    if constexpr (PH == 0) {
      for (uint32_t i = tid; i < cap * (64 + SETS * 256) + (1 + n_grp) * bw; i += kThreads) lds[i] = 0;
      if (tid == 0) *count = 0;
    } else if constexpr (PH == 1 || PH == 5) {
      uint32_t bad = 0;
      const uint32_t here = g0 + n_grp <= a.G ? n_grp : a.G - g0;
      for (uint32_t x = tid; x < here * a.T; x += kThreads) {
        const uint32_t gi = quot(x, a.terms), t = x - gi * a.T;
        const uint32_t src = a.idx[(size_t)(g0 + gi) * a.T + t];
        const int32_t* w = a.w + (size_t)(g0 + gi) * a.F * a.T;
        int32_t wf[kRows];
#pragma unroll
        for (uint32_t f = 0; f < kRows; ++f) wf[f] = w[(size_t)(f < a.F ? f : a.F - 1) * a.T + t];        // (all loads together)
        uint32_t any = 0;
#pragma unroll
        for (uint32_t f = 0; f < kRows; ++f) {
          const bool beyond = (wf[f] > a.w_abs_max) | (wf[f] < -a.w_abs_max);
          bad += beyond & (f < a.F);
          if (beyond | (f >= a.F)) wf[f] = 0;
          any |= (uint32_t)wf[f];
        }
        bad += src >= a.n_in;
        if (src >= a.n_in || any == 0) continue;
        const uint32_t word = src / 32, bit = 1u << (src % 32);
        if constexpr (PH == 1) {
          lds_or(bits + word, bit);
        } else {
          uint32_t slot;
          if (lds_or(claim + gi * bw + word, bit) & bit) slot = *total + lds_add(count, 1);
          else slot = first[word] + (uint32_t)__builtin_popcount(bits[word] & (bit - 1));
          l_off[slot] = src * (2u * a.k * a.n * 4);                  // in bytes (the host checked that it fits)
          const uint32_t set = SETS == 1 ? 0 : gi, row = SETS == 1 ? gi * a.F : 0;
          uint8_t* bytes = reinterpret_cast<uint8_t*>(l_w + (set * cap + slot / 64) * 256 + slot / 4 % 4 * 64 + slot / 16 % 4) + slot % 4 + row * 16;
#pragma unroll
          for (uint32_t f = 0; f < kRows; ++f)
            if (SETS > 1 || f < a.F) bytes[f * 16] = (uint8_t)wf[f];
        }
      }
      if (PH == 1 && tb == 0)
        for (; bad != 0; --bad) atomic_inc64(a.bad_counter);
    } else if constexpr (PH == 2) {
      uint32_t n = 0;
      for (uint32_t i = w0; i < w1; ++i) n += (uint32_t)__builtin_popcount(bits[i]);
      part[tid] = n;
    } else if constexpr (PH == 3) {
      if (tid < 16) {
        uint32_t n = 0;
        for (int i = 0; i < 16; ++i) n += part[16 * tid + i];
        part[kThreads + tid] = n;
      }
    } else if constexpr (PH == 4) {
      uint32_t n = 0;
      for (int i = 0; i < tid / 16; ++i) n += part[kThreads + i];
      for (int i = tid / 16 * 16; i < tid; ++i) n += part[i];
      if (tid == kThreads - 1) *total = n + part[tid];
      for (uint32_t i = w0; i < w1; ++i) {
        first[i] = n;
        n += (uint32_t)__builtin_popcount(bits[i]);
      }
    } else {
      const uint32_t used = wave_uniform(*total + *count);
      Sums wsum[SETS];
#pragma unroll
      for (int gi = 0; gi < SETS; ++gi) weight_sums(l_w + gi * cap * 256, chunks(used), lane, wsum[gi]);
      for (uint32_t st = 0; st < a.steps; ++st) {
        const uint32_t t = tile0 + st * kStreams + wave;
        if (t >= tiles) break;
        U4 u[SETS][4];
        tile<SETS, false>(a, t, l_off, l_w, cap * 256, (used + 15) / 16 * 16, lane, wsum, u);
#pragma unroll
        for (uint32_t gi = 0; gi < SETS; ++gi)
#pragma unroll
          for (uint32_t r = 0; r < 4; ++r) {
            const uint32_t row = lane / 16 * 4 + r, in_set = SETS == 1 ? quot(row, a.filters) : 0;
            if (SETS > 1 || in_set < n_grp) store(a, row - in_set * a.F, g0 + gi + in_set, t, lane, u[gi][r]);
          }
      }
    }
  }
};
// MacPair, measured, us, the kernel above / this one: 16 filters x 576 terms (3 x 3 padded, 8 x 8 map), 64 groups, n = 8192, k = 10 1502 / 1249;
// 12 x 144, 100 groups, k = 8 704 / 562; 16 x 25 (5 x 5, stride 2), 144 groups 523 / 439; 16 x 144, 36 groups, n = 16384, k = 16 1273 / 1000; no input
// shared (2 x 2, stride 2), 16 x 192, 16 groups 356 / 352.
// Bound: inputs from beyond L2.  The first of these gathers 13.7 GB (24 above) but misses L2 for 8.5 GB of them (5.2 above, inputs
// 2.7): 256 waves of a die are at twice as many tiles, 8 MiB of inputs, and drift apart.  Measured and left out, same layer: a wave per quarter of the
// slots, so that four share a tile (sums added through LDS: 1554, two barriers and four reductions per tile), tiles of 32
// coefficients (8-byte loads: 1494), one wave per SIMD with two buffers of inputs (1425 - 1527).  A second loop body for the last terms
// does not hold the sums in registers (100 spilled).
struct MacPair : MacUnion<2> {
  // Tiles per wave at most.  A union leaves out the terms without weight, so that the workgroups at a map's padded border are done sooner and
  // neighbours drift apart in L2, the more the longer they run; shorter runs build the union more often.  Long rows take four tiles: us, 8 /
  // 4 tiles, 16 filters, n = 8192, 3 x 3 padded: 576 terms, 64 groups, k = 10 1339 / 1256, 100 groups, k = 8 1967 / 1815 (with weights on the
  // padding too 1593 / 1620), 504, 144 groups 2484 / 2305; 5 x 5 padded, 600, 144 groups 2043 / 1824.  Without padding they cost up to 8 %:
  // 5 x 5, 600 terms, 64 groups 966 / 1046, 1000 of k = 6 +5 %, 2 x 2, 800 of k = 4 +2 %.  Below, the loss is larger than the gain: 3 x 3
  // padded, 360 terms, 144 groups -7 %, 288, 64 groups 686 / 698; without padding 400 (5 x 5), 64 groups +9 %, 12 x 144, 100 groups 562 / 591;
  // 25 (5 x 5, stride 2), 144 groups 436 / 500.
  static uint32_t max_steps(const MacArgs& a) { return a.T >= 512 ? 4 : 8; }
  static size_t lds_bytes(size_t T, size_t n_in) { return MacUnion<2>::lds_bytes(2, T, n_in); }
};
struct MacPack : MacUnion<1> {
  static constexpr uint32_t kLeastPerUnit = 2;
  // Tiles per wave at most.  What building a union costs (the terms of all its groups) is spread over its own terms times the tiles; many long workgroups
  // come in one to three uneven rounds.  So unions that are long for what they are built of take few tiles (us, 8 / 4 / 2 / 1: 7 x 575, 9 groups, n = 16384,
  // k = 13 852 / 743 / 672 / 582, vector form 703; 4 x 416, 36 groups, n = 8192, k = 11 725 / 624 / 549 / 486, 644; 8 x 72, 169 groups, n = 2048, k = 3 55 / 47 / 38
  // / 48, 81), others eight (1 x 46, 69 groups over 46 inputs, n = 32768, k = 17 148 with eight, 185 with two).  The union is estimated as in
  // mac_takes_pairs.  Of 3900 calls 982 take 3 % or more less than with eight tiles, 49 more, four of them over 10 %; one tile is better still for some and up to 39 %
  // worse where two make enough workgroups.
  static uint32_t max_steps(const MacArgs& a) {
    const double T = a.T, groups = a.pack < a.G ? a.pack : a.G, gathered = (double)a.G * T / a.n_in;
    const double of_rows = T * (1 + (groups - 1) / std::sqrt(gathered > 1 ? gathered : 1.0)), terms = of_rows < a.n_in ? of_rows : a.n_in;
    const double kept = terms * terms / (groups * T);
    return kept >= 120 ? 2 : kept >= 60 ? 4 : 8;
  }
};

// ---------------------------------------------------------------- helpers for KeyGen / Encrypt / Decrypt
// small signed polynomial(s) [count][n] -> residues [count][k][n]
struct SmallToRnsArgs {
  const int32_t* small;
  uint32_t* out;
  const Mod* mods;
  uint32_t k, n;
};
struct SmallToRnsKernel {
  static constexpr int kThreads = kEwThreads;
  static constexpr int kPhases = 1;
  struct Regs {};
  template <int PH>
  HCNN_HD static void phase(const SmallToRnsArgs& a, unsigned bid, int tid, uint32_t*, Regs&) {
    const uint32_t per_poly = a.n / kThreads;
    const size_t poly = bid / per_poly;
    const uint32_t c = (bid % per_poly) * kThreads + tid;
    const int32_t v = a.small[poly * a.n + c];
    for (uint32_t l = 0; l < a.k; ++l) a.out[(poly * a.k + l) * a.n + c] = small_to_res(v, ldc(a.mods, l));
  }
};

// Pointwise c = a (*) b over rows; row r of a is a_rows[r % a_cycle], likewise b; limb = r % k.
// mode: 0 -> c = a*b ; 1 -> c = -(a*b)
struct PointMulArgs {
  const uint32_t* a;
  const uint32_t* b;
  uint32_t* c;
  const Mod* mods;
  uint32_t k, n;
  uint32_t a_cycle, b_cycle;   // in rows
  uint32_t negate;
};
struct PointMulKernel {
  static constexpr int kThreads = kEwThreads;
  static constexpr int kPhases = 1;
  struct Regs {};
  template <int PH>
  HCNN_HD static void phase(const PointMulArgs& a, unsigned bid, int tid, uint32_t*, Regs&) {
    const uint32_t per_row = a.n / kThreads;
    const size_t row = bid / per_row;
    const uint32_t c = (bid % per_row) * kThreads + tid;
    const Mod m = ldc(a.mods, row % a.k);
    const uint32_t x = a.a[(row % a.a_cycle) * a.n + c];
    const uint32_t y = a.b[(row % a.b_cycle) * a.n + c];
    uint32_t r = mul_mod(x, y, m);
    if (a.negate && r != 0) r = m.p - r;
    a.c[row * a.n + c] = r;
  }
};

// out[row] = x[row] + small[poly(row)] ; rows are [count][k][n]
struct AddSmallArgs {
  const uint32_t* x;
  const int32_t* small;        // [count][n]
  uint32_t* out;
  const Mod* mods;
  uint32_t k, n;
  uint32_t subtract_small;     // 1: out = x - small
  uint32_t out_poly_rows, out_row0;   // output row = poly*out_poly_rows + out_row0 + l
};
struct AddSmallKernel {
  static constexpr int kThreads = kEwThreads;
  static constexpr int kPhases = 1;
  struct Regs {};
  template <int PH>
  HCNN_HD static void phase(const AddSmallArgs& a, unsigned bid, int tid, uint32_t*, Regs&) {
    const uint32_t per_row = a.n / kThreads;
    const size_t row = bid / per_row;                  // (poly, l)
    const uint32_t c = (bid % per_row) * kThreads + tid;
    const size_t poly = row / a.k;
    const uint32_t l = (uint32_t)(row % a.k);
    const Mod m = ldc(a.mods, l);
    const uint32_t sv = small_to_res(a.small[poly * a.n + c], m);
    const uint32_t r = a.subtract_small ? sub_mod(a.x[row * a.n + c], sv, m.p) : add_mod(a.x[row * a.n + c], sv, m.p);
    a.out[(poly * a.out_poly_rows + a.out_row0 + l) * a.n + c] = r;
  }
};

// evk[i][0][i] += s2[i] for i < k  (g_i = 1 mod q_i and 0 mod every other prime)
struct AddDiagArgs {
  uint32_t* evk;          // [k][2][k][n]
  const uint32_t* s2;     // [k][n]
  const Mod* mods;
  uint32_t k, n;
};
struct AddDiagKernel {
  static constexpr int kThreads = kEwThreads;
  static constexpr int kPhases = 1;
  struct Regs {};
  template <int PH>
  HCNN_HD static void phase(const AddDiagArgs& a, unsigned bid, int tid, uint32_t*, Regs&) {
    const uint32_t per_row = a.n / kThreads;
    const uint32_t i = bid / per_row;
    const uint32_t c = (bid % per_row) * kThreads + tid;
    uint32_t* dst = a.evk + (((size_t)i * 2 + 0) * a.k + i) * a.n + c;
    *dst = add_mod(*dst, a.s2[(size_t)i * a.n + c], ldc(a.mods, i).p);
  }
};

// Decrypt rounding: x [count][k][n] (c0 + c1*s mod q) -> m = round(t*x/q) mod t, t of up to 47 bits.
// r = [t*x]_q centred is converted to the single modulus t; m = -r * q^-1 mod t = sum_i z_i * b_i + v * b_k with
// b_i = -(q/q_i) q^-1 and b_k = (q mod t) q^-1 = 1 mod t.  The constants are cut into 16-bit pieces: every piece's sum stays
// below (k + 1) 2^46, and three 64-bit remainders put an output together, whatever k is.
struct DecRoundArgs {
  const uint32_t* x;
  uint32_t* m_out;         // 32-bit plaintext words, or null:
  uint64_t* m_out64;       // 64-bit ones
  BConvDev bc;             // source side only (zmul = t*(q/q_i)^-1, xmul = t)
  const uint32_t* tab;     // [k][3]: 16-bit pieces of b_i, least significant first
  const uint32_t* cts;     // HALVES: [count][2][k][n]
  const NttLimb* limbs;    // [k]
  // (in this order the compiler loads the arguments in one turn: with t in front of n and band in two, 10 decryptions, n = 8192, k = 8 16.21 / 16.36 us)
  uint32_t n;
  uint32_t band;
  uint64_t t;
  unsigned long long* fallback_counter;
};
// HALVES: x holds c1*s without the last stage of its inverse transforms and without c0, both taken while loading (positions as in ScaleKernel).
// FOURS: four primes or more (each_prime).
template <bool HALVES, bool FOURS>
struct DecRoundKernel {
  static constexpr int kThreads = kEwThreads;
  static constexpr int kPhases = 1;
  struct Regs {};
  static size_t lds_bytes(uint32_t ks) { return (size_t)2 * ks * kThreads * 4; }
  template <int PH>
  HCNN_HD static void phase(const DecRoundArgs& a, unsigned bid, int tid, uint32_t* lds, Regs&) {
    const uint32_t ks = a.bc.ks, n = a.n;
    const uint32_t per_poly = n / kThreads;
    const size_t poly = bid / per_poly;
    const uint32_t half = HALVES ? ((uint32_t)tid >> 5) & 1u : 0;
    const uint32_t first = HALVES ? (bid % per_poly) * (kThreads / 2) + ((uint32_t)tid >> 6) * 32 + ((uint32_t)tid & 31u)
                                  : (bid % per_poly) * kThreads + tid;
    const uint32_t c = first + half * (n / 2);
    const uint32_t* src = a.x + poly * ks * n + first;
    uint32_t* zcol = lds + tid;
    uint32_t* gcol = lds + (size_t)ks * kThreads + tid;
    const uint32_t* c0 = HALVES ? a.cts + poly * 2 * ks * n + c : nullptr;
    auto in = [&](uint32_t i) -> uint32_t {
      const uint32_t* row = src + (size_t)i * n;
      if constexpr (!HALVES) return row[0];
      const NttLimb* m = a.limbs + i;
      const InvRoot* top = &m->inv_r;        // (the workgroups transform the secret themselves: a product of two plain rows carries 2^-32)
      const uint32_t p = ldc(&m->m.p, 0);
      // (below 3 p: the conversion takes any 32-bit value)
      return (uint32_t)split_root((int32_t)row[0], (int32_t)row[n / 2], split_root_factors(ldc(&top->c0, 0), ldc(&top->w, 0), half), p, ldc(&m->pinv, 0)) +
             p + c0[(size_t)i * n];
    };
    const uint32_t v = bconv_prepare<FOURS>(a.bc, in, zcol, gcol, kThreads, a.band, a.fallback_counter);
    uint64_t s0 = v, s1 = 0, s2 = 0;
    each_prime<FOURS>(ks, [&](uint32_t i) {
      const uint64_t z = zcol[i * kThreads];
      s0 += z * ldc(a.tab, 3 * i);
      s1 += z * ldc(a.tab, 3 * i + 1);
      s2 += z * ldc(a.tab, 3 * i + 2);
    });
    uint64_t r = s2 % a.t;                       // below 2^47: the shifted sums stay below 2^63 + 2^52
    r = ((r << 16) + s1) % a.t;
    r = ((r << 16) + s0) % a.t;
    if (a.m_out) a.m_out[poly * n + c] = (uint32_t)r;
    else         a.m_out64[poly * n + c] = r;
  }
};

// ---------------------------------------------------------------- counter-based sampling
// Every output element is a fixed function of (seed, stream, element index): the word source is Philox4x32 with
// 10 rounds (Salmon et al., SC'11) keyed by the seed, with counter (index low, index high, stream, kind*2^24 +
// attempt); a call gives four words, used in order, and a sampler that needs more moves on to attempt + 1.
struct PhiloxWords { uint32_t w[4]; };
HCNN_HD PhiloxWords philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0, uint32_t k1) {
  for (int round = 0; round < 10; ++round) {
    const uint64_t p0 = (uint64_t)c0 * 0xD2511F53u, p1 = (uint64_t)c2 * 0xCD9E8D57u;
    const uint32_t n0 = (uint32_t)(p1 >> 32) ^ c1 ^ k0, n2 = (uint32_t)(p0 >> 32) ^ c3 ^ k1;
    c1 = (uint32_t)p1; c3 = (uint32_t)p0; c0 = n0; c2 = n2;
    k0 += 0x9E3779B9u; k1 += 0xBB67AE85u;
  }
  PhiloxWords r; r.w[0] = c0; r.w[1] = c1; r.w[2] = c2; r.w[3] = c3;
  return r;
}
enum { kSampleTernary = 1, kSampleGaussian = 2, kSampleUniform = 3 };
constexpr uint32_t kSampleMaxAttempts = 256;   // 1024 words: no sampler comes anywhere near (rejection odds <= 2^-29 per try,
                                               // or 1 - 4p/2^32 for a prime p > 2^29 that is not close to 2^30)
struct SampleArgs {
  void* out;                 // int32 [count][n] (ternary, Gaussian) or uint32 [count][k][n] (uniform)
  const Mod* mods;           // uniform: [k]
  const uint32_t* gauss_t;   // Gaussian: 20 thresholds, T[v] = floor(2^32 * P(|X| <= v))
  uint64_t seed, total;      // total elements
  uint32_t stream, kind, k, n;
};
struct SampleKernel {
  static constexpr int kThreads = kEwThreads;
  static constexpr int kPhases = 1;
  struct Regs {};
  template <int PH>
  HCNN_HD static void phase(const SampleArgs& a, unsigned bid, int tid, uint32_t*, Regs&) {
    const uint64_t idx = (uint64_t)bid * kThreads + (uint64_t)tid;
    if (idx >= a.total) return;
    const uint32_t k0 = (uint32_t)a.seed, k1 = (uint32_t)(a.seed >> 32);
    uint32_t p = 0, lim = 0;
    if (a.kind == kSampleUniform) {
      p = ldc(a.mods, (uint32_t)((idx / a.n) % a.k)).p;
      lim = p * (uint32_t)(0x100000000ull / p);                    // accepted words: below the largest multiple of p
    }
    for (uint32_t attempt = 0; attempt < kSampleMaxAttempts; ++attempt) {
      const PhiloxWords r = philox4x32_10((uint32_t)idx, (uint32_t)(idx >> 32), a.stream, (a.kind << 24) + attempt, k0, k1);
      if (a.kind == kSampleGaussian) {
        for (int s = 0; s < 4; s += 2) {
          const uint32_t x = r.w[s], y = r.w[s + 1];
          if (x >= ldc(a.gauss_t, 19)) continue;                    // beyond the cut: redraw
          int32_t mag = 0;
          for (uint32_t v = 0; v < 20; ++v) mag += ldc(a.gauss_t, v) <= x ? 1 : 0;
          reinterpret_cast<int32_t*>(a.out)[idx] = (y & 1u) ? -mag : mag;
          return;
        }
      } else {
        for (int s = 0; s < 4; ++s) {
          const uint32_t x = r.w[s];
          if (a.kind == kSampleTernary) {
            if (x == 0xFFFFFFFFu) continue;                         // 2^32 - 1 words split evenly over three values
            reinterpret_cast<int32_t*>(a.out)[idx] = (int32_t)(x % 3u) - 1;
          } else {
            if (x >= lim) continue;
            reinterpret_cast<uint32_t*>(a.out)[idx] = x % p;
          }
          return;
        }
      }
    }
    reinterpret_cast<uint32_t*>(a.out)[idx] = 0;                    // not reached in practice (see kSampleMaxAttempts)
  }
};

// Noise read-out: x [count][k][n] (c0 + c1*s mod q) -> bits[count] = bit length of max_j |r_j|, r = [t*x]_q centred.
// Exact: the residues of the non-negative remainder R = t*x mod q are turned into mixed-radix digits, R > (q-1)/2
// is decided on the digits, |r| = R or q - R is rebuilt as a multiword integer by Horner's rule on the digits, and its
// bit length is folded into the ciphertext's maximum.  bits[] must be zero on entry.
struct NoiseArgs {
  const uint32_t* x;
  uint32_t* bits;
  BConvDev bc;             // src q with xmul = t (the table of the decrypt rounding)
  uint32_t n;
};
struct NoiseKernel {
  static constexpr int kThreads = kEwThreads;
  static constexpr int kPhases = 1;
  struct Regs {};
  static size_t lds_bytes(uint32_t ks) { return (size_t)2 * ks * kThreads * 4; }
  template <int PH>
  HCNN_HD static void phase(const NoiseArgs& a, unsigned bid, int tid, uint32_t* lds, Regs&) {
    const uint32_t ks = a.bc.ks, n = a.n;
    const uint32_t per_poly = n / kThreads;
    const size_t poly = bid / per_poly;
    const uint32_t c = (bid % per_poly) * kThreads + tid;
    const uint32_t* src = a.x + poly * ks * n + c;
    uint32_t* dig = lds + tid;                                   // mixed-radix digits
    uint32_t* word = lds + (size_t)ks * kThreads + tid;          // multiword |r|, least significant first
    for (uint32_t i = 0; i < ks; ++i)
      dig[i * kThreads] = shoup_mul(src[(size_t)i * n], ldc(a.bc.xmul, i), ldc(a.bc.src_mod, i).p);
    if (garner_gt_half(a.bc, dig, kThreads)) {
      // digits of q - R: zero while the lower digits of R are zero, q_i - d_i at the first non-zero digit,
      // q_i - 1 - d_i above it
      bool low_zero = true;
      for (uint32_t i = 0; i < ks; ++i) {
        const uint32_t d = dig[i * kThreads], qi = ldc(a.bc.src_mod, i).p;
        if (low_zero) {
          if (d != 0) { dig[i * kThreads] = qi - d; low_zero = false; }
        } else {
          dig[i * kThreads] = qi - 1 - d;
        }
      }
    }
    // value = d_0 + q_0*(d_1 + q_1*(d_2 + ...)): Horner from the top digit; it stays below q < 2^(30 ks)
    for (uint32_t w = 0; w < ks; ++w) word[w * kThreads] = 0;
    for (int i = (int)ks - 1; i >= 0; --i) {
      uint64_t carry = dig[i * kThreads];
      const uint64_t qi = ldc(a.bc.src_mod, (uint32_t)i).p;
      for (uint32_t w = 0; w < ks; ++w) {
        const uint64_t v = (uint64_t)word[w * kThreads] * qi + carry;
        word[w * kThreads] = (uint32_t)v;
        carry = v >> 32;
      }
    }
    uint32_t bits = 0;
    for (int w = (int)ks - 1; w >= 0; --w) {
      uint32_t v = word[w * kThreads];
      if (v != 0) {
        uint32_t len = 0;
        while (v) { ++len; v >>= 1; }
        bits = 32u * (uint32_t)w + len;
        break;
      }
    }
    if (bits) atomic_max32(a.bits + poly, bits);
  }
};

}  // namespace hcnn
