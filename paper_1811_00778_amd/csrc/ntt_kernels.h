// Batched negacyclic NTT over 30-bit primes, one workgroup per (polynomial, limb) row.
//
// Forward: Cooley-Tukey butterflies with the powers of psi merged into the
// twiddles, natural order in, bit-reversed order out (index j holds the value at
// psi^(2*brev(j)+1)).  Inverse: Gentleman-Sande butterflies with the inverse
// twiddles in the reverse stage order, n^-1 merged into the last stage.
//
// The log2(n) stages are cut into passes of at most LOGR stages.  In a pass every
// thread keeps R = 2^LOGR residues in registers and runs complete radix-2^NS
// networks on them; between passes the row lives in LDS (one barrier per transform, see first_net).
// The first pass reads HBM with unit stride across lanes, the last pass writes HBM.
//
// Residues are SIGNED inside a transform and the stages are taken two at a time, as one
// radix-4 butterfly whose products are summed in 64 bits before a shared Montgomery
// reduction (sredc).  What bounds these kernels is VALU issue, and on this device a
// multiplication, a 64-bit multiply-add, v_min_u32 and v_add3_u32 all issue at 34-36 T
// lane-instructions/s, a plain 32-bit addition or subtraction at 57-61 T.  Counted in
// multiplications, four residues through two stages cost 17 (7 multiply-adds, 4 reductions
// of 2, 4 additions at one half) against 24 of four lazy Shoup butterflies (each 3 for the
// product, 1.5 for the conditional subtraction, 1.5 for sum and difference).  There is no
// conditional subtraction: with |x| < 2^31 on entry every output of a forward radix-4
// butterfly lies in (-2p, 2p), and with |x| <= p on entry every output of an inverse one
// lies in (-p, p), whatever the number of stages (see r4_fwd, r4_inv).  An odd log2(n) adds
// one radix-2 stage at the root of the tree: first in the forward transform, where the
// inputs are still small enough to need no reduction, last in the inverse.
//
// Twiddle tables: the radix-4 butterfly rooted at node m+i of the stage with m groups
// (node m+i = psi^brev_{log n}(m+i)) needs five constants, all centred and carrying the
// factor 2^32 of the reduction: W = tw[node], V = tw[2 node], V*W, U = tw[2 node + 1] (one
// 16-byte word) and -U*W.  A network rooted at node r uses the sub-tree r, 4r.., 16r.., ...
#pragma once
#include "modarith.h"

namespace hcnn {

struct alignas(16) R4Twiddle {
  int32_t w, v, vw, u;
};
struct TwTable {
  const R4Twiddle* quad;    // [L][n/2], index = node
  const int32_t* nuw;       // [L][n/2], -u*w
};
// Constants of the outermost butterfly of an inverse transform (node 1), with the output scaling folded in:
// odd log2(n): c0 = scale, w = tw^-1 * scale; even: all six of a radix-4 butterfly
struct InvRoot {
  int32_t c0, w, v, u, vw, nuw;
};

struct NttLimb {
  Mod m;
  int32_t rc;           // 2^32 mod p, centred: 1 in the form of the twiddles
  uint32_t pinv;        // -p^-1 mod 2^32
  int32_t zero;         // 0, unknown to the compiler: zero - w is a negated constant and stays one (it would turn a visible
                        // negation into a product and a 64-bit subtraction)
  int32_t w1;           // forward twiddle of node 1 (the radix-2 stage of an odd log2(n))
  int32_t key_scale;    // 2^64 mod p, centred: sredc(x * key_scale) = x * 2^32
  int32_t byte_c[3];    // 2^40, 2^48, 2^56 mod p, centred (byte planes of MacMfma)
  InvRoot inv;          // scale = n^-1
  InvRoot inv_r;        // scale = n^-1 * 2^32: the tensor-forming loads leave a factor 2^-32 on every product
  InvRoot inv_z;        // scale = n^-1 * (R/p)^-1: the primes of the shared-basis relinearisation (product R)
};
// Shared-basis relinearisation: a key product modulo q_j q_j', two neighbouring primes of the ciphertext at a time (pair g: j = 2g,
// j' = 2g + 1; the last prime of an odd basis alone), is computed modulo the four primes p_0 .. p_3 and taken to modulo q_j and q_j'.
// With z_r = [x_r (R/p_r)^-1] in (-p_r, p_r) and |X| < R/64, sum_r z_r R/p_r = X + v R with v = round(sum_r z_r/p_r), and
// that sum lies within 1/64 of an integer: fp32 decides it.
constexpr uint32_t kSharedPrimes = 4;
struct RelinCrt {
  int32_t c[kSharedPrimes];         // R/p_r * 2^32 mod q_j, centred
  int32_t cv;                       // -R * 2^32 mod q_j, centred
};
struct RelinCrtInv { float f[kSharedPrimes]; };      // 1 / p_r
HCNN_HD int32_t relin_crt_round(const int32_t (&z)[kSharedPrimes], const RelinCrtInv& f) {
  const float v = (float)z[0] * f.f[0] + (float)z[1] * f.f[1] + (float)z[2] * f.f[2] + (float)z[3] * f.f[3];
  return (int32_t)(v < 0.0f ? v - 0.5f : v + 0.5f);
}
HCNN_HD uint32_t relin_crt(const int32_t (&z)[kSharedPrimes], int32_t v, const RelinCrt& k, uint32_t q, uint32_t qinv) {
  // |z| < p < 2^30 - 2n, |c| <= q/2, |v| <= 4: the sum is below 2^61, and |reduced| <= 4 (p/2^30) q/8 + q/2 + 1 < q
  const int64_t s = (int64_t)z[0] * k.c[0] + (int64_t)z[1] * k.c[1] + (int64_t)z[2] * k.c[2] + (int64_t)z[3] * k.c[3] + (int64_t)v * k.cv;
  return canon_p(sredc(s, q, qinv), q);
}
// A key coefficient modulo q_j q_j' from its residues a, a' is a + q_j t with t = [(a' - a) q_j^-1] modulo q_j', taken in
// (-5/8 q_j', 5/8 q_j'), and so within 5/8 q_j q_j' + q_j of zero.
struct RelinPair {
  int32_t inv;                      // q_j^-1 * 2^32 mod q_j', centred; 0 for the prime without a partner (t = 0)
  int32_t q[kSharedPrimes];         // q_j * 2^32 mod p_r, centred
};

// Encryption: floor(q/t) * m as products in front of the last reduction of an inverse transform, m taken in 32-bit words less
// 2^31 (signed operands); the constants carry the factor 2^32 of the reduction and are centred.
struct EncScale {
  int32_t lo, hi;       // floor(q/t), floor(q/t) * 2^32
  int32_t c32, c64;     // what the 2^31 taken off a 32-bit, a 64-bit word leave out
};

// Row r (= workgroup index) belongs to group r / cycle and limb limb_base + r % cycle.
// Its data sits at row (group * group_rows + row0 + r % cycle) of the in / out arrays, so a
// launch can pick one polynomial out of every ciphertext of a batch.
// The last stage of an inverse transform left at its halves (NttInv, SPLIT = 1): element `half * n/2 + i` of the row from elements i and
// i + n/2 as they were left, signed in (-p, p); c0, w: the root constants with the output scaling.  Result in (-p, p): two
// products of at most p * p/2.
struct SplitRoot { int32_t x, y; };
HCNN_HOSTDEV SplitRoot split_root_factors(int32_t c0, int32_t w, uint32_t half) {
  return half ? SplitRoot{w, -w} : SplitRoot{c0, c0};
}
HCNN_HD int32_t split_root(int32_t lo, int32_t hi, const SplitRoot& f, uint32_t p, uint32_t pinv) {
  return sredc(untraced((int64_t)lo * f.x) + (int64_t)hi * f.y, p, pinv);
}

// Fused input / output stages (template parameter IO of the kernels):
//   kNttPlain       rows are read and written as they are
//   kNttLoadDigit   forward only: row (ct, i, j) reads digit i of y2, i.e. row (ct*3+2)*k + i of `in`
//                   = y[n_ct][3][k][n], taken as it is (every prime lies in (2^29, 2^30), so a digit is below
//                   2*q_j); output rows dense [ct][i][j], left signed in [-p, p)
//   kNttLoadTensor  inverse only: row (ct, b, l) reads c0^ = in[(ct*2)*L + l], c1^ = in[(ct*2+1)*L + l]
//                   and transforms c0^*c0^, 2*c0^*c1^ or c1^*c1^ for b = 0, 1, 2 (HMult step 1, c = c')
//   kNttLoadTensorMul  inverse only: the general tensor of HMult step 1 for two different operands;
//                   `in` holds the first, `aux` the second (same [ct][2][L][n] layout):
//                   c0^*c0'^, c0^*c1'^ + c1^*c0'^, c1^*c1'^
//   kNttStoreAdd    inverse only: row (ct, b, j) adds aux row (ct*3+b)*k + j (aux = y) on the way out
//   kNttStoreLazy   forward only: the output is left signed, in [-p, p) (for rows whose only reader is the
//                   tensor-forming load)
//   kNttStoreKey    forward only: the output is multiplied by 2^32 and centred (evaluation-key rows: the sums of their
//                   products with the digits go through one Montgomery reduction, and |key| <= p/2 leaves room for more)
// The tensor-forming loads leave their output lazily reduced, in [0, 2p): its only reader multiplies it
// by a constant with Shoup's method, which takes any 32-bit operand.
//   kNttFusedMac    forward only, inside RelinFused: workgroup (ct, j) transforms digit `iter` of y2 modulo q_j
//                   (loaded like kNttLoadDigit) and, instead of storing, adds its products with the two key
//                   rows evk^[iter][0][j], evk^[iter][1][j] (`aux`) to 64-bit sums held in registers
//   kNttFromRegs0/1 inverse only, inside RelinFused: the input is the register-held sum of component 0 / 1;
//                   the output adds y row (ct, b, j) (`aux`) like kNttStoreAdd and goes to out row (ct, b, j)
enum NttIo { kNttPlain = 0, kNttLoadDigit = 1, kNttLoadTensor = 2, kNttStoreAdd = 3, kNttLoadTensorMul = 4,
             kNttStoreLazy = 5, kNttFusedMac = 6, kNttFromRegs0 = 7, kNttFromRegs1 = 8,
             kNttFusedMac16 = 9, kNttFusedMacAny = 10,     // the fused inner product for k <= 8, k <= 16, any k
             kNttToRegs0 = 11, kNttToRegs1 = 12,           // forward, inside TensorFused: c0 / c1 of workgroup (ct, limb); the
                                                           // transformed row stays in registers, signed in [-p, p)
             kNttTensorRegs0 = 13, kNttTensorRegs1 = 14, kNttTensorRegs2 = 15,      // inverse, inside TensorFused: component b
                                                           // of the tensor formed from those registers (as kNttLoadTensor)
             kNttStoreKey = 16,
             // forward, inside CryptFused: the encryption's u (small signed values, [ct][n], limb by limb) or the
             // decryption's c1 into registers; kNttSmallKey: the secret's rows, stored like kNttStoreKey
             kNttSmallToRegs = 17, kNttSmallKey = 18, kNttCtToRegs = 19,
             // inverse, inside CryptFused: the registers times a key row, plus what Encrypt / Decrypt add
             kNttEncOut0 = 20, kNttEncOut1 = 21, kNttDecOut = 22,
             // inverse, shared-basis relinearisation: row (ct, o, r) with the scaling of inv_z, output signed in (-p, p):
             // to memory, or (inside RelinBack) to registers and, from the last, through the base change to the outputs
             kNttBackRow = 23, kNttBack0 = 24, kNttBack1 = 25, kNttBack2 = 26, kNttBack3 = 32,
             // forward, shared-basis relinearisation: digit rows and key rows, stored in tiles of 64 coefficients (the key
             // product reads all rows of a tile: whole kilobytes in one place instead of 256 bytes from every row):
             // digits [ct][r][tile][i][64], key [r][tile][i][o][64]; the sums lie in [ct][r][tile][o][64], o = (b, pair).
             // A key row is made modulo p_r from the rows of the pair's two primes while loading
             kNttDigitTile = 27, kNttKeyTile = 28,
             // decryption of few ciphertexts: the secret's row into registers too, and the product of the two rows
             kNttSecretToRegs = 29, kNttDecOwn = 30,
             kNttPlainFew = 31 };    // forward: as kNttPlain, with the stage split of the launches that leave compute units idle

// Per-thread state of TensorFused: the two transformed polynomials of the ciphertext, one limb.
template <int R>
struct TensorRegs {
  int32_t c0[R], c1[R];
};

// Per-thread state of RelinFused: the iteration (digit) and the two inner-product sums of every residue the
// thread holds after the last forward pass.
template <int R>
struct RelinRegs {
  uint32_t iter;
  int64_t s0[R], s1[R];
};
struct NoRegs {};
// Per-thread state of RelinBack: all but the last residue of every coefficient.
template <int R>
struct BackRegs {
  int32_t z[kSharedPrimes - 1][R];
  int32_t next[R];          // what the thread takes of the next row
};
// Per-thread state of CryptFused: one transformed polynomial (and, where it makes its own, the key row).
template <int R>
struct RowRegs {
  int32_t c0[R], c1[R];
};

struct NttArgs {
  const uint32_t* in;
  uint32_t* out;            // may equal `in`
  const uint32_t* aux;      // kNttStoreAdd: the addend; kNttLoadTensorMul: the second operand
  TwTable tw;
  const NttLimb* limbs;     // [L]
  FastDiv cycle;            // limbs per group of rows
  FastDiv share;            // one-kernel relinearisation: rows of a group that share a die
  uint32_t limb_base;
  FastDiv digits;           // digit loads: digits per ciphertext; kNttKeyTile, kNttBackRow: outputs (b, pair)
  uint32_t tile_words;      // tiled rows: words from one tile of a row to its next
  const RelinCrt* crt;      // kNttBack3: [k]
  RelinCrtInv crt_inv;
  const RelinPair* pair;    // kNttKeyTile: one per pair, and
  uint32_t k;               // the primes of the ciphertext (kNttBack3 too)
  uint32_t in_group_rows, in_row0;
  uint32_t out_group_rows, out_row0;
  uint32_t n_rows;          // rows of this launch (the grid may be padded, see ntt_logical_row)
  const int32_t* small;     // kNttSmallToRegs, kNttSmallKey: the signed polynomials; kNttEncOut0/1: the errors
  const uint32_t* msg;      // kNttEncOut0: the plaintexts in 32-bit or
  const uint64_t* msg64;    // 64-bit words (the other pointer is null), and
  const EncScale* scale;    // [L]
  uint32_t own_limbs;       // kNttStoreLazy with `aux` set: rows of the first own_limbs limbs of every group are read from
                            // aux, laid out [group][own_limbs][n] (a ciphertext's own limbs), the others from `in`
};

// Workgroups are handed to the 8 accelerator dies round-robin by index, and each die has its own
// L2.  The fused loads read one source row from several workgroups (a digit row feeds k transforms,
// a c0^/c1^ row feeds two tensor components); this maps the workgroup index to a row so that the
// `share` rows that read the same source run on the same die, next to each other in time.
// Rows are numbered unit*share + within for the digit load (within = j) and the caller converts
// for the tensor load.  Returns n_rows or more for the padding workgroups of the last round.
constexpr uint32_t kNttXcds = 8;
HCNN_HD uint32_t ntt_grouped_index(uint32_t bid, FastDiv share) {
  const uint32_t xcd = bid % kNttXcds, local = bid / kNttXcds, q = quot(local, share);
  return (q * kNttXcds + xcd) * share.d + (local - q * share.d);
}
inline size_t ntt_grouped_grid(size_t rows, size_t share) {
  const size_t units = rows / share;
  return (units + kNttXcds - 1) / kNttXcds * kNttXcds * share;
}

// NET consecutive words of a row from word `first`, 16 bytes at a time (rows and networks are 16-byte aligned)
template <int NET>
HCNN_HD void load_row(int32_t (&v)[NET], const uint32_t* src, uint32_t first) {
  static_assert(NET % 4 == 0, "whole 16-byte words");
#pragma unroll
  for (int e = 0; e < NET; e += 4) {
    const U4 t = ld4_at(src, (first + (uint32_t)e) * 4);
    v[e] = (int32_t)t.x; v[e + 1] = (int32_t)t.y; v[e + 2] = (int32_t)t.z; v[e + 3] = (int32_t)t.w;
  }
}

// LDS layout: one unused word after every 32, which spreads the power-of-two strides of the passes
// over the 32 banks.  The map a -> a + a/32 is additive over operands with disjoint bit fields (no
// carries), and the element e of a network sits at base | (e << LOG_TLAST) with those bits of base
// clear: its LDS word is pad(base) + pad(e << LOG_TLAST), a register plus a compile-time offset.
HCNN_HD constexpr uint32_t lds_swz(uint32_t i) { return i + (i >> 5); }
template <int LOG_TLAST>
HCNN_HD constexpr uint32_t lds_elem(uint32_t sbase, int e) {
  return sbase + lds_swz((uint32_t)e << LOG_TLAST);
}

// Stages per pass of every ring and thread shape.  The first pass takes the odd stage of an odd log2(n); every other
// pass is a whole number of radix-4 levels.  The last forward pass (the first inverse one) has every thread store (load)
// 2^ns consecutive residues: two stages there make it one 16-byte word per lane, so that the lanes of a wave touch
// consecutive words.
// PLAIN: the forward transforms of the public entry points, which only move rows.  At n = 2048 and 4096 they keep that rule
// once every compute unit has a row (four passes / three, us: 4096 rows of n = 4096 28.0 / 33.2, 1024 9.6 / 12.2, of n = 2048 6.3 / 7.0;
// 64 rows 4.5 / 4.2 and 4.0 / 3.5: kNttPlainFew).  Everything else takes a pass less there: the inverse gains nothing from the
// fourth (4096 rows 27.5 / 27.5 and 14.5 / 14.4, 4 rows 3.8 / 3.7 and 3.5 / 3.1), and inside the squaring, the encryption and
// the decryption the pass counts for more (n = 4096: 1000 squarings 621 / 593, one 29.2 / 27.0).
template <int LOGN, int LOGR, bool PLAIN = false>
struct NttGeom;
template <int LOGN, int LOGR>
struct NttGeom<LOGN, LOGR, true> : NttGeom<LOGN, LOGR, false> {};
#define HCNN_GEOM_SPEC(LOGN_, LOGR_, PLAIN_, NP_, ...)                                                \
  template <>                                                                                          \
  struct NttGeom<LOGN_, LOGR_, PLAIN_> {                                                               \
    static constexpr int N = 1 << LOGN_;                                                               \
    static constexpr int R = 1 << LOGR_;                                                               \
    static constexpr int kThreads = N / R;                                                             \
    static constexpr int kPhases = NP_;                                                                \
    static constexpr size_t kLdsBytes = (size_t)(N + N / 32) * 4;                                      \
    static constexpr int kNs[NP_] = {__VA_ARGS__};                                                     \
    static constexpr int s0(int ph) { int s = 0; for (int i = 0; i < ph; ++i) s += kNs[i]; return s; } \
    static constexpr int ns(int ph) { return kNs[ph]; }                                                \
  };
HCNN_GEOM_SPEC(10, 4, false, 3, 4, 4, 2)
HCNN_GEOM_SPEC(11, 4, false, 3, 3, 4, 4)
HCNN_GEOM_SPEC(11, 4, true, 4, 3, 4, 2, 2)
HCNN_GEOM_SPEC(12, 4, false, 3, 4, 4, 4)
HCNN_GEOM_SPEC(12, 4, true, 4, 4, 4, 2, 2)
HCNN_GEOM_SPEC(13, 4, false, 4, 3, 4, 4, 2)
HCNN_GEOM_SPEC(14, 4, false, 4, 4, 4, 4, 2)
HCNN_GEOM_SPEC(14, 5, false, 4, 4, 4, 4, 2)      // the half rows of n = 32768's two-workgroup forward transform
HCNN_GEOM_SPEC(15, 5, false, 4, 5, 4, 4, 2)
#undef HCNN_GEOM_SPEC

// Which networks a thread takes.  The first forward pass (the last inverse one) joins elements of the whole row; after it
// no stage reaches beyond 1024 consecutive residues, and those belong to one wave in every other pass (wave w of W takes the
// blocks of 1024 residues w, w + W, ...).  So only one exchange of a transform crosses waves and needs a barrier; the
// others go through LDS words that no other wave touches, which are in order by themselves.
// First network of a thread, and how far behind its elements those of network c lie (a compile-time distance whose bits are
// clear in every position of the first one: addresses are one register plus a constant).
template <class G, int PH>
HCNN_HD uint32_t first_net(int tid) {
  constexpr int NET = 1 << G::ns(PH);
  if constexpr (PH == 0 || NET >= 16) return (uint32_t)tid;
  else return wave_uniform((uint32_t)tid / 64) * (1024 / NET) + (uint32_t)tid % 64;
}
template <class G, int PH>
HCNN_HD constexpr uint32_t net_offset(int c) {
  constexpr int NET = 1 << G::ns(PH), kPerBlock = NET >= 16 ? 1 : 16 / NET;
  if (PH == 0) return (uint32_t)(G::kThreads * c);
  return (uint32_t)(G::kThreads * 16 * (c / kPerBlock) + c % kPerBlock * 64 * NET);
}

// Two Cooley-Tukey stages on (x0, x1, x2, x3): pairs (0,2), (1,3) with W, then (0,1) with V and (2,3) with U.
// Twiddles c are centred and carry 2^32, so sredc(c * x) is the product: |sum of two products| <= p |x|max, which the
// reduction brings to p |x|max / 2^32 + p/2 <= p for any 32-bit x; every output is a sum or difference of two: in (-2p, 2p).
HCNN_HD void r4_fwd(int32_t& x0, int32_t& x1, int32_t& x2, int32_t& x3, const R4Twiddle& t, int32_t nuw, const NttLimb& L) {
  const uint32_t p = L.m.p;
  const int64_t e = (int64_t)x0 * L.rc;
  const int32_t A = sredc(e + (int64_t)x2 * t.w, p, L.pinv);
  const int32_t C = sredc(e + (int64_t)x2 * (L.zero - t.w), p, L.pinv);
  const int32_t P = sredc((int64_t)x1 * t.v + (int64_t)x3 * t.vw, p, L.pinv);
  const int32_t Q = sredc((int64_t)x1 * t.u + (int64_t)x3 * nuw, p, L.pinv);
  x0 = A + P;
  x1 = A - P;
  x2 = C + Q;
  x3 = C - Q;
}

// Two Gentleman-Sande stages: pairs (0,1) with V and (2,3) with U, then (0,2), (1,3) with W (inverse twiddles).
// c0 is the constant of the untwisted output (2^32, or the scaling of the last level).  With |x| <= p the sums and differences
// fit 32 bits, two products of them stay below 2 p^2 and every output in (-p, p).
HCNN_HD void r4_inv(int32_t& x0, int32_t& x1, int32_t& x2, int32_t& x3, int32_t c0, const R4Twiddle& t, int32_t nuw, const NttLimb& L) {
  const uint32_t p = L.m.p;
  const int32_t s1 = x0 + x1, d1 = x0 - x1, s2 = x2 + x3, d2 = x2 - x3;
  // (untraced: the compiler would factor c0 out, into a 64-bit sum and a 64-bit product)
  x0 = sredc(untraced((int64_t)s1 * c0) + (int64_t)s2 * c0, p, L.pinv);
  x1 = sredc((int64_t)d1 * t.v + (int64_t)d2 * t.u, p, L.pinv);
  x2 = sredc((int64_t)s1 * t.w + (int64_t)s2 * (L.zero - t.w), p, L.pinv);
  x3 = sredc((int64_t)d1 * t.vw + (int64_t)d2 * nuw, p, L.pinv);
}

// The same with something added to every output before its reduction (three 64-bit products of a 32-bit value and a centred
// constant at most: together with the two products below 6 * 2^60, outputs in (-2p, 2p)).
HCNN_HD void r4_inv_add(int32_t& x0, int32_t& x1, int32_t& x2, int32_t& x3, int32_t c0, const R4Twiddle& t, int32_t nuw,
                        const int64_t (&add)[4], const NttLimb& L) {
  const uint32_t p = L.m.p;
  const int32_t s1 = x0 + x1, d1 = x0 - x1, s2 = x2 + x3, d2 = x2 - x3;
  x0 = sredc(untraced(add[0] + (int64_t)s1 * c0) + (int64_t)s2 * c0, p, L.pinv);
  x1 = sredc(untraced(add[1] + (int64_t)d1 * t.v) + (int64_t)d2 * t.u, p, L.pinv);
  x2 = sredc(untraced(add[2] + (int64_t)s1 * t.w) + (int64_t)s2 * (L.zero - t.w), p, L.pinv);
  x3 = sredc(untraced(add[3] + (int64_t)d1 * t.vw) + (int64_t)d2 * nuw, p, L.pinv);
}

// Workgroup index of the split forms -> half and row (both halves of a row on one die, next to each other in time).
HCNN_HD uint32_t split_half(uint32_t bid) { return (bid / kNttXcds) & 1u; }
HCNN_HD uint32_t split_row(uint32_t bid) { return bid / (2 * kNttXcds) * kNttXcds + bid % kNttXcds; }
inline size_t split_grid(size_t rows) { return 2 * ((rows + kNttXcds - 1) / kNttXcds * kNttXcds); }

// ------------------------------------------------------------------------- forward
// SPLIT = 1: two workgroups per row.  The first stage of the forward transform pairs element i with element
// i + n/2 and leaves two halves that never meet again; workgroup (row, half) computes its half of that stage while
// loading (it reads both halves of the row, the second reader out of L2) and then runs the remaining log2(n) - 1
// stages on n/2 residues.  Half the LDS and half the threads per workgroup: for the largest ring, whose whole row
// fills the LDS of a compute unit, two workgroups fit where one did, and they are out of step with each other.
template <int LOGN, int LOGR, int IO = kNttPlain, int SPLIT = 0>
struct NttFwd {
  static constexpr bool kFused = IO == kNttFusedMac || IO == kNttFusedMac16 || IO == kNttFusedMacAny;
  static constexpr bool kRowToRegs = IO == kNttSmallToRegs || IO == kNttCtToRegs || IO == kNttSecretToRegs;
  static constexpr bool kToRegs = IO == kNttToRegs0 || IO == kNttToRegs1 || kRowToRegs;
  static constexpr bool kSmallIn = IO == kNttSmallToRegs || IO == kNttSmallKey || IO == kNttSecretToRegs;
  static constexpr bool kKeyOut = IO == kNttStoreKey || IO == kNttSmallKey || IO == kNttKeyTile;
  static constexpr bool kTileOut = IO == kNttDigitTile || IO == kNttKeyTile;
  static constexpr bool kDigitRow = IO == kNttLoadDigit || IO == kNttDigitTile;
  static_assert(IO == kNttPlain || IO == kNttPlainFew || kDigitRow || IO == kNttStoreLazy || kKeyOut || kFused || kToRegs,
                "forward NTT: plain, digit load, lazy or key store, fused inner product or register output");
  static_assert(SPLIT == 0 || (SPLIT == 1 && !kFused && IO != kNttSmallToRegs && LOGN % 2 == 1),
                "the split form stores its rows or keeps them for the tensor or the decryption");
  using G = NttGeom<LOGN - SPLIT, LOGR, IO == kNttPlain>;      // the stages after the split one
  static constexpr int kThreads = G::kThreads;
  static constexpr int kPhases = G::kPhases;
  static constexpr bool kDigitIn = kDigitRow || kFused;
  using Regs = std::conditional_t<kFused, RelinRegs<G::R>, std::conditional_t<kRowToRegs, RowRegs<G::R>, std::conditional_t<kToRegs, TensorRegs<G::R>, NoRegs>>>;
  // A whole row of n = 32768 in one workgroup (the public transform, in place): the two blocks of a wave lie further apart than the 64 KiB
  // that an LDS instruction's offset reaches, so that every network has addresses of its own, and the last pass hands its networks out
  // across the workgroup again, which stores 16 KiB in one piece, behind a second barrier (us, as the other rings / this; the first part
  // alone, the second: 400 polynomials of 12 limbs 376 / 341; 358, 355; 128 of 18 182 / 174; 176, 181; 10 of 24 19.8 / 18.2; 19.0, 19.0).
  static constexpr bool kWholeRow = LOGN == 15 && SPLIT == 0 && !kFused && !kToRegs;
  // one exchange across waves (first_net), the first
  static constexpr bool wave_sync(int ph) { return ph != 0 && !(kWholeRow && ph == kPhases - 2); }
  // workgroups of a launch over `slots` row positions (a multiple of the die count for the split form)
  static size_t grid(size_t slots) { return SPLIT ? split_grid(slots) : slots; }

  template <int PH>
  HCNN_HD static void phase(const NttArgs& a, unsigned bid, int tid, uint32_t* lds, Regs& regs) {
    constexpr int N = 1 << LOGN, R = G::R;                 // N: residues of a row in memory
    constexpr int LOGM = LOGN - SPLIT;                     // stages S0 .. of this workgroup run on 2^LOGM residues
    constexpr int S0 = G::s0(PH), NS = G::ns(PH), NET = 1 << NS, C = R / NET;
    constexpr int LOG_TLAST = LOGM - S0 - NS, TLAST = 1 << LOG_TLAST;
    constexpr bool kFirst = PH == 0, kLast = PH == kPhases - 1;
    constexpr bool kOdd = NS % 2 == 1;                     // one radix-2 stage, at the root of the whole tree
    static_assert(!kOdd || (kFirst && !SPLIT), "only the root stage is taken alone");
    if constexpr (kFused || kToRegs) tid = opaque(tid);

    uint32_t half = 0;
    if constexpr (SPLIT) {
      // both halves of a row on one die, next to each other in time
      half = split_half(bid);
      bid = split_row(bid);
      if constexpr (!kDigitIn && !kRowToRegs) {
        if (bid >= a.n_rows) return;                       // padding workgroups of the last round
      }
    }
    if constexpr (kDigitIn || kRowToRegs) {
      bid = ntt_grouped_index(bid, kFused ? a.share : a.cycle);      // the k transforms of one digit row (or small row) share a die
      if (bid >= a.n_rows) return;
    }
    const uint32_t group = quot(bid, a.cycle), within = bid - group * a.cycle.d, limb = a.limb_base + within;
    const NttLimb L = ldc(a.limbs, limb);
    const uint32_t p = L.m.p;
    const R4Twiddle* tq = a.tw.quad + (size_t)limb * (N / 2);
    const int32_t* tn = a.tw.nuw + (size_t)limb * (N / 2);
    const uint32_t* gin;
    uint32_t* gout = nullptr;
    const uint32_t* gin_pair = nullptr;   // kNttKeyTile: the row of the pair's second prime, and its constants
    int32_t pair_inv = 0, pair_q = 0;
    uint32_t pair_p = 0, pair_pinv = 0;
    const uint32_t* key0 = nullptr;       // kNttFusedMac: evk^[iter][0][j]; component 1 lies k rows further
    if constexpr (kFused) {
      const uint32_t kk = a.cycle.d;                   // rows are (ct, j)
      gin = a.in + ((size_t)group * 3 * kk + 2 * kk + regs.iter) * N;
      key0 = a.aux + ((size_t)regs.iter * 2 * kk + limb) * N;
      if (kFirst && regs.iter == 0) {
#pragma unroll
        for (int r = 0; r < R; ++r) { regs.s0[r] = 0; regs.s1[r] = 0; }
      }
    } else if constexpr (kDigitRow) {
      const uint32_t kk = a.digits.d, ct = quot(group, a.digits);     // group = (ct, digit)
      gin = a.in + ((size_t)ct * 3 * kk + 2 * kk + (group - ct * kk)) * N;
    } else if constexpr (kSmallIn) {
      gin = reinterpret_cast<const uint32_t*>(a.small) + (IO == kNttSecretToRegs ? 0 : (size_t)group * N);
    } else if constexpr (IO == kNttKeyTile) {
      const uint32_t outs = a.digits.d, i = quot(group, a.digits), o = group - i * outs;          // group = (digit, b, pair)
      const uint32_t b = o >= outs / 2 ? 1u : 0u, j0 = 2 * (o - b * (outs / 2)), j1 = j0 + 1 < a.k ? j0 + 1 : j0;
      gin = a.in + ((size_t)(i * 2 + b) * a.k + j0) * N;
      gin_pair = gin + (size_t)(j1 - j0) * N;
      if constexpr (kFirst) {
        const NttLimb Q = ldc(a.limbs, j1);
        pair_inv = ldc(&a.pair[j0 / 2].inv, 0); pair_q = ldc(a.pair[j0 / 2].q, a.out_row0); pair_p = Q.m.p; pair_pinv = Q.pinv;
      }
    } else if constexpr (IO == kNttCtToRegs) {
      gin = a.in + ((size_t)(group * 2 + 1) * a.cycle.d + within) * N;
    } else if constexpr (kToRegs) {
      // workgroup (ct, l): polynomial c0 or c1 of the ciphertext; its own limbs come from the ciphertext (`aux`,
      // [ct][2][own_limbs][n]), the auxiliary limbs from the extension buffer (`in`, [ct][2][L][n])
      const uint32_t LL = a.cycle.d, poly = IO == kNttToRegs1 ? 1u : 0u;
      const size_t grp = (size_t)group * 2 + poly;
      if (bid >= a.n_rows) return;
      gin = limb < a.own_limbs ? a.aux + (grp * a.own_limbs + limb) * N : a.in + (grp * LL + limb) * N;
    } else {
      gin = a.in + ((size_t)group * a.in_group_rows + a.in_row0 + within) * N;
      if constexpr (IO == kNttStoreLazy) {
        if (a.aux != nullptr && within < a.own_limbs) gin = a.aux + ((size_t)group * a.own_limbs + within) * N;
      }
    }
    if constexpr (IO == kNttDigitTile) {
      const uint32_t kk = a.digits.d, ct = quot(group, a.digits);
      gout = a.out + (size_t)(ct * kSharedPrimes + within) * (N / 64) * a.tile_words + (group - ct * kk) * 64;
    } else if constexpr (IO == kNttKeyTile) {
      gout = a.out + (size_t)a.out_row0 * (N / 64) * a.tile_words + (size_t)group * 64;
    } else if constexpr (!kFused && !kToRegs)
      gout = a.out + ((size_t)group * a.out_group_rows + a.out_row0 + within) * N + (size_t)half * (N / 2);

    // The radix-2 stage of node 1 on rows with residues in [0, 2^30) (canonical ones, or digits of another prime): |T| is below
    // 2^30 / 8 + p / 2, X + T and X - T stay within 1.63 * 2^30 and the stage needs no other reduction.  Small signed values
    // (any 32 bits) are reduced on the X side; the T side and the radix-4 levels take them as they are.
    // split form: this half's output of the pair (i, i + n/2), on the way in.
    auto root_x = [&](int32_t x) -> int32_t { return kSmallIn ? sredc((int64_t)x * L.rc, p, L.pinv) : x; };
    auto load_word = [&](uint32_t at, uint32_t e_off) -> int32_t {       // element at + e_off, e_off uniform
      const int32_t x = (int32_t)ld_at(gin + e_off, at * 4);
      if constexpr (kFirst && IO == kNttKeyTile) {
        // |x rc| and |t q| are below 2^59: the value lies in (-p, p)
        const int32_t t = sredc((int64_t)((int32_t)ld_at(gin_pair + e_off, at * 4) - x) * pair_inv, pair_p, pair_pinv);
        return sredc((int64_t)x * L.rc + (int64_t)t * pair_q, p, L.pinv);
      } else {
        return x;
      }
    };
    auto load_first = [&](uint32_t at, uint32_t e_off) -> int32_t {
      const int32_t x = load_word(at, e_off);
      if constexpr (SPLIT) {
        const int32_t X = root_x(x), T = sredc((int64_t)load_word(at, e_off + N / 2) * L.w1, p, L.pinv);
        return half ? X - T : X + T;
      } else {
        return x;
      }
    };

    constexpr bool kAcross = kWholeRow && kLast;
    const uint32_t nu = kAcross ? (uint32_t)tid : first_net<G, PH>(tid), o = nu & (TLAST - 1);
    uint32_t i0 = nu >> LOG_TLAST;
    if constexpr (TLAST >= 64) i0 = wave_uniform(i0);               // (scalar twiddle loads)
    const uint32_t base0 = i0 * (uint32_t)(NET * TLAST) + o;        // network 0: element e at base0 + e*TLAST
    // node of the twiddle tree over the whole row (network 0): the half's own sub-tree in the split form
    const uint32_t root0 = SPLIT ? ((2u + half) << S0) + i0 : (1u << S0) + i0;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      // network c lies `far` behind network 0: a compile-time distance of every access (off), or part of its own addresses
      const uint32_t far = kAcross ? (uint32_t)(kThreads * NET * c) : net_offset<G, PH>(c);
      const uint32_t off = kWholeRow ? 0 : far, i_off = off / (NET * TLAST);
      const uint32_t base = base0 + (far - off), sbase = lds_swz(base), root = root0 + (far - off) / (NET * TLAST);
      int32_t v[NET];
#pragma unroll
      for (int e = 0; e < NET; ++e)
        v[e] = kFirst ? load_first(base, off + (uint32_t)e * TLAST) : (int32_t)lds[lds_elem<LOG_TLAST>(sbase, e) + lds_swz(off)];
      if constexpr (kOdd) {
#pragma unroll
        for (int x = 0; x < NET / 2; ++x) {
          const int32_t X = root_x(v[x]), T = sredc((int64_t)v[x + NET / 2] * L.w1, p, L.pinv);
          v[x] = X + T;
          v[x + NET / 2] = X - T;
        }
      }
#pragma unroll
      for (int l = kOdd ? 1 : 0; l < NS; l += 2) {
        const int q = NET >> (l + 2);
#pragma unroll
        for (int h = 0; h < (1 << l); ++h) {
          const R4Twiddle t = ldc_at(tq + h + (i_off << l), (root << l) * 16);
          const int32_t nuw = ldc_at(tn + h + (i_off << l), (root << l) * 4);
#pragma unroll
          for (int x = 0; x < q; ++x) {
            const int b = h * 4 * q + x;
            r4_fwd(v[b], v[b + q], v[b + 2 * q], v[b + 3 * q], t, nuw, L);
          }
        }
      }
      if constexpr (kLast && kFused) {
        // The transformed digit times the key rows (|key| <= p/2), added to the 64-bit sums.  With the digit as it is, in
        // (-2p, 2p), 8 products stay below 8 p^2 < 2^63 (kNttFusedMac, k <= 8); brought into [-p, p), 16 products do
        // (kNttFusedMac16, k <= 16), and kNttFusedMacAny folds the sums to 2^60 (two products) before digits 16, 29, 42, ...
        const uint32_t* key1 = key0 + (size_t)a.cycle.d * N;
        int32_t e0[NET], e1[NET];
        load_row<NET>(e0, key0 + off, base);
        load_row<NET>(e1, key1 + off, base);
        if constexpr (IO == kNttFusedMacAny) {
          if (regs.iter >= 16 && (regs.iter - 16) % 13 == 0) {
#pragma unroll
            for (int e = 0; e < NET; ++e) {
              regs.s0[c * NET + e] = sfold(regs.s0[c * NET + e], L.rc);
              regs.s1[c * NET + e] = sfold(regs.s1[c * NET + e], L.rc);
            }
          }
        }
#pragma unroll
        for (int e = 0; e < NET; ++e) {
          const int32_t d = IO == kNttFusedMac ? v[e] : half_range(v[e], p);
          regs.s0[c * NET + e] += (int64_t)d * e0[e];
          regs.s1[c * NET + e] += (int64_t)d * e1[e];
        }
      } else if constexpr (kLast && kToRegs) {
#pragma unroll
        for (int e = 0; e < NET; ++e) {
          if constexpr (IO == kNttToRegs1 || IO == kNttSecretToRegs) regs.c1[c * NET + e] = half_range(v[e], p);
          else                             regs.c0[c * NET + e] = half_range(v[e], p);
        }
      } else if constexpr (kLast) {
        static_assert(!kLast || TLAST == 1, "the last pass holds consecutive residues");
        uint32_t r[NET];
#pragma unroll
        for (int e = 0; e < NET; ++e) {
          if constexpr (IO == kNttStoreLazy || kDigitRow) r[e] = (uint32_t)half_range(v[e], p);
          else if constexpr (kKeyOut) {
            const uint32_t x = canon_p(sredc((int64_t)v[e] * L.key_scale, p, L.pinv), p);
            r[e] = x > p / 2 ? x - p : x;
          } else r[e] = canon_2p(v[e], p);
        }
#pragma unroll
        for (int e = 0; e < NET; e += 4) {
          U4 t;
          t.x = r[e]; t.y = r[e + 1]; t.z = r[e + 2]; t.w = r[e + 3];
          if constexpr (kTileOut)
            st4_at(gout + (size_t)((off + (SPLIT ? half * (N / 2) : 0)) / 64) * a.tile_words + e, ((base >> 6) * a.tile_words + (base & 63u)) * 4, t);
          else
            st4_at(gout + off + e, base * 4, t);
        }
      } else {
#pragma unroll
        for (int e = 0; e < NET; ++e) lds[lds_elem<LOG_TLAST>(sbase, e) + lds_swz(off)] = (uint32_t)v[e];
      }
    }
  }
};

// ------------------------------------------------------------------------- inverse
// SPLIT = 1 (odd log2(n)): two workgroups per row, all stages but the last, a single one that joins the halves: the reader of the row takes it while
// loading (split_root).  The halves are left signed in (-p, p), without the output scaling.  Half the LDS and half the threads per
// workgroup, as in the forward transform, and (n = 32768) no pass of five stages.
template <int LOGN, int LOGR, int IO = kNttPlain, int SPLIT = 0>
struct NttInv {
  static_assert(SPLIT == 0 || (SPLIT == 1 && LOGN % 2 == 1 && (IO == kNttLoadTensor || IO == kNttLoadTensorMul || IO == kNttTensorRegs0 ||
                IO == kNttTensorRegs1 || IO == kNttTensorRegs2 || IO == kNttBackRow || IO == kNttDecOwn)),
                "rows whose reader takes the last stage");
  static_assert(IO == kNttPlain || IO == kNttLoadTensor || IO == kNttStoreAdd || IO == kNttLoadTensorMul ||
                IO == kNttFromRegs0 || IO == kNttFromRegs1 || IO == kNttTensorRegs0 || IO == kNttTensorRegs1 ||
                IO == kNttTensorRegs2 || IO == kNttEncOut0 || IO == kNttEncOut1 || IO == kNttDecOut || IO == kNttDecOwn || IO == kNttBackRow || IO == kNttBack0 ||
                IO == kNttBack1 || IO == kNttBack2 || IO == kNttBack3, "inverse NTT io mode");
  using G = NttGeom<LOGN - SPLIT, LOGR>;
  static constexpr int kThreads = G::kThreads;
  static constexpr int kPhases = G::kPhases;
  // workgroups of a launch over `rows` rows, or of three components of rows / 3 pairs
  static size_t grid(size_t rows) {
    if (IO == kNttLoadTensor || IO == kNttLoadTensorMul) return ntt_grouped_grid(rows, 3) << SPLIT;
    return SPLIT ? split_grid(rows) : rows;
  }
  // a 1024-thread workgroup whose row leaves LDS for a second one: keep the registers within what two of them need
  // (the plain transform of n = 16384 took 68 and ran alone on its compute unit, a third slower per row)
  static constexpr int kMinWavesPerSimd = SPLIT ? 4 : (G::kThreads == 1024 && 2 * G::kLdsBytes <= 160 * 1024) ? 8 : 1;
  static constexpr bool wave_sync(int ph) { return ph != kPhases - 2; }        // one exchange across waves (first_net)
  static constexpr bool kFromRegs = IO == kNttFromRegs0 || IO == kNttFromRegs1;
  static constexpr bool kTensorRegs = IO == kNttTensorRegs0 || IO == kNttTensorRegs1 || IO == kNttTensorRegs2;
  static constexpr bool kBack = IO == kNttBack0 || IO == kNttBack1 || IO == kNttBack2 || IO == kNttBack3;
  static constexpr int kBackRow = IO == kNttBack3 ? 3 : IO - kNttBack0;
  static constexpr bool kEncOut = IO == kNttEncOut0 || IO == kNttEncOut1, kDecOut = IO == kNttDecOut || IO == kNttDecOwn, kKeyRegs = kEncOut || kDecOut;
  using Regs = std::conditional_t<kFromRegs, RelinRegs<G::R>, std::conditional_t<kTensorRegs, TensorRegs<G::R>,
               std::conditional_t<kKeyRegs, RowRegs<G::R>, std::conditional_t<kBack, BackRegs<G::R>, NoRegs>>>>;

  template <int PHI>
  HCNN_HD static void phase(const NttArgs& a, unsigned bid, int tid, uint32_t* lds, Regs& regs) {
    constexpr int PH = kPhases - 1 - PHI;   // mirrors forward pass PH
    constexpr int N = 1 << LOGN, R = G::R;                // N: residues of a row in memory
    constexpr int S0 = G::s0(PH), NS = G::ns(PH), NET = 1 << NS, C = R / NET;
    constexpr int LOG_TLAST = LOGN - SPLIT - S0 - NS, TLAST = 1 << LOG_TLAST;
    constexpr bool kFirst = PHI == 0, kLast = PHI == kPhases - 1;   // kLast <=> S0 == 0
    constexpr bool kOdd = NS % 2 == 1;

    uint32_t half = 0;
    if constexpr (SPLIT && IO != kNttLoadTensor && IO != kNttLoadTensorMul) {
      half = split_half(bid);
      bid = split_row(bid);
      if constexpr (!kKeyRegs) {
        if (bid >= a.n_rows) return;
      }
    }
    if constexpr (IO == kNttLoadTensor || IO == kNttLoadTensorMul) {
      // the three components of one (ciphertext, limb) pair read the same c0^ / c1^ rows: same die
      const uint32_t LL = a.cycle.d;
      const uint32_t xcd = bid % kNttXcds;
      uint32_t local = bid / kNttXcds;
      if constexpr (SPLIT) {
        // (the halves of a pair one after the other: they share nothing)
        half = local / 3 & 1u;
        local = local / 6 * 3 + local % 3;
      }
      const uint32_t unit = local / 3 * kNttXcds + xcd, b = local % 3, ct = quot(unit, a.cycle);   // unit = ct*L + l
      bid = (ct * 3 + b) * LL + (unit - ct * LL);               // row (ct, b, l)
      if (unit >= a.n_rows / 3) return;
    }
    if constexpr (kFromRegs || kKeyRegs) {
      if constexpr (kKeyRegs) tid = opaque(tid);
      bid = ntt_grouped_index(bid, kFromRegs ? a.share : a.cycle);   // the same workgroup -> (ct, j) map as the forward transforms
      if (bid >= a.n_rows) return;
    }
    if constexpr (kTensorRegs) {
      tid = opaque(tid);
      if (bid >= a.n_rows) return;
    }
    const uint32_t unit_ct = kBack ? quot(bid, a.digits) : 0, unit_o = bid - unit_ct * a.digits.d;     // RelinBack: (ct, o)
    if constexpr (kBack) {
      tid = opaque(tid);
      bid = bid * kSharedPrimes + kBackRow;            // row (ct, o, r)
    }
    const uint32_t group = quot(bid, a.cycle), within = bid - group * a.cycle.d, limb = a.limb_base + within;
    const NttLimb L = ldc(a.limbs, limb);
    const uint32_t p = L.m.p;
    const R4Twiddle* tq = a.tw.quad + (size_t)limb * (N / 2);
    const int32_t* tn = a.tw.nuw + (size_t)limb * (N / 2);
    const uint32_t* gin = nullptr;
    const uint32_t* gin2 = nullptr;       // kNttLoadTensor: the c1^ row
    uint32_t comp = 0;                    // kNttLoadTensor: tensor component b
    const uint32_t* gmul0 = nullptr;      // kNttLoadTensorMul: rows c0^, c1^ of the first operand and
    const uint32_t* gmul1 = nullptr;      // c0'^, c1'^ of the second
    if constexpr (IO == kNttLoadTensor) {
      const uint32_t LL = a.cycle.d, ct = group / 3;
      comp = group % 3;
      gin2 = a.in + ((size_t)(ct * 2 + 1) * LL + within) * N;       // c1^
      gin = comp == 2 ? gin2 : gin2 - (size_t)LL * N;                 // c0^ unless b = 2
    } else if constexpr (IO == kNttLoadTensorMul) {
      const uint32_t LL = a.cycle.d, ct = group / 3;
      comp = group % 3;
      const size_t row0 = ((size_t)ct * 2 * LL + within) * N;        // component 0 of this limb
      gmul0 = a.in + row0;
      gmul1 = a.aux + row0;
      // b = 0: c0*c0' ; b = 2: c1*c1' ; b = 1: c0*c1' + c1*c0'
      gin = gmul0 + (comp == 2 ? (size_t)LL * N : 0);
      gin2 = gmul1 + (comp == 0 ? 0 : (size_t)LL * N);
    } else if constexpr (kKeyRegs && IO != kNttDecOwn) {
      gin = a.in + ((IO == kNttEncOut1 ? (size_t)a.cycle.d : 0) + within) * N;      // key row of this limb
    } else if constexpr (IO == kNttBackRow || kBack) {
      const uint32_t ct = kBack ? unit_ct : quot(group, a.digits), o = group - ct * a.digits.d;
      gin = a.in + (size_t)(ct * kSharedPrimes + within) * (N / 64) * a.tile_words + o * 64;
    } else if constexpr (!kFromRegs && !kTensorRegs && !kKeyRegs) {
      gin = a.in + ((size_t)group * a.in_group_rows + a.in_row0 + within) * N;
    }
    uint32_t* gout;
    const uint32_t* gaux = nullptr;
    if constexpr (kFromRegs) {
      const uint32_t kk = a.cycle.d, b = IO == kNttFromRegs1 ? 1u : 0u;
      gout = a.out + ((size_t)(group * 2 + b) * kk + within) * N;
      gaux = a.aux + ((size_t)(group * 3 + b) * kk + within) * N;
    } else if constexpr (kTensorRegs) {
      const uint32_t LL = a.cycle.d, b = IO == kNttTensorRegs0 ? 0u : (IO == kNttTensorRegs1 ? 1u : 2u);
      gout = a.out + ((size_t)(group * 3 + b) * LL + within) * N;       // d row (ct, b, l)
    } else if constexpr (kEncOut) {
      gout = a.out + ((size_t)(group * 2 + (IO == kNttEncOut1 ? 1 : 0)) * a.cycle.d + within) * N;
    } else if constexpr (kBack) {
      // o = (b, pair), a.digits of them: result and y row (ct, b, j) of the pair's first prime
      const uint32_t b = unit_o >= a.digits.d / 2 ? 1u : 0u, j = 2 * (unit_o - b * (a.digits.d / 2));
      gout = a.out + ((size_t)(unit_ct * 2 + b) * a.k + j) * N;
      gaux = a.aux + ((size_t)(unit_ct * 3 + b) * a.k + j) * N;
    } else if constexpr (kDecOut) {
      gout = a.out + (size_t)bid * N;
      gaux = a.aux + ((size_t)group * 2 * a.cycle.d + within) * N;                   // c0
    } else {
      gout = a.out + ((size_t)group * a.out_group_rows + a.out_row0 + within) * N;
    }
    if constexpr (SPLIT) {
      const size_t at = (size_t)half * (N / 2);
      gout += at;
      if constexpr (IO == kNttBackRow) gin += at / 64 * a.tile_words;
      else if constexpr (!kTensorRegs && IO != kNttDecOwn) gin += at;
      if constexpr (IO == kNttLoadTensor || IO == kNttLoadTensorMul) gin2 += at;
      if constexpr (IO == kNttLoadTensorMul) { gmul0 += at; gmul1 += at; }
    }
    if constexpr (IO == kNttStoreAdd) {
      const uint32_t kk = a.cycle.d;
      gaux = a.aux + ((size_t)(group / 2) * 3 * kk + (size_t)(group % 2) * kk + within) * N;
    }

    const uint32_t nu = first_net<G, PH>(tid), o = nu & (TLAST - 1);
    uint32_t i0 = nu >> LOG_TLAST;
    if constexpr (TLAST >= 64) i0 = wave_uniform(i0);
    const uint32_t base = i0 * (uint32_t)(NET * TLAST) + o;
    const uint32_t sbase = lds_swz(base);
    const uint32_t root = SPLIT ? ((2u + half) << S0) + i0 : (1u << S0) + i0;
    if constexpr (kLast && kBack && IO != kNttBack3) {
      // the next row's words are on their way during this row's last pass
      constexpr int F = kPhases - 1, NET_F = 1 << G::ns(F);
      const uint32_t first = first_net<G, F>(tid) * NET_F;
      const uint32_t* next = gin + (size_t)(N / 64) * a.tile_words;
#pragma unroll
      for (int c = 0; c < R / NET_F; ++c) {
        int32_t w[NET_F];
        load_row<NET_F>(w, next + (size_t)(net_offset<G, F>(c) / 64) * a.tile_words, (first >> 6) * a.tile_words + (first & 63u));
#pragma unroll
        for (int e = 0; e < NET_F; ++e) regs.next[c * NET_F + e] = w[e];
      }
      sched_fence();
    }
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const uint32_t off = net_offset<G, PH>(c), i_off = off / (NET * TLAST);
      int32_t v[NET];
      static_assert(!kFirst || TLAST == 1, "the first pass holds consecutive residues");
      if constexpr (kFirst && kFromRegs) {
        // the sums sit where the last forward pass left its residues, which is where this pass takes them; the key
        // carries the factor 2^32 of the reduction.  |sfold| / 2^32 + p/2 <= p
#pragma unroll
        for (int e = 0; e < NET; ++e)
          v[e] = sredc(sfold(IO == kNttFromRegs1 ? regs.s1[c * NET + e] : regs.s0[c * NET + e], L.rc), p, L.pinv);
      } else if constexpr (kFirst && kTensorRegs) {
        // c0^*c0^, 2*c0^*c1^ or c1^*c1^ from the registers of the two forward transforms (values in [-p, p)); products
        // carry the factor 2^-32 of the reduction and stay in (-p, p)
#pragma unroll
        for (int e = 0; e < NET; ++e) {
          const int32_t x = untraced(IO == kNttTensorRegs2 ? regs.c1[c * NET + e] : regs.c0[c * NET + e]);
          const int32_t y = IO == kNttTensorRegs1 ? untraced(regs.c1[c * NET + e]) : x;
          v[e] = sredc((int64_t)(IO == kNttTensorRegs1 ? untraced(x + x) : x) * y, p, L.pinv);
        }
      } else if constexpr (kFirst && IO == kNttDecOwn) {
        // two plain rows: the product carries 2^-32, which the output scaling takes out
#pragma unroll
        for (int e = 0; e < NET; ++e)
          v[e] = sredc((int64_t)untraced(regs.c0[c * NET + e]) * untraced(regs.c1[c * NET + e]), p, L.pinv);
      } else if constexpr (kFirst && kKeyRegs) {
        // |row| <= p, |key| <= p/2: products stay within (-p, p)
        int32_t y[NET];
        load_row<NET>(y, gin + off, base);
#pragma unroll
        for (int e = 0; e < NET; ++e) v[e] = sredc((int64_t)untraced(regs.c0[c * NET + e]) * y[e], p, L.pinv);
      } else if constexpr (kFirst && kBack && IO != kNttBack0) {
#pragma unroll
        for (int e = 0; e < NET; ++e) v[e] = regs.next[c * NET + e];
      } else if constexpr (kFirst && (IO == kNttBackRow || kBack)) {
        load_row<NET>(v, gin + (size_t)(off / 64) * a.tile_words, (base >> 6) * a.tile_words + (base & 63u));
      } else if constexpr (kFirst) {
        load_row<NET>(v, gin + off, base);
        if constexpr (IO == kNttLoadTensorMul) {
          // v = c0^ (b = 0, 1) or c1^ (b = 2);  y = c0'^ (b = 0) or c1'^ (b = 1, 2); all in [-p, p).  The cross term is
          // summed in 64 bits
          int32_t y[NET];
          load_row<NET>(y, gin2 + off, base);
          if (comp == 1) {                 // + c1^ * c0'^
            int32_t u[NET], w[NET];
            load_row<NET>(u, gmul0 + (size_t)a.cycle.d * N + off, base);
            load_row<NET>(w, gmul1 + off, base);
#pragma unroll
            for (int e = 0; e < NET; ++e) v[e] = sredc((int64_t)v[e] * y[e] + (int64_t)u[e] * w[e], p, L.pinv);
          } else {
#pragma unroll
            for (int e = 0; e < NET; ++e) v[e] = sredc((int64_t)v[e] * y[e], p, L.pinv);
          }
        }
        if constexpr (IO == kNttLoadTensor) {
          // gin was pointed at c0^ (b = 0, 1) or c1^ (b = 2); only b = 1 needs the second row.  Products carry the
          // factor 2^-32 of the reduction
          if (comp == 1) {
            int32_t y[NET];
            load_row<NET>(y, gin2 + off, base);
#pragma unroll
            for (int e = 0; e < NET; ++e) v[e] = sredc((int64_t)(v[e] + v[e]) * y[e], p, L.pinv);
          } else {
#pragma unroll
            for (int e = 0; e < NET; ++e) v[e] = sredc((int64_t)v[e] * v[e], p, L.pinv);
          }
        }
      } else {
#pragma unroll
        for (int e = 0; e < NET; ++e) v[e] = (int32_t)lds[lds_elem<LOG_TLAST>(sbase, e) + lds_swz(off)];
      }
      constexpr bool kMont = IO == kNttLoadTensor || IO == kNttLoadTensorMul || kTensorRegs || IO == kNttDecOwn;
      constexpr bool kZ = IO == kNttBackRow || kBack;
      const InvRoot& top = kMont ? L.inv_r : kZ ? L.inv_z : L.inv;       // node 1: the output scaling folded in
#pragma unroll
      for (int l = NS - 2; l >= (kOdd ? 1 : kLast && kEncOut ? 2 : 0); l -= 2) {
        const int q = NET >> (l + 2);
#pragma unroll
        for (int h = 0; h < (1 << l); ++h) {
          const bool outer = kLast && l == 0 && !SPLIT;
          const R4Twiddle t = outer ? R4Twiddle{top.w, top.v, top.vw, top.u} : ldc_at(tq + h + (i_off << l), (root << l) * 16);
          const int32_t nuw = outer ? top.nuw : ldc_at(tn + h + (i_off << l), (root << l) * 4), c0 = outer ? top.c0 : L.rc;
#pragma unroll
          for (int x = 0; x < q; ++x) {
            const int b = h * 4 * q + x;
            r4_inv(v[b], v[b + q], v[b + 2 * q], v[b + 3 * q], c0, t, nuw, L);
          }
        }
      }
      if constexpr (kOdd && !(kLast && kEncOut)) {
        static_assert(!kOdd || kLast, "only the root stage is taken alone");
#pragma unroll
        for (int x = 0; x < NET / 2; ++x) {
          const int32_t X = v[x], Y = v[x + NET / 2];
          v[x] = sredc((int64_t)(X + Y) * top.c0, p, L.pinv);
          v[x + NET / 2] = sredc((int64_t)(X - Y) * top.w, p, L.pinv);
        }
      }
      if constexpr (kLast && kBack && IO != kNttBack3) {
#pragma unroll
        for (int e = 0; e < NET; ++e) regs.z[kBackRow][c * NET + e] = opaque(v[e]);      // (in a register of its own, not half of a 64-bit one)
      } else if constexpr (kLast && IO == kNttBack3) {
        const uint32_t j0 = 2 * (unit_o >= a.digits.d / 2 ? unit_o - a.digits.d / 2 : unit_o);
        const bool pair = j0 + 1 < a.k;
        const uint32_t j1 = pair ? j0 + 1 : j0;
        const uint32_t p0 = ldc(a.limbs, j0).m.p, p1 = ldc(a.limbs, j1).m.p, pinv0 = ldc(a.limbs, j0).pinv, pinv1 = ldc(a.limbs, j1).pinv;
        const RelinCrt k0 = ldc(a.crt, j0), k1 = ldc(a.crt, j1);
        const uint32_t second = pair ? N : 0;
        // four elements at a time: the rest of the registers holds residues
        constexpr int CH = 4;
#pragma unroll
        for (int e0 = 0; e0 < NET; e0 += CH) {
          uint32_t y0[CH], y1[CH];
#pragma unroll
          for (int e = 0; e < CH; ++e) {
            y0[e] = ld_at(gaux + off + (e0 + e) * TLAST, base * 4);
            y1[e] = ld_at(gaux + second + off + (e0 + e) * TLAST, base * 4);
          }
#pragma unroll
          for (int e = 0; e < CH; ++e) {
            const int32_t z[kSharedPrimes] = {regs.z[0][c * NET + e0 + e], regs.z[1][c * NET + e0 + e],
                                              regs.z[2][c * NET + e0 + e], v[e0 + e]};
            const int32_t round = relin_crt_round(z, a.crt_inv);
            y0[e] = add_mod(relin_crt(z, round, k0, p0, pinv0), y0[e], p0);
            y1[e] = add_mod(relin_crt(z, round, k1, p1, pinv1), y1[e], p1);
          }
#pragma unroll
          for (int e = 0; e < CH; ++e) {
            st_at(gout + off + (e0 + e) * TLAST, base * 4, y0[e]);
            if (pair) st_at(gout + N + off + (e0 + e) * TLAST, base * 4, y1[e]);
          }
          sched_fence();
        }
      } else if constexpr (kLast && (SPLIT || IO == kNttBackRow)) {
#pragma unroll
        for (int e = 0; e < NET; ++e) st_at(gout + off + e * TLAST, base * 4, (uint32_t)v[e]);
      } else if constexpr (kLast && kEncOut) {
        // The root level with + e (+ floor(q/t) * m) in front of its reductions: a product each, where the canonical residues of
        // e and m were found and added before (784 encryptions at n = 8192, k = 8: 311 us then, 265 now).  Eight elements at a
        // time; the next eight words of e and m are on their way while these are stored.
        const uint32_t* ge = reinterpret_cast<const uint32_t*>(a.small) + (size_t)group * N + off;
        auto root_level = [&](auto wide) {
          constexpr bool kWide = decltype(wide)::value, kMsg = IO == kNttEncOut0;
          constexpr int CH = NET / 8;
          const uint32_t pos = (uint32_t)opaque((int)base);       // (in this block: the accesses keep their scalar bases)
          const EncScale sc = kMsg ? ldc(a.scale, within) : EncScale{};
          const int64_t left_out = kMsg ? (kWide ? sc.c64 : sc.c32) : 0;
          auto at = [&](int ch, int j) { return kOdd ? j % 2 * (NET / 2) + ch * 4 + j / 2 : j % 4 * (NET / 4) + ch * 2 + j / 4; };
          uint32_t err[2][8], lo[2][8], hi[2][8];
          auto load = [&](int ch) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
              const int e = at(ch, j) * TLAST;
              err[ch % 2][j] = ld_at(ge + e, pos * 4);
              if constexpr (kMsg && !kWide) lo[ch % 2][j] = ld_at(a.msg + (size_t)group * N + off + e, pos * 4);
              if constexpr (kMsg && kWide) {
                const uint32_t* w = reinterpret_cast<const uint32_t*>(a.msg64 + (size_t)group * N + off + e);
                lo[ch % 2][j] = ld_at(w, pos * 8);
                hi[ch % 2][j] = ld_at(w + 1, pos * 8);
              }
            }
          };
          auto addend = [&](int ch, int j) {
            // (untraced: one chain of multiply-adds; the compiler would sum the products separately and add in 64 bits)
            int64_t x = untraced(left_out + (int64_t)(int32_t)err[ch % 2][j] * L.rc);
            if constexpr (kMsg) x = untraced(x + (int64_t)(int32_t)(lo[ch % 2][j] ^ 0x80000000u) * sc.lo);
            if constexpr (kMsg && kWide) x = untraced(x + (int64_t)(int32_t)(hi[ch % 2][j] ^ 0x80000000u) * sc.hi);
            return x;
          };
          load(0);
#pragma unroll
          for (int ch = 0; ch < CH; ++ch) {
            if (ch + 1 < CH) load(ch + 1);
            if constexpr (kOdd) {
#pragma unroll
              for (int j = 0; j < 8; j += 2) {
                int32_t &x = v[at(ch, j)], &y = v[at(ch, j + 1)];
                const int32_t X = x, Y = y;
                x = sredc(addend(ch, j) + (int64_t)(X + Y) * top.c0, p, L.pinv);
                y = sredc(addend(ch, j + 1) + (int64_t)(X - Y) * top.w, p, L.pinv);
              }
            } else {
#pragma unroll
              for (int j = 0; j < 8; j += 4) {
                const int64_t add[4] = {addend(ch, j), addend(ch, j + 1), addend(ch, j + 2), addend(ch, j + 3)};
                r4_inv_add(v[at(ch, j)], v[at(ch, j + 1)], v[at(ch, j + 2)], v[at(ch, j + 3)], top.c0,
                           R4Twiddle{top.w, top.v, top.vw, top.u}, top.nuw, add, L);
              }
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) st_at(gout + off + at(ch, j) * TLAST, pos * 4, canon_2p(v[at(ch, j)], p));
          }
        };
        if (IO != kNttEncOut0 || a.msg != nullptr) root_level(std::false_type{});
        else root_level(std::true_type{});
      } else if constexpr (kLast && (IO == kNttStoreAdd || kFromRegs || (kDecOut && !SPLIT))) {
        // all loads of the addend before the first store (the compiler must assume the buffers alias)
        uint32_t addend[NET];
#pragma unroll
        for (int e = 0; e < NET; ++e) addend[e] = ld_at(gaux + off + e * TLAST, base * 4);
#pragma unroll
        for (int e = 0; e < NET; ++e) st_at(gout + off + e * TLAST, base * 4, add_mod(canon_p(v[e], p), addend[e], p));
      } else if constexpr (kLast) {
        constexpr bool kLazyOut = IO == kNttLoadTensor || IO == kNttLoadTensorMul || kTensorRegs;
#pragma unroll
        for (int e = 0; e < NET; ++e) st_at(gout + off + e * TLAST, base * 4, kLazyOut ? (uint32_t)v[e] + p : canon_p(v[e], p));
      } else {
#pragma unroll
        for (int e = 0; e < NET; ++e) lds[lds_elem<LOG_TLAST>(sbase, e) + lds_swz(off)] = (uint32_t)v[e];
      }
    }
  }
};

// Several transforms of one workgroup, one after the other, P phases each: is transform t (forward up to `fwd` of them) done
// with phase ph without a barrier behind it?  Its own exchange takes one.  Between two transforms none is needed where they
// alternate between two row buffers (whoever writes a buffer again has passed the barrier of the transform in between, and so has
// every wave that read it), nor in front of an inverse transform that follows a forward one (it starts inside its waves' own words).
// Two buffers where the registers leave no room for a further workgroup anyway; otherwise the workgroup that one buffer leaves
// room for is worth more than the barriers (n = 8192, us, one / two buffers: tensor of 512 ciphertexts, three workgroups per
// compute unit / two, 516 / 588; 784 encryptions 319 / 345).
constexpr bool seq_wave_sync(int ph, int P, int fwd, int buffers) {
  const int t = ph / P, r = ph % P;
  if (r == P - 1) return buffers == 2 || t + 1 == fwd;
  return t < fwd ? r != 0 : r != P - 2;
}
template <class G, int BUFFERS>
HCNN_HD uint32_t* seq_buffer(uint32_t* lds, uint32_t t) { return BUFFERS == 2 ? lds + (t & 1u) * (uint32_t)(G::kLdsBytes / 4) : lds; }

// ------------------------------------------------------------------------- relinearisation in one kernel
// Workgroup (ct, j): for every digit i of y2[ct] -- forward transform modulo q_j, products with the two key rows
// added to register-held sums -- then the two sums go back through the inverse transform and leave as
// c'_b = y_b + sum_i evk[i][b] * digit_i (HMult step 3).  Neither the transformed digits nor the sums touch memory.
struct RelinFusedArgs {
  const uint32_t* y;        // [n_ct][3][k][n]
  const uint32_t* evk;      // [k][2][k][n], transformed
  uint32_t* out;            // [n_ct][2][k][n]
  TwTable tw_fwd;
  TwTable tw_inv;
  const NttLimb* limbs;
  uint32_t k;
  uint32_t n_rows;          // n_ct * k
  FastDiv cycle;            // k
  FastDiv share;            // k or k / 2: limbs of a ciphertext that run on one die (relin_share)
};

template <int LOGN, int LOGR, int MAC = kNttFusedMacAny>
struct RelinFused {
  using G = NttGeom<LOGN, LOGR>;
  using Fwd = NttFwd<LOGN, LOGR, MAC>;
  using Inv0 = NttInv<LOGN, LOGR, kNttFromRegs0>;
  using Inv1 = NttInv<LOGN, LOGR, kNttFromRegs1>;
  static constexpr int P = G::kPhases;
  static constexpr int kBuffers = 2;
  static constexpr size_t kLdsBytes = kBuffers * G::kLdsBytes;
  static constexpr int kThreads = G::kThreads;
  static constexpr int kLoopPhases = P;
  // room for two workgroups per compute unit (one of 1024 threads)
  static constexpr int kMinWavesPerSimd = G::kThreads >= 1024 ? 4 : (G::kThreads / 256 * 2 > 0 ? G::kThreads / 256 * 2 : 1);
  static constexpr int kPhases = 3 * P;
  using Regs = RelinRegs<G::R>;
  HCNN_HD static uint32_t loop_count(const RelinFusedArgs& a) { return a.k; }
  static constexpr bool wave_sync(int ph) { return seq_wave_sync(ph, P, 1, kBuffers); }

  template <int PH>
  HCNN_HD static void phase(const RelinFusedArgs& a, unsigned bid, int tid, uint32_t* lds, Regs& regs) {
    NttArgs na{};
    na.limbs = a.limbs; na.cycle = a.cycle; na.share = a.share; na.limb_base = 0; na.n_rows = a.n_rows;
    if constexpr (PH < P) {
      na.in = a.y; na.aux = a.evk; na.tw = a.tw_fwd;
      Fwd::template phase<PH>(na, bid, tid, seq_buffer<G, kBuffers>(lds, regs.iter), regs);
    } else {
      na.aux = a.y; na.out = a.out; na.tw = a.tw_inv;
      lds = seq_buffer<G, kBuffers>(lds, a.k + (PH < 2 * P ? 0 : 1));
      if constexpr (PH < 2 * P) Inv0::template phase<PH - P>(na, bid, tid, lds, regs);
      else Inv1::template phase<PH - 2 * P>(na, bid, tid, lds, regs);
    }
  }
};

// ------------------------------------------------------------------------- squaring tensor in one kernel
// Workgroup (ct, l): forward transforms of c0 and c1 modulo limb l (l < k: read from the ciphertext; else from the
// extension buffer), kept in registers, then the three tensor components c0^2, 2 c0 c1, c1^2 through the inverse
// transform into d[ct][b][l] (HMult step 1 with both operands equal).  The transformed operands never touch memory.
struct TensorFusedArgs {
  const uint32_t* cts;      // [n_ct][2][k][n]
  const uint32_t* ext;      // [n_ct][2][L][n], rows k..L-1 of every polynomial valid
  uint32_t* d;              // [n_ct][3][L][n]
  TwTable tw_fwd;
  TwTable tw_inv;
  const NttLimb* limbs;
  uint32_t k, L;
  uint32_t n_rows;          // n_ct * L
  FastDiv cycle;            // L
  FastDiv cts_div;          // n_ct: pairs in the order of the limbs (n >= 16384); 0: of the ciphertexts
};

// SPLIT = 1 (n = 32768): workgroup (ct, l, half), both ends as in the split transforms: it reads whole rows of c0 and c1, keeps its halves and leaves
// its halves of the three components without the last stage.  Us, 32 ciphertexts of 24 + 26 limbs: the two separate kernels with a whole row per
// inverse workgroup 681, with half a row 600, this one 497 (1024 MiB through memory: 230).
template <int LOGN, int LOGR, int SPLIT = 0>
struct TensorFused {
  using G = NttGeom<LOGN - SPLIT, LOGR>;
  static size_t grid(size_t pairs) { return SPLIT ? split_grid(pairs) : pairs; }
  static constexpr int P = G::kPhases;
  static constexpr int kBuffers = LOGN == 14 && LOGR == 4 ? 2 : 1;
  static constexpr size_t kLdsBytes = kBuffers * G::kLdsBytes;
  static constexpr int kThreads = G::kThreads;
  static constexpr int kPhases = 5 * P;
  static constexpr int kMinWavesPerSimd = 4;     // 128 registers: two 512-thread or four 256-thread workgroups per compute unit
  using Regs = TensorRegs<G::R>;
  static constexpr bool wave_sync(int ph) { return seq_wave_sync(ph, P, 2, kBuffers); }

  // Large launches from n = 16384 on: every die takes its share of the pairs in the order of the limbs, so that its L2 holds the twiddles of the one or two limbs at
  // work (5/3 n words a limb and direction: 7.1 MiB at n = 16384, L = 34).  Us, squarings with the pairs in the order of the ciphertexts / of the
  // limbs: n = 32768, k = 24, 32 ciphertexts 1729 / 1688, k = 12 807 / 790; n = 16384, k = 16, 225 3198 / 3159, k = 12, 300 3199 / 3158.  At n = 8192,
  // where the twiddles of all limbs stay in L2, 720 of 8 primes 1978 / 1972, but 1520 of 11 (a network) 7580 / 7605.
  HCNN_HD static unsigned pair_of(const TensorFusedArgs& a, unsigned i) {
    const uint32_t die = i % kNttXcds, share = a.n_rows / kNttXcds, rest = a.n_rows % kNttXcds;
    const uint32_t at = die * share + (die < rest ? die : rest) + i / kNttXcds, l = quot(at, a.cts_div);
    return (at - l * a.cts_div.d) * a.L + l;
  }
  HCNN_HD static unsigned place(const TensorFusedArgs& a, unsigned bid) {
    if (LOGN < 14 || a.cts_div.d == 0) return bid;
    if constexpr (!SPLIT) return pair_of(a, bid);
    if (split_row(bid) >= a.n_rows) return bid;
    const uint32_t row = pair_of(a, split_row(bid));
    return row / kNttXcds * 2 * kNttXcds + split_half(bid) * kNttXcds + row % kNttXcds;
  }

  template <int PH>
  HCNN_HD static void phase(const TensorFusedArgs& a, unsigned bid, int tid, uint32_t* lds, Regs& regs) {
    lds = seq_buffer<G, kBuffers>(lds, PH / P);
    bid = place(a, bid);
    NttArgs na{};
    na.limbs = a.limbs; na.cycle = a.cycle; na.limb_base = 0; na.n_rows = a.n_rows;
    if constexpr (PH < 2 * P) {
      na.in = a.ext; na.aux = a.cts; na.own_limbs = a.k; na.tw = a.tw_fwd;
      if constexpr (PH < P) NttFwd<LOGN, LOGR, kNttToRegs0, SPLIT>::template phase<PH>(na, bid, tid, lds, regs);
      else NttFwd<LOGN, LOGR, kNttToRegs1, SPLIT>::template phase<PH - P>(na, bid, tid, lds, regs);
    } else {
      na.out = a.d; na.tw = a.tw_inv;
      if constexpr (PH < 3 * P) NttInv<LOGN, LOGR, kNttTensorRegs0, SPLIT>::template phase<PH - 2 * P>(na, bid, tid, lds, regs);
      else if constexpr (PH < 4 * P) NttInv<LOGN, LOGR, kNttTensorRegs1, SPLIT>::template phase<PH - 3 * P>(na, bid, tid, lds, regs);
      else NttInv<LOGN, LOGR, kNttTensorRegs2, SPLIT>::template phase<PH - 4 * P>(na, bid, tid, lds, regs);
    }
  }
};

// ------------------------------------------------------------------------- shared-basis relinearisation, last part
// Workgroup (ct, o = (b, pair)): the four rows acc[ct][o][r] back to coefficients, from modulo p_0 .. p_3 to modulo the pair's two
// primes, plus y_b: one read of the sums, one write of the result.  (The largest ring does not hold three rows beside the one in
// work in its registers: kNttBackRow and RelinCombine.)
// Bound: one 1024-thread workgroup per compute unit, in step with itself.  A row's words are loaded during the last pass of the row before
// (n = 16384, k = 16, 225 ciphertexts 690 -> 648 us; 397 by bytes); with three rows parked and the next one's words that takes all 128 registers and spills
// 14 (60 bytes of scratch a lane).
struct RelinBackArgs {
  const uint32_t* acc;      // [n_ct][4][n/64][outputs][64]
  const uint32_t* y;        // [n_ct][3][k][n]
  uint32_t* out;            // [n_ct][2][k][n]
  TwTable tw_inv;
  const NttLimb* limbs;
  const RelinCrt* crt;
  RelinCrtInv crt_inv;
  uint32_t limb_base;       // of the four primes
  FastDiv outputs;          // (b, pair)
  uint32_t k;
};
template <int LOGN, int LOGR>
struct RelinBack {
  using G = NttGeom<LOGN, LOGR>;
  static constexpr int P = G::kPhases;
  static constexpr int kBuffers = 2;
  static constexpr size_t kLdsBytes = kBuffers * G::kLdsBytes;
  static constexpr int kThreads = G::kThreads;
  static constexpr int kPhases = (int)kSharedPrimes * P;
  static constexpr int kMinWavesPerSimd = 4;
  using Regs = BackRegs<G::R>;
  static constexpr bool wave_sync(int ph) { return seq_wave_sync(ph, P, 0, kBuffers); }
  template <int PH>
  HCNN_HD static void phase(const RelinBackArgs& a, unsigned bid, int tid, uint32_t* lds, Regs& regs) {
    lds = seq_buffer<G, kBuffers>(lds, PH / P);
    NttArgs na{};
    na.in = a.acc; na.aux = a.y; na.out = a.out; na.tw = a.tw_inv; na.limbs = a.limbs; na.limb_base = a.limb_base;
    na.cycle = FastDiv{kSharedPrimes, 0x40000000u}; na.tile_words = a.outputs.d * 64;
    na.digits = a.outputs; na.crt = a.crt; na.crt_inv = a.crt_inv; na.k = a.k;
    if constexpr (PH < P) NttInv<LOGN, LOGR, kNttBack0>::template phase<PH>(na, bid, tid, lds, regs);
    else if constexpr (PH < 2 * P) NttInv<LOGN, LOGR, kNttBack1>::template phase<PH - P>(na, bid, tid, lds, regs);
    else if constexpr (PH < 3 * P) NttInv<LOGN, LOGR, kNttBack2>::template phase<PH - 2 * P>(na, bid, tid, lds, regs);
    else NttInv<LOGN, LOGR, kNttBack3>::template phase<PH - 3 * P>(na, bid, tid, lds, regs);
  }
};

// ------------------------------------------------------------------------- encryption and decryption
// Workgroup (ct, l), one row in registers from the forward transform to the last store:
//   encryption  u -> forward; times pk0^, back, + e1 + floor(q/t) m -> c0; times pk1^, back, + e2 -> c1
//   decryption  c1 -> forward; times s^, back, + c0 -> x
// OWN (decryption of few ciphertexts): the workgroup transforms s itself instead of waiting for a launch that does
// (10 ciphertexts at n = 8192, k = 8: 23.4 -> 20.7 us; 4 at n = 1024, k = 2: 14.1 -> 11.6).
// As separate launches the same work moves every row through memory five times in between (and was cut into batches of 64
// for its buffers): 784 encryptions at n = 8192, k = 8 took 1312 us.
struct CryptArgs {
  const uint32_t* key;      // [2][k][n] (encryption) or [k][n]: transformed, as kNttStoreKey leaves it
  const int32_t* u;         // encryption: [n_ct][n]; OWN: s [n]
  const int32_t* e1;
  const int32_t* e2;
  const uint32_t* msg;      // as in NttArgs
  const uint64_t* msg64;
  const EncScale* scale;
  const uint32_t* cts;      // decryption: [n_ct][2][k][n]
  uint32_t* out;            // [n_ct][2][k][n] or [n_ct][k][n]
  TwTable tw_fwd;
  TwTable tw_inv;
  const NttLimb* limbs;
  uint32_t n_rows;          // n_ct * k
  FastDiv cycle;            // k
};

// SPLIT (decryption, n = 8192 and 32768): workgroup (ct, l, half), both ends as in the split transforms; c0 and the last stage are left to the rounding.
template <int LOGN, int LOGR, bool ENC, bool OWN = false, int SPLIT = 0>
struct CryptFused {
  static_assert(!SPLIT || (OWN && !ENC), "an encryption's rows are results, and a call small enough for halves transforms its own secret");
  using G = NttGeom<LOGN - SPLIT, LOGR>;
  static size_t grid(size_t slots) { return SPLIT ? split_grid(slots) : slots; }
  static constexpr int P = G::kPhases;
  // (a decryption that finds the key's transform has no exchange between its two transforms that a second buffer would spare a barrier, and
  // with one two workgroups of n = 16384 fit a compute unit: 500 ciphertexts, k = 8 358 us with two buffers, 322 with one)
  static constexpr int kBuffers = LOGN == 14 && (ENC || OWN) ? 2 : 1;
  static constexpr size_t kLdsBytes = kBuffers * G::kLdsBytes;
  static constexpr int kThreads = G::kThreads;
  static constexpr int kPhases = (ENC || OWN ? 3 : 2) * P;
  static constexpr int kMinWavesPerSimd = 4;
  using Regs = RowRegs<G::R>;
  static constexpr bool wave_sync(int ph) { return seq_wave_sync(ph, P, OWN ? 2 : 1, kBuffers); }

  template <int PH>
  HCNN_HD static void phase(const CryptArgs& a, unsigned bid, int tid, uint32_t* lds, Regs& regs) {
    lds = seq_buffer<G, kBuffers>(lds, PH / P);
    NttArgs na{};
    na.limbs = a.limbs; na.cycle = a.cycle; na.n_rows = a.n_rows;
    if constexpr (OWN) {
      na.small = a.u; na.in = a.cts; na.out = a.out; na.aux = a.cts;
      na.tw = PH < 2 * P ? a.tw_fwd : a.tw_inv;
      if constexpr (PH < P) NttFwd<LOGN, LOGR, kNttSecretToRegs, SPLIT>::template phase<PH>(na, bid, tid, lds, regs);
      else if constexpr (PH < 2 * P) NttFwd<LOGN, LOGR, kNttCtToRegs, SPLIT>::template phase<PH - P>(na, bid, tid, lds, regs);
      else NttInv<LOGN, LOGR, kNttDecOwn, SPLIT>::template phase<PH - 2 * P>(na, bid, tid, lds, regs);
    } else if constexpr (PH < P) {
      na.tw = a.tw_fwd; na.small = a.u; na.in = a.cts;
      NttFwd<LOGN, LOGR, ENC ? kNttSmallToRegs : kNttCtToRegs>::template phase<PH>(na, bid, tid, lds, regs);
    } else {
      na.tw = a.tw_inv; na.in = a.key; na.out = a.out; na.aux = a.cts;
      na.msg = a.msg; na.msg64 = a.msg64; na.scale = a.scale;
      na.small = PH < 2 * P ? a.e1 : a.e2;
      if constexpr (!ENC) NttInv<LOGN, LOGR, kNttDecOut>::template phase<PH - P>(na, bid, tid, lds, regs);
      else if constexpr (PH < 2 * P) NttInv<LOGN, LOGR, kNttEncOut0>::template phase<PH - P>(na, bid, tid, lds, regs);
      else NttInv<LOGN, LOGR, kNttEncOut1>::template phase<PH - 2 * P>(na, bid, tid, lds, regs);
    }
  }
};

}  // namespace hcnn
