// The host-side rules of the library that no entry point shows, for tests/test_host_rules.py: the library's source with
// plain functions around them.
#include "../paper_1811_00778_amd/csrc/hcnn.cpp"

extern "C" {

// Groups per workgroup of the scalar MAC's matrix form on a device of `units` compute units, 0: the vector form.
int rule_mac_matrix_groups(uint32_t units, uint32_t n, uint32_t k, uint32_t n_in, uint32_t G, uint32_t F, uint32_t T, int32_t w_abs_max) {
  hcnn_ctx c;
  c.n = n; c.k = k; c.compute_units = units; c.max_lds = max_lds_bytes();
  MacArgs a{};
  a.k = k; a.n = n; a.n_in = n_in; a.G = G; a.F = F; a.T = T; a.w_abs_max = w_abs_max;
  return mac_matrix_groups(&c, (size_t)G * (2 * k * n / (kEwThreads * kEwVec)), a);
}
// Does a call whose workgroups take two groups form the union of their rows?
int rule_mac_takes_pairs(uint32_t units, uint32_t n, uint32_t k, uint32_t n_in, uint32_t G, uint32_t T) {
  hcnn_ctx c;
  c.compute_units = units; c.max_lds = max_lds_bytes();
  MacArgs a{};
  a.k = k; a.n = n; a.n_in = n_in; a.G = G; a.T = T;
  return mac_takes_pairs(&c, a);
}
// Groups that a call of few filters sums side by side, 0: the vector form.
uint32_t rule_mac_pack_groups(uint32_t units, uint32_t n, uint32_t k, uint32_t n_in, uint32_t G, uint32_t F, uint32_t T, int32_t w_abs_max) {
  hcnn_ctx c;
  c.compute_units = units; c.max_lds = max_lds_bytes();
  MacArgs a{};
  a.k = k; a.n = n; a.n_in = n_in; a.G = G; a.F = F; a.T = T; a.w_abs_max = w_abs_max;
  return mac_pack_groups(&c, a);
}
// Tiles per wave of MacMfma<1> (groups = 1), MacMfma<2> (2) or MacPair (0).
uint32_t rule_mac_matrix_steps(uint32_t groups, uint32_t units, uint32_t n, uint32_t k, uint32_t G, uint32_t T) {
  hcnn_ctx c;
  c.compute_units = units;
  MacArgs a{};
  a.k = k; a.n = n; a.G = G; a.T = T;
  return groups == 0 ? mac_matrix_steps<MacPair>(&c, a) : groups == 1 ? mac_matrix_steps<MacMfma<1>>(&c, a) : mac_matrix_steps<MacMfma<2>>(&c, a);
}
// Tiles per wave of MacPack.
uint32_t rule_mac_pack_steps(uint32_t units, uint32_t n, uint32_t k, uint32_t n_in, uint32_t G, uint32_t F, uint32_t T) {
  hcnn_ctx c;
  c.compute_units = units;
  MacArgs a{};
  a.k = k; a.n = n; a.n_in = n_in; a.G = G; a.F = F; a.T = T; a.pack = 16 / F;
  return mac_matrix_steps<MacPack>(&c, a);
}
size_t rule_mac_matrix_lds(uint32_t groups, size_t T) {
  return groups == 2 ? MacMfma<2>::lds_bytes(T) : MacMfma<1>::lds_bytes(T);
}

// LDS of a workgroup of the decryption that reads the secret's transform (n = 16384).
size_t rule_decrypt_lds() { return CryptFused<14, 4, false>::kLdsBytes; }

// Do the inverse transforms of `rows` rows of a squaring's tensor take two workgroups per row?
int rule_splits_tensor_rows(uint32_t units, uint32_t n, size_t rows) {
  hcnn_ctx c;
  c.logn = (uint32_t)__builtin_ctz(n); c.compute_units = units;
  return splits_tensor_rows(&c, rows);
}

// Does a decryption take two workgroups per row?
int rule_decrypts_by_halves(uint32_t units, uint32_t n, uint32_t k, size_t n_ct) {
  hcnn_ctx c;
  c.logn = (uint32_t)__builtin_ctz(n); c.k = k; c.compute_units = units;
  return decrypts_by_halves(&c, n_ct);
}

// Does a squaring's internal batch take the one-kernel tensor, and from how many workgroups on whatever their rounds (0: never)?
static hcnn_ctx tensor_ctx(uint32_t units, uint32_t per_unit, uint32_t n, uint32_t k, uint32_t k_aux) {
  hcnn_ctx c;
  c.logn = (uint32_t)__builtin_ctz(n); c.k = k; c.kp = k_aux; c.compute_units = units; c.tensor_fused_wgs = per_unit;
  return c;
}
int rule_takes_tensor_fused(uint32_t units, uint32_t per_unit, uint32_t n, uint32_t k, uint32_t k_aux, size_t n_ct) {
  const hcnn_ctx c = tensor_ctx(units, per_unit, n, k, k_aux);
  return takes_tensor_fused(&c, n_ct);
}
size_t rule_tensor_fused_least(uint32_t n) {
  const hcnn_ctx c = tensor_ctx(256, 1, n, 1, 1);
  return tensor_fused_least(&c);
}

// Workgroups from which the one-kernel relinearisation takes n_ct ciphertexts that are not whole rounds.
size_t rule_relin_fused_least(uint32_t units, uint32_t n, uint32_t k, size_t n_ct, int with_rounds) {
  hcnn_ctx c;
  c.logn = (uint32_t)__builtin_ctz(n); c.k = k; c.compute_units = units;
  return relin_fused_least(&c, n_ct, with_rounds);
}

// Do n_ct ciphertexts take it to the last, `whole` of which fill its rounds, with per_unit workgroups on a compute unit?
int rule_relin_fused_takes_rest(uint32_t units, uint32_t per_unit, uint32_t n, uint32_t k, size_t n_ct, size_t whole) {
  hcnn_ctx c;
  c.n = n; c.logn = (uint32_t)__builtin_ctz(n); c.k = k; c.compute_units = units; c.relin_fused_wgs = per_unit;
  return relin_fused_takes_rest(&c, n_ct, whole);
}

// Ciphertexts for whose separate kernels the work buffer has room.
size_t rule_relin_split_most(uint32_t n, uint32_t k, size_t fused_round) {
  hcnn_ctx c;
  c.logn = (uint32_t)__builtin_ctz(n); c.k = k;
  return relin_split_most(&c, fused_round);
}

// Pair (one workgroup of n <= 16384) or, n = 32768, place (half of a pair) that workgroup `bid` of the one-kernel tensor takes in the order of the limbs.
uint32_t rule_tensor_place(uint32_t split, uint32_t n_ct, uint32_t L, uint32_t bid) {
  TensorFusedArgs a{};
  a.L = L; a.n_rows = n_ct * L; a.cts_div = fast_div(n_ct);
  return split ? TensorFused<15, 5, 1>::place(a, bid) : TensorFused<14, 5>::place(a, bid);
}

// Limbs of a ciphertext that share a die in the one-kernel relinearisation, and the (ciphertext, limb) row of one of its workgroups.
uint32_t rule_relin_share(uint32_t n, uint32_t k) {
  hcnn_ctx c;
  c.n = n; c.k = k;
  return relin_share(&c);
}
uint32_t rule_relin_grid(uint32_t rows, uint32_t share) { return (uint32_t)ntt_grouped_grid(rows, share); }
uint32_t rule_relin_row(uint32_t bid, uint32_t share) { return ntt_grouped_index(bid, fast_div(share)); }

// Smallest batch that takes the shared-basis relinearisation, 0: none.
size_t rule_shared_basis_min(uint32_t n, uint32_t k, uint32_t k_aux) {
  hcnn_ctx c;
  c.n = n; c.k = k; c.kp = k_aux;
  while ((1u << c.logn) < n) ++c.logn;
  return shared_basis_min(&c);
}

}  // extern "C"
