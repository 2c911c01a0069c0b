"""Kernel sources checked on the CPU: the library compiled with -DHCNN_HOSTEMU runs the same
kernel phase bodies and host orchestration as loops, and must match the oracle bit for bit.
(The product path itself is tested in test_gpu_parity.py; nothing here touches a GPU.)"""
import numpy as np
import pytest

import emu
import parity_cases as pc
from paper_1811_00778_amd import _capi


class EmuBackend:
    def __init__(self):
        self.lib = emu.lib()

    def make_ctx(self, n, q, p, t):
        return emu.EmuContext(n, q, p, t)

    @staticmethod
    def dev(a):
        return emu.aligned(np.ascontiguousarray(a))

    @staticmethod
    def host(buf):
        return buf


@pytest.fixture(scope="module")
def backend():
    return EmuBackend()


class SharedBasisBackend(EmuBackend):
    def make_ctx(self, n, q, p, t):
        return emu.EmuContext(n, q, p, t, emu.lib_shared_basis())


@pytest.mark.parametrize("n,k,count", [(1024, 2, 3), (1024, 17, 9), (1024, 26, 1), (2048, 5, 8), (4096, 3, 2), (16384, 2, 2), (32768, 2, 2)])
def test_square_relin_shared_basis(n, k, count):
    """The shared-basis relinearisation: both of its last parts, groups of eight ciphertexts and a remainder, bases on
    both sides of its folds; residues at the ends of the transforms' ranges."""
    backend = SharedBasisBackend()
    pc.check_square_relin(backend, n, k, n_random=count, n_genuine=0, check_decrypt=False)
    if n <= 2048:
        pc.check_transform_ranges(backend, n)


def test_second_key_finds_the_room_for_its_copy_that_the_first_did_not():
    """A device without memory for the copy of the key modulo the shared primes: the other forms until a key is set that finds it."""
    n, k, backend = 1024, 3, SharedBasisBackend()
    s = pc.Setup(backend, n, k)
    cts = pc.gen.uniform_residues(s.rng, s.q, n, lead=(3, 2))
    want = np.stack([pc.fv.square_relin(s.octx, c, s.evk) for c in cts])
    s.ctx.set_profile(True)

    def through_shared_primes():
        s.ctx.reset_stats()
        assert np.array_equal(s.ctx.ct_square_relin(backend.dev(cts)), want)
        return s.ctx.profile()["relin_mac"][1] == 3 * (n // 64)          # one workgroup of eight ciphertexts per tile, counted three times

    with emu.device(emu.lib_shared_basis(), largest=2 * k * k * n * 4):
        s.ctx.set_relin_key(backend.dev(s.evk))
    assert not through_shared_primes()
    with emu.device(emu.lib_shared_basis(), largest=2 * k * k * n * 4):
        s.ctx.set_relin_key(backend.dev(s.evk))
    assert not through_shared_primes()
    s.ctx.set_relin_key(backend.dev(s.evk))
    assert through_shared_primes()
    s.ctx.set_relin_key(backend.dev(s.evk))
    assert through_shared_primes()
    s.ctx.close()


@pytest.mark.parametrize("n,k", [(8192, 2)])
def test_square_relin_rows_by_two_workgroups(n, k):
    # (this build runs every squaring of these rings as the device runs its smallest ones)
    pc.check_square_relin(SharedBasisBackend(), n, k, n_random=1, n_genuine=0)
    pc.check_square_relin(SharedBasisBackend(), n, k, n_random=1, n_genuine=0, force_exact=True)


@pytest.mark.parametrize("n,k,n_polys,rows", [(1024, 2, 3, None), (2048, 3, 2, 3), (4096, 2, 1, 2),
                                             (8192, 2, 1, 1), (16384, 1, 1, 1), (32768, 1, 10, 1)])
def test_ntt_all_sizes(backend, n, k, n_polys, rows):
    pc.check_ntt(backend, n, k, n_polys, rows)


@pytest.mark.parametrize("n", [2048, 4096])
def test_ntt_of_few_rows(backend, n):
    pc.check_ntt(backend, n, 1, 1, None)          # one row for this build's one compute unit: a pass less


@pytest.mark.parametrize("n", [1024, 2048])
def test_transform_ranges_at_both_ends_of_the_prime_interval(backend, n):
    pc.check_transform_ranges(backend, n)


@pytest.mark.parametrize("n,k", [(1024, 2), (2048, 3)])
def test_keygen_encrypt_decrypt(backend, n, k):
    pc.check_keygen_encrypt_decrypt(backend, n, k)


def test_decrypt_rows_by_two_workgroups():
    # (this build decrypts at n = 8192 as the device does the smallest calls; n = 32768 always goes by halves)
    pc.check_keygen_encrypt_decrypt(SharedBasisBackend(), 8192, 2, count=2)


@pytest.mark.parametrize("n,k,t", [(8192, 5, 65537), (8192, 6, pc.WIDE_T), (32768, 5, 65537)])
def test_decrypt_by_halves_with_every_comparison_exact(n, k, t):
    pc.check_decrypt_exact(SharedBasisBackend(), n, k, t)          # (this build takes halves at both rings)


@pytest.mark.parametrize("n,k", [(4096, 3), (8192, 2), (16384, 2), (32768, 2)])
def test_encrypt_decrypt_of_every_ring(backend, n, k):
    pc.check_keygen_encrypt_decrypt(backend, n, k, count=1)


@pytest.mark.parametrize("n,k", [(1024, 1), (1024, 2), (8192, 8), (32768, 24)])
def test_first_decryption_of_a_context_finds_its_work_buffer(backend, n, k):
    """A decryption or noise read-out of up to 33 ciphertexts after key generation or one encryption allocates nothing."""
    cand = _capi.gen_primes(backend.lib, n, k)
    s, e = np.zeros(n, np.int32), np.zeros((1, n), np.int32)
    a, m = np.zeros((k, n), np.uint32), np.zeros((1, n), np.uint32)
    s[1], pk = 1, np.zeros((2, k, n), np.uint32)
    for after in ("keygen", "encrypt"):
        ctx = backend.make_ctx(n, cand, [], 65537)
        if after == "keygen":
            ctx.keygen(s, a, e[0])
        else:
            ctx.encrypt(pk, m, e, e, e)
        held = ctx.scratch_bytes()
        for count in ((1, 10) if n > 8192 else (1, 10, 25, 33)):
            x = np.zeros((count, 2, k, n), np.uint32)
            x[-1, 1] = 1
            ctx.decrypt(s, x)
            if n == 1024:
                ctx.noise_bits(s, x)
            assert ctx.scratch_bytes() == held, (after, count)
        ctx.close()


def test_work_of_a_large_squaring_leaves_the_small_work_buffer_alone(backend):
    """The first squaring after key generation frees nothing, and a decryption after it finds what it had."""
    s = pc.Setup(backend, 1024, 2)
    kr = {x: backend.dev(v) for x, v in s.kr.items()}
    x = backend.dev(pc.gen.uniform_residues(s.rng, s.q, 1024, lead=(40, 2)))
    s.ctx.set_relin_key(backend.dev(s.evk))
    assert s.ctx.scratch_bytes() == 0
    s.ctx.ct_square_relin(x)
    large = s.ctx.scratch_bytes()
    s.ctx.keygen(kr["s"], kr["a"], kr["e"], kr["a_evk"], kr["e_evk"])
    small = s.ctx.scratch_bytes() - large
    assert 0 < small < large
    for call in (lambda: s.ctx.ct_square_relin(x[:3]), lambda: s.ctx.decrypt(kr["s"], x), lambda: s.ctx.ct_square_relin(x)):
        call()
        assert s.ctx.scratch_bytes() == small + large
    s.ctx.close()


@pytest.mark.parametrize("n,k", [(1024, 2), (2048, 5)])
def test_scalar_mac(backend, n, k):
    pc.check_scalar_mac(backend, n, k)
    pc.check_mac_linear_in_ntt_domain(backend, n, k)


@pytest.mark.parametrize("G,F,T,bound", [(5, 16, 25, 7), (4, 14, 31, 127), (6, 10, 96, 127), (3, 11, 97, 15), (2, 16, 130, 31),
                                         (1, 8, 64, 127), (1, 13, 81, 7), (1, 16, 1000, 127), (9, 16, 48, 1)])
def test_scalar_mac_matrix_form(backend, G, F, T, bound):
    k = 1 if G == 1 else 2                       # one group: few enough coefficients for this build's single compute unit
    form = 2 if G in (2, 9) else 1
    assert emu.rules().rule_mac_matrix_groups(1, 1024, k, pc.MATRIX_INPUTS, G, F, T, bound) == form
    assert form == 1 or not emu.rules().rule_mac_takes_pairs(1, 1024, k, pc.MATRIX_INPUTS, G, T)          # (not the union form)
    pc.check_scalar_mac_matrix_form(backend, G, F, T, bound, k=k)


def test_scalar_mac_matrix_form_with_several_tiles_per_wave(backend):
    for G, F, T, bound, form, steps in ((3, 11, 97, 31, 1, 2), (7, 14, 25, 7, 2, 8)):
        assert emu.rules().rule_mac_matrix_groups(1, 1024, 3, pc.MATRIX_INPUTS, G, F, T, bound) == form
        assert form == 1 or not emu.rules().rule_mac_takes_pairs(1, 1024, 3, pc.MATRIX_INPUTS, G, T)
        assert emu.rules().rule_mac_matrix_steps(form, 1, 1024, 3, G, T) == steps
        pc.check_scalar_mac_matrix_tiles(backend, 3, G, F, T, bound)
    # eight tiles per wave, the last block of tiles beyond the ciphertext by half
    assert emu.rules().rule_mac_matrix_steps(1, 1, 1024, 9, 3, 97) == 8
    pc.check_scalar_mac_matrix_tiles(backend, 9, 3, 11, 97, 31)


@pytest.mark.parametrize("c_in,side,f,stride,pad,F,base,ring", pc.PACK_CASES)
def test_scalar_mac_groups_side_by_side(backend, c_in, side, f, stride, pad, F, base, ring):
    G, T, n_in = ((side + 2 * pad - f) // stride + 1) ** 2, c_in * f * f, base + c_in * side * side
    assert emu.rules().rule_mac_pack_groups(1, *ring, n_in, G, F, T, 15) == emu.rules().rule_mac_pack_groups(256, *ring, n_in, G, F, T, 15) == 16 // F
    pc.check_scalar_mac_pairs(backend, c_in, side, f, stride, pad, F, base, *ring)


def test_scalar_mac_sixteen_groups_of_one_filter(backend):
    pc.check_scalar_mac_one_filter(backend, 1024, 4)


def test_scalar_mac_one_filter_in_a_launch_that_takes_sixteen_groups_a_set(backend):
    assert [emu.rules().rule_mac_pack_groups(units, *pc.PACK_ONE_FILTER, 15) for units in (1, 256)] == [16, 16]
    pc.check_scalar_mac_one_filter_per_set(backend)


@pytest.mark.parametrize("c_in,side,f,stride,pad,F,base,ring", pc.PAIR_CASES)
def test_scalar_mac_over_the_union_of_two_rows(backend, c_in, side, f, stride, pad, F, base, ring):
    G, T, n_in = ((side + 2 * pad - f) // stride + 1) ** 2, c_in * f * f, base + c_in * side * side
    assert emu.rules().rule_mac_matrix_groups(1, *ring, n_in, G, F, T, 15) == 2
    assert emu.rules().rule_mac_takes_pairs(1, *ring, n_in, G, T)
    pc.check_scalar_mac_pairs(backend, c_in, side, f, stride, pad, F, base, *ring)


def test_square_relin_tiny_config(backend):
    pc.check_square_relin(backend, 1024, 2)


def test_square_relin_chunked_ragged(backend):
    pc.check_square_relin(backend, 1024, 3, n_random=4, n_genuine=1, chunk=2)
    pc.check_square_relin(backend, 1024, 3, n_random=5, n_genuine=1)      # one group of four sharing key loads + two singles
    pc.check_square_relin(backend, 1024, 3, n_random=2, n_genuine=0, chunk=2, relin_order=1)   # ciphertext-major order forced


def test_square_relin_batch_split_into_rounds_and_remainder(backend):
    """The default policy sizes its rounds from the occupancy that the platform layer reports for the compiled
    kernels (this build: a fixed count for its single compute unit).  A batch of three rounds of the one-kernel
    relinearisation plus two ciphertexts, large enough for the one-kernel tensor, must take the mixed route: the
    tensor in one kernel, the whole rounds through the one-kernel relinearisation, the two left over through the
    separate kernels."""
    s = pc.Setup(backend, 1024, 2)
    s.ctx.set_relin_key(backend.dev(s.evk))
    rnd, L = s.ctx.relin_fused_round(), 2 + len(s.p)
    assert rnd >= 1
    n_ct = 3 * rnd + 2
    assert n_ct * L >= s.ctx.tensor_fused_threshold()
    cts = pc.gen.uniform_residues(s.rng, s.q, 1024, lead=(n_ct, 2))
    s.ctx.set_profile(True)
    out = backend.host(s.ctx.ct_square_relin(backend.dev(cts)))
    prof = s.ctx.profile()
    assert prof["tensor"][0] == 1 and prof["tensor"][1] == n_ct * L * 5
    assert prof["relin_fused"][0] == 1 and prof["relin_fused"][1] == 3 * rnd * 2 * (2 + 2)
    assert prof["relin_mac"][0] == 1 and prof["ntt_fwd"][1] == 2 * 2 * 2            # the two left over: digit rows only
    for i in (0, 3 * rnd - 1, 3 * rnd, 3 * rnd + 1):
        assert np.array_equal(out[i], pc.fv.square_relin(s.octx, cts[i], s.evk)), i
    # a batch below the tensor threshold and below 3/4 of a round: separate kernels throughout
    s.ctx.reset_stats()
    small = max(1, (3 * rnd - 1) // 4)
    s.ctx.ct_square_relin(backend.dev(cts[:small]))
    prof = s.ctx.profile()
    if small * L < s.ctx.tensor_fused_threshold() and small * 4 < rnd * 3:
        assert prof["tensor"][0] == 0 and prof["relin_fused"][0] == 0 and prof["relin_mac"][0] >= 1
    s.ctx.close()


def test_one_kernel_tensor_is_taken_where_its_rounds_are_filled(backend):
    """Batches on both sides of 7/8 fill in one to seven rounds: the policy that the binding reports is the one that
    runs, and from the reported threshold on it always does."""
    s = pc.Setup(backend, 1024, 2)
    s.ctx.set_relin_key(backend.dev(s.evk))
    s.ctx.set_profile(True)
    cts = backend.dev(pc.gen.uniform_residues(s.rng, s.q, 1024, lead=(24, 2)))
    L, took = 2 + len(s.p), []
    for n_ct in range(1, 25):
        s.ctx.reset_stats()
        s.ctx.ct_square_relin(cts[:n_ct])
        took.append(s.ctx.profile()["tensor"][0] == 1)
        assert took[-1] == s.ctx.takes_tensor_fused(n_ct), n_ct
        assert took[-1] or n_ct * L < s.ctx.tensor_fused_threshold()
    assert took[2] and not took[3] and not took[4] and took[5] and not took[7] and took[8]      # 15, 20, 25, 30, 40, 45 pairs, rounds of 16
    slots = 16
    assert s.ctx.tensor_fused_threshold() == 98
    assert all(8 * p >= 7 * slots * -(-p // slots) for p in range(98, 1000)) and 8 * 97 < 7 * slots * -(-97 // slots)
    s.ctx.close()


def test_square_relin_noalloc_equals_allocating_entry_point(backend):
    """The entry point that works in the library's static array: same residues as hcnn_ct_square_relin on two calls in
    a row (the second smaller), no work buffer allocated; a parameter set beyond the array is refused."""
    from paper_1811_00778_amd import _capi
    s = pc.Setup(backend, 1024, 3)
    s.ctx.set_relin_key(backend.dev(s.evk))
    for count in (11, 2):
        cts = backend.dev(pc.gen.uniform_residues(s.rng, s.q, 1024, lead=(count, 2)))
        out = s.ctx.ct_square_relin_noalloc(cts, np.zeros_like(cts))
        assert s.ctx.scratch_bytes() == 0
        assert np.array_equal(out[count - 1], pc.fv.square_relin(s.octx, cts[count - 1], s.evk))
        ref = emu.EmuContext(1024, s.q, s.p, s.t)
        ref.set_relin_key(backend.dev(s.evk))
        assert np.array_equal(out, ref.ct_square_relin(cts))
        ref.close()
    s.ctx.close()
    big = pc.Setup(backend, 32768, 30, with_keys=False)
    x = backend.dev(np.zeros((1, 2, 30, 32768), dtype=np.uint32))
    with pytest.raises(_capi.HcnnError) as err:
        big.ctx.ct_square_relin_noalloc(x, np.zeros_like(x))
    assert err.value.code == _capi.ERR["SCRATCH"]
    big.ctx.close()


def test_square_relin_exact_comparison_path(backend):
    pc.check_square_relin(backend, 1024, 2, force_exact=True)
    pc.check_square_relin(backend, 2048, 4, n_random=1, n_genuine=1, force_exact=True)


def test_square_relin_more_than_16_limbs(backend):
    # k = 17 > 16 exercises the intermediate reductions of the 64-bit inner products
    pc.check_square_relin(backend, 1024, 17, n_random=1, n_genuine=1)


@pytest.mark.parametrize("k,k_aux,big_t", [(3, 4, False), (5, 6, False), (6, 7, False), (7, 8, False), (8, 9, False),
                                           (9, 10, False), (10, 11, False), (11, 12, False), (12, 13, False),
                                           (4, 6, True), (6, 8, True), (8, 10, True), (10, 12, True), (11, 13, True),
                                           (12, 14, True), (14, 16, True), (16, 18, True), (24, 26, True)])
def test_square_relin_register_variants_of_standard_bases(backend, k, k_aux, big_t):
    # the basis sizes of the benchmark configurations, at a ring degree the oracle finishes quickly;
    # a larger plaintext modulus makes k' = k + 2 necessary already at n = 1024
    t = pc.slot_prime_above(1024, 1 << 22) if big_t else 65537
    pc.check_square_relin(backend, 1024, k, n_random=1, n_genuine=1, t=t, expect_k_aux=k_aux)
    pc.check_square_relin(backend, 1024, k, n_random=1, n_genuine=0, t=t, force_exact=True)


def test_square_relin_at_a_degree_with_die_aware_block_orders(backend):
    # n = 8192: 8 coefficient tiles per row, the size from which the inner-product kernel orders its
    # workgroups by accelerator die; three ciphertexts so that the ciphertext index is exercised too
    pc.check_square_relin(backend, 8192, 2, n_random=3, n_genuine=0)
    pc.check_square_relin(backend, 8192, 2, n_random=6, n_genuine=0, relin_order=2)    # key-major order forced
    # one ciphertext: the forced one-kernel relinearisation takes its single-round form (16 residues per thread)
    pc.check_square_relin(backend, 8192, 2, n_random=1, n_genuine=0)


def test_square_relin_largest_ring_two_workgroups_per_forward_row(backend):
    # n = 32768: the forward transforms run as two workgroups per row, out of place, the extended rows staged in the
    # array of the tensor
    pc.check_square_relin(backend, 32768, 2, n_random=2, n_genuine=0)


def test_largest_ring_with_whole_rows_and_with_halves():
    """n = 32768, 18 rows of the tensor: whole-row inverse transforms in front of the scaling while the rows, but not their halves, find a
    compute unit each; both ends of that range, squaring and product."""
    n, k, backend = 32768, 2, EmuBackend()
    s = pc.Setup(backend, n, k)
    cts = pc.gen.uniform_residues(s.rng, s.q, n, lead=(2, 2))
    square, product = pc.fv.square_relin(s.octx, cts[0], s.evk), pc.fv.hmult(s.octx, cts[0], cts[1], s.evk)
    rows = 3 * (k + len(s.p))
    for units, split in ((2 * rows, True), (2 * rows - 1, False), (rows, False), (rows - 1, True)):
        assert emu.rules().rule_splits_tensor_rows(units, n, rows) == split
        with emu.device(emu.lib(), units=units):
            ctx = backend.make_ctx(n, s.q, s.p, s.t)
        ctx.set_relin_key(backend.dev(s.evk))
        ctx.set_profile(True)
        assert np.array_equal(ctx.ct_square_relin(backend.dev(cts[:1]))[0], square), units
        assert ctx.profile()["tensor"][0] == 0
        assert np.array_equal(ctx.ct_mul_relin(backend.dev(cts[:1]), backend.dev(cts[1:]))[0], product), units
        ctx.close()


@pytest.mark.parametrize("k,options", [(2, dict(force_exact=True)), (3, dict(relin_order=1))])
def test_square_relin_largest_ring_by_halves(backend, k, options):
    # n = 32768: inverse transforms left at the halves of their rows, the scaling takes their last stage; the one-kernel tensor
    # (taken here by default) with the exact comparison in the scaling, and the separate kernels
    pc.check_square_relin(backend, 32768, k, n_random=1, n_genuine=0, **options)


def test_measure_ceiling_arguments(backend):
    # the diagnostic rejects an unknown probe; the host emulation does not time its launches and reports 0
    from paper_1811_00778_amd import _capi
    import ctypes
    s = pc.Setup(backend, 1024, 2, with_keys=False)
    v = ctypes.c_double(-1.0)
    lib = s.ctx.raw.lib
    assert lib.hcnn_measure_ceiling(s.ctx.raw.handle, len(_capi.CEILINGS), ctypes.byref(v)) == _capi.ERR["ARG"]
    assert lib.hcnn_measure_ceiling(s.ctx.raw.handle, -1, ctypes.byref(v)) == _capi.ERR["ARG"]
    assert lib.hcnn_measure_ceiling(s.ctx.raw.handle, 0, None) == _capi.ERR["NULL"]
    assert lib.hcnn_measure_ceiling(s.ctx.raw.handle, len(_capi.CEILINGS) - 1, ctypes.byref(v)) == 0 and v.value == 0.0
    s.ctx.close()


@pytest.mark.parametrize("k", [1, 9, 10, 11, 12, 13, 19, 20, 21, 22, 30])
def test_square_relin_folds_of_the_base_changes(backend, k):
    """Numbers of primes on both sides of the sums' folds (12 products, then 9 more), smallest and largest instance."""
    pc.check_square_relin(backend, 1024, k, n_random=1, n_genuine=0)


def test_general_hmult(backend):
    pc.check_mul_relin(backend, 1024, 2)
    pc.check_mul_relin(backend, 2048, 3, force_exact=True)
    pc.check_mul_relin(backend, 1024, 8)


def test_conv_square_layer(backend):
    pc.check_conv_layer_small(backend)


def test_random_parameter_sweep(backend):
    pc.check_random_sweep(backend, 6, seed=7, sizes=(1024,))


def test_counter_based_samplers(backend):
    pc.check_samplers(backend, 1024, 2)
    pc.check_samplers(backend, 2048, 3, seed_id=2)


def test_noise_read_out(backend):
    pc.check_noise_bits(backend, 1024, 2)
    pc.check_noise_bits(backend, 1024, 5)


def test_wide_plaintext_modulus(backend):
    pc.check_wide_plaintext(backend)
    pc.check_wide_plaintext(backend, 1024, 5, seed_id=2, force_exact=True)


def test_plaintext_crt_channels(backend):
    pc.check_crt_channels(backend)


def test_small_network_layer_by_layer(backend):
    pc.check_small_network(backend)


def test_wrappers_check_every_shape_before_the_call(backend):
    """The C ABI takes bare pointers, so the Python wrappers are the only place where a wrongly sized buffer can be
    caught before a kernel reads or writes past it: each argument's full shape is checked, and a scalar MAC whose
    output overlaps its input is refused."""
    n, k = 1024, 2
    s = pc.Setup(backend, n, k)
    ctx, dev = s.ctx, backend.dev
    kr = s.kr
    good = dict(s=dev(kr["s"]), a=dev(kr["a"]), e=dev(kr["e"]), a_evk=dev(kr["a_evk"]), e_evk=dev(kr["e_evk"]))
    ctx.keygen(**good)
    for name, bad in (("s", np.zeros(n // 2, np.int32)), ("a", np.zeros((k + 1, n), np.uint32)),
                      ("e", np.zeros((2, n), np.int32)), ("a_evk", np.zeros((k, k, n // 2), np.uint32)),
                      ("e_evk", np.zeros((k + 1, n), np.int32))):
        with pytest.raises(ValueError):
            ctx.keygen(**dict(good, **{name: dev(bad)}))
    with pytest.raises(ValueError):
        ctx.keygen(good["s"], good["a"], good["e"], good["a_evk"], None)
    slots, polys, er, cts = s.encrypt_oracle(2)
    pk, m, u, e1, e2 = dev(s.pk), dev(polys), dev(er["u"]), dev(er["e1"]), dev(er["e2"])
    ctx.encrypt(pk, m, u, e1, e2)
    with pytest.raises(ValueError):
        ctx.encrypt(dev(np.zeros((2, k, n // 2), np.uint32)), m, u, e1, e2)
    with pytest.raises(ValueError):
        ctx.encrypt(pk, m, dev(er["u"][:1]), e1, e2)
    with pytest.raises(ValueError):
        ctx.encrypt(pk, m, u, e1, dev(np.zeros((2, n + 4), np.int32)))
    dcts = dev(cts)
    with pytest.raises(ValueError):
        ctx.decrypt(dev(np.zeros(n + 1, np.int32)), dcts)
    with pytest.raises(ValueError):
        ctx.noise_bits(dev(np.zeros((1, n), np.int32)), dcts)
    ctx.set_relin_key(dev(s.evk))
    with pytest.raises(ValueError):
        ctx.ct_mul_relin(dcts, dcts, out=dev(np.zeros((1, 2, k, n), np.uint32)))
    with pytest.raises(ValueError):
        ctx.ct_square_relin(dcts, out=dev(np.zeros((3, 2, k, n), np.uint32)))
    idx, w = dev(np.array([[0, 1]], np.uint32)), dev(np.ones((1, 1, 2), np.int32))
    with pytest.raises(ValueError):
        ctx.ct_scalar_mac(dcts, idx, w, 1, out=dcts[:1].reshape((1, 1, 2, k, n)))        # overlaps its input
    with pytest.raises(ValueError):
        ctx.ct_scalar_mac(dcts, idx, dev(np.ones((1, 1, 3), np.int32)), 1)
    ctx.close()
