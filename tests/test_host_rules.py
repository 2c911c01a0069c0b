"""The library's dispatch rules, called as plain functions on the CPU (tests/host_rules.cpp): the sizes at which a rule can go
wrong are too large, or of too large a device, to be run through the entry points."""
import pytest

import emu
from paper_1811_00778_amd import _capi, network
from paper_1811_00778_amd._ops import OpsMixin


@pytest.fixture(scope="module")
def rules():
    return emu.rules()


# (858993409 terms: 13421773 times 320 words is 2^32 + 64)
@pytest.mark.parametrize("T", [1, 64, 65, 3264, 3265, (1 << 20) - 1, 1 << 20, (1 << 20) + 1, 858993409, 0xffffffff])
@pytest.mark.parametrize("bound", [0, 1, 127])
def test_matrix_form_tables_fit_the_lds_that_a_launch_asks_for(rules, T, bound):
    """A staged group takes 64 offsets and 256 weight words per 64 terms; a row whose tables do not fit stays with the
    vector forms, whatever the bound on its weights."""
    for groups in (1, 2):
        assert rules.rule_mac_matrix_lds(groups, T) == groups * ((T + 63) // 64) * 320 * 4
    for G, F in ((1, 1), (1, 16), (2, 16), (7, 16), (4, 3)):
        form = rules.rule_mac_matrix_groups(256, 1024, 2, 100, G, F, T, bound)
        assert form in (0, 1, 2) and form <= max(G, 1)
        if form:
            assert rules.rule_mac_matrix_lds(form, T) <= 64 * 1024 and T * bound <= 1 << 20
        if T > 3264:
            assert form == 0


@pytest.mark.parametrize("n,k,n_in,G,F,T,form", [
    (8192, 8, 784, 144, 5, 25, 0),            # few filters: vector
    (8192, 8, 784, 144, 13, 25, 0), (8192, 8, 784, 144, 14, 24, 0), (8192, 8, 784, 144, 14, 25, 2),
    (8192, 10, 4096, 64, 9, 576, 0), (8192, 10, 4096, 64, 10, 95, 0), (8192, 10, 4096, 256, 10, 96, 2),
    (8192, 10, 4096, 64, 16, 576, 2),
    (8192, 10, 2048, 16, 16, 192, 2), (8192, 10, 2048, 16, 16, 191, 0),        # every input gathered 1.5 times, or less
    (8192, 10, 2048, 16, 16, 128, 0), (1024, 2, 2048, 16, 16, 128, 2),         # ... where the launch fills the chip
    (8192, 8, 100, 2, 10, 96, 2), (8192, 8, 100, 3, 10, 96, 1), (8192, 8, 100, 6, 10, 96, 1), (8192, 8, 100, 7, 10, 96, 2),
    (8192, 8, 845, 1, 8, 64, 1), (8192, 8, 845, 1, 8, 63, 0), (8192, 8, 845, 1, 7, 64, 0),
    (32768, 24, 64, 1, 16, 64, 0),            # one group that fills the chip
    (8192, 8, 2000, 9, 16, 1600, 2), (8192, 8, 2000, 9, 16, 1601, 1),          # two groups' tables in 64 KiB, or one's
    (8192, 8, 4000, 9, 4, 3264, 0), (8192, 8, 4000, 9, 5, 3264, 1), (8192, 8, 4000, 9, 16, 3265, 0),
])
def test_form_of_the_scalar_mac(rules, n, k, n_in, G, F, T, form):
    """Both sides of every line of the rule, on a device of 256 compute units."""
    assert rules.rule_mac_matrix_groups(256, n, k, n_in, G, F, T, 15) == form
    assert rules.rule_mac_matrix_groups(256, n, k, n_in, G, F, T, 128) == 0          # weights beyond a signed byte


@pytest.mark.parametrize("groups,n,k,G,T,steps", [
    (1, 1024, 2, 130, 1601, 1), (1, 1024, 9, 130, 1601, 8),                       # 1 block at eight tiles per wave (2 at four, 4 at two), 5
    (1, 8192, 3, 130, 1700, 4), (1, 8192, 4, 130, 1700, 8),                       # 12, 16
    (1, 8192, 5, 130, 1700, 4), (1, 8192, 7, 130, 1700, 8),                       # 20, 28
    (2, 1024, 2, 600, 25, 4), (2, 1024, 3, 300, 25, 8), (2, 2048, 3, 256, 1200, 4),      # 4, 6, 12
    (0, 1024, 2, 600, 300, 2), (0, 1024, 3, 600, 144, 4), (0, 2048, 3, 256, 144, 8),     # 2, 3, 6
    (0, 4096, 3, 256, 288, 4), (0, 4096, 5, 256, 288, 4), (0, 4096, 6, 256, 288, 8), (0, 4096, 7, 256, 288, 8),       # 12, 20, 24, 28
    (0, 8192, 8, 64, 511, 8), (0, 8192, 8, 64, 512, 4), (0, 2048, 3, 256, 576, 2),       # long rows start from four tiles: 128 blocks, 12
    (0, 8192, 8, 32, 25, 8), (0, 8192, 8, 30, 25, 4), (0, 8192, 8, 9, 25, 2), (0, 1024, 3, 7, 25, 1),      # too few workgroups
])
def test_tiles_per_wave_of_the_matrix_forms(rules, groups, n, k, G, T, steps):
    """No die waits for a last round that few of them have; blocks of tiles at the number that a form starts from beside the cases."""
    assert rules.rule_mac_matrix_steps(groups, 256, n, k, G, T) == steps


@pytest.mark.parametrize("n,k,n_in,G,T,pairs", [
    (8192, 8, 8191, 64, 576, 1), (8192, 8, 8192, 64, 576, 0),                      # inputs of 4 GiB
    (8192, 8, 1000, 64, 1088, 1), (8192, 8, 1000, 64, 1089, 0),                    # tables of 80 KiB: terms
    (1024, 3, 115552, 1000, 300, 1), (1024, 3, 115553, 1000, 300, 0),              # ... inputs
    (8192, 8, 81, 31, 25, 1), (8192, 8, 81, 30, 25, 0), (8192, 8, 81, 9, 25, 0),   # short rows: 8, 4, 2 tiles per wave
    (8192, 8, 81, 32, 25, 1), (8192, 8, 81, 33, 25, 0),                            # 16 and 17 pairs: four and five rounds of workgroups
    (8192, 8, 900, 30, 95, 0), (8192, 8, 900, 30, 96, 1),                          # longer ones: 4 tiles per wave
    (8192, 8, 900, 9, 270, 0), (8192, 8, 900, 9, 271, 1), (8192, 8, 900, 14, 238, 0), (8192, 8, 900, 14, 239, 1),      # 2
    (8192, 8, 2429, 30, 144, 1), (8192, 8, 2430, 30, 144, 0),                      # inputs that fewer rows share
    (2048, 3, 7500, 576, 142, 0), (2048, 3, 7500, 576, 143, 1), (2048, 4, 9408, 729, 48, 1),     # blocks of tiles for six dies, for all
    (4096, 3, 800, 300, 59, 0), (4096, 3, 800, 300, 60, 1),                        # 12 blocks of eight tiles, taken at four
    (1024, 2, 800, 1000, 147, 0), (1024, 2, 800, 1000, 148, 1),                    # a ring of 64 tiles: two per wave whatever the groups
    (1024, 3, 12274, 225, 370, 0), (1024, 3, 12274, 225, 371, 1),                  # one
    (8192, 10, 4096, 64, 576, 1),
])
def test_calls_that_form_the_union_of_two_rows(rules, n, k, n_in, G, T, pairs):
    """Both sides of every line, on a device of 256 compute units."""
    assert rules.rule_mac_takes_pairs(256, n, k, n_in, G, T) == pairs


@pytest.mark.parametrize("n,k,n_in,G,F,T,bound,groups", [
    (8192, 8, 784, 144, 5, 25, 15, 3), (8192, 8, 784, 144, 1, 25, 127, 16), (8192, 8, 784, 144, 8, 25, 15, 2), (8192, 8, 784, 144, 9, 25, 15, 0),
    (8192, 8, 784, 144, 5, 25, 128, 0),                                            # weights beyond a signed byte
    (8192, 8, 800, 112, 5, 25, 15, 3), (8192, 8, 801, 112, 5, 25, 15, 0),          # inputs gathered 3.5 times
    (8192, 8, 2916, 63, 6, 277, 15, 0), (8192, 8, 2916, 63, 6, 278, 15, 2), (8192, 8, 2916, 64, 6, 273, 15, 2), (4096, 8, 2916, 63, 6, 277, 15, 2),
    (8192, 8, 2101, 63, 6, 199, 15, 2), (8192, 8, 2100, 63, 6, 200, 15, 2), (8192, 8, 2101, 63, 6, 200, 15, 0),    # few groups of many terms
    (2048, 2, 720, 64, 1, 125, 15, 0), (2048, 3, 720, 64, 1, 125, 15, 16),         # 128, 192 workgroups
    (8192, 8, 8191, 1200, 2, 27, 15, 8), (8192, 8, 8192, 1200, 2, 27, 15, 0),      # inputs of 4 GiB
    (1024, 1, 1000, 10000, 8, 1568, 15, 2), (1024, 1, 1000, 10000, 8, 1569, 15, 0),    # tables of 64 KiB
])
def test_calls_of_few_filters_that_sum_groups_side_by_side(rules, n, k, n_in, G, F, T, bound, groups):
    assert rules.rule_mac_pack_groups(256, n, k, n_in, G, F, T, bound) == groups


@pytest.mark.parametrize("n,k,n_in,G,F,T,groups", [
    # multiply-adds a coefficient times workgroups of the vector form per compute unit: below 150, from there on
    (2048, 4, 25, 25, 3, 9, 0), (4096, 3, 81, 36, 1, 16, 0),
    (8192, 4, 50, 9, 3, 22, 0), (8192, 4, 50, 9, 3, 23, 5), (4096, 4, 64, 33, 4, 9, 0), (4096, 4, 64, 34, 4, 9, 4),
    # one and two filters in launches that do not fill the chip
    (2048, 3, 490, 16, 1, 160, 0), (2048, 3, 720, 63, 1, 125, 0), (2048, 3, 720, 64, 1, 125, 16),
    (2048, 4, 1176, 25, 2, 216, 0), (2048, 4, 1176, 31, 2, 216, 0), (2048, 4, 1176, 32, 2, 216, 8), (2048, 4, 1176, 31, 3, 216, 5),
])
def test_small_calls_of_few_filters_stay_in_the_vector_form(rules, n, k, n_in, G, F, T, groups):
    assert rules.rule_mac_pack_groups(256, n, k, n_in, G, F, T, 15) == groups


@pytest.mark.parametrize("n,k,n_in,G,F,T,steps", [
    (8192, 8, 784, 144, 5, 25, 8),
    # four groups of 5 x 5 rows, r = 6.25: unions of 2.2 rows, 1.21 T terms of them for what they are built of
    (8192, 8, 1568, 400, 4, 24, 8), (8192, 8, 3200, 400, 4, 50, 4), (8192, 8, 6336, 400, 4, 99, 4), (8192, 8, 6400, 400, 4, 100, 2),
    (32768, 17, 46, 69, 1, 46, 8), (32768, 17, 1024, 69, 1, 1024, 4),      # all groups over the same inputs: a sixteenth
    (16384, 13, 1127, 9, 7, 575, 2), (8192, 11, 2106, 36, 4, 416, 2), (2048, 4, 3200, 49, 6, 288, 2), (2048, 4, 1152, 16, 6, 288, 1),
])
def test_long_unions_of_groups_side_by_side_take_few_tiles_per_wave(rules, n, k, n_in, G, F, T, steps):
    assert rules.rule_mac_pack_steps(256, n, k, n_in, G, F, T) == steps


def test_network_plan_puts_16_outputs_into_rows_that_the_matrix_form_takes(rules):
    """The length and the weights up to which the plan relies on the matrix form for rows that the vector form cannot stage."""
    T, weight = network._MATRIX_TERMS, network._MATRIX_WEIGHT
    for units, n, k in ((256, 1024, 2), (256, 32768, 24), (1, 1024, 1)):
        for G in (1, 2, 4, 9):
            form = lambda terms, bound: rules.rule_mac_matrix_groups(units, n, k, 5000, G, 16, terms, bound)
            assert form(T, weight) == 1 and form(T + 1, weight) == 0 and form(T, weight + 1) == 0 and form(1000, weight) > 0


@pytest.mark.parametrize("n,k,least", [(32768, 11, 0), (32768, 12, 16), (32768, 13, 5), (32768, 17, 5), (32768, 18, 4), (32768, 32, 4),
                                       (16384, 15, 0), (16384, 16, 64), (16384, 32, 64), (8192, 32, 0)])
def test_smallest_batch_of_the_shared_basis_relinearisation(rules, n, k, least):
    assert rules.rule_shared_basis_min(n, k, k + 1) == least
    assert rules.rule_shared_basis_min(n, k, 0) == 0           # no auxiliary primes: no squarings


@pytest.mark.parametrize("n,k,n_ct,halves", [
    (8192, 8, 16, True), (8192, 8, 17, False), (8192, 2, 64, True), (8192, 2, 65, False), (8192, 10, 8, True), (8192, 10, 9, False), (8192, 10, 12, False),
    (8192, 16, 1, True), (8192, 17, 1, False), (8192, 26, 2, False), (32768, 4, 28, True), (32768, 6, 16, True), (32768, 6, 17, False), (32768, 6, 18, False),
    (32768, 10, 11, False), (32768, 12, 8, True), (32768, 12, 9, False), (32768, 16, 8, True), (32768, 24, 1, False), (4096, 4, 1, False), (16384, 8, 1, False),
])
def test_decryptions_by_halves_fit_the_compute_units_of_every_die(rules, n, k, n_ct, halves):
    assert bool(rules.rule_decrypts_by_halves(256, n, k, n_ct)) == halves


def test_two_decryption_workgroups_of_the_second_largest_ring_fit_a_compute_unit(rules):
    assert 2 * rules.rule_decrypt_lds() <= 160 * 1024


@pytest.mark.parametrize("n_ct,L", [(1, 5), (1, 8), (3, 17), (7, 9), (64, 17), (225, 34), (32, 50)])
def test_one_kernel_tensor_takes_every_pair_once_in_the_order_of_the_limbs(rules, n_ct, L):
    rows = n_ct * L
    pairs = [rules.rule_tensor_place(0, n_ct, L, i) for i in range(rows)]
    assert sorted(pairs) == list(range(rows))
    for die in range(8):                                       # each die's limbs ascend, and its share of the pairs is even
        limbs = [p % L for p in pairs[die::8]]
        assert limbs == sorted(limbs) and len(limbs) in (rows // 8, rows // 8 + 1)
    # two workgroups per pair: (pair, half) of a place as the split transforms read it; those past the last pair stay past it
    places = [rules.rule_tensor_place(1, n_ct, L, i) for i in range(2 * -(-rows // 8) * 8)]
    taken = [(b // 16 * 8 + b % 8, b // 8 % 2) for b in places]
    assert sorted(t for t in taken if t[0] < rows) == [(p, h) for p in range(rows) for h in (0, 1)]
    assert [p for p, h in taken if p < rows and h == 0] == pairs


@pytest.mark.parametrize("n,least", [(1024, 448), (2048, 640), (4096, 320), (8192, 384), (16384, 0), (32768, 320)])
def test_binding_reports_the_rule_of_the_one_kernel_tensor(rules, n, least):
    """What the binding works out from the library's figures against the rule itself, on a device of 256 compute units."""
    assert rules.rule_tensor_fused_least(n) == least
    k, k_aux, per_unit = 3, 5, 2

    class Raw:
        stats = {_capi.STAT_TENSOR_FUSED_WGS: 256 * per_unit, _capi.STAT_TENSOR_FUSED_LEAST: least}

        def stat(self, which):
            return self.stats[which]

    ops = OpsMixin()
    ops.raw = Raw()
    ops.raw.n, ops.raw.k, ops.raw.k_aux = n, k, k_aux
    took = [ops.takes_tensor_fused(n_ct) for n_ct in range(1, 700)]
    assert took == [bool(rules.rule_takes_tensor_fused(256, per_unit, n, k, k_aux, n_ct)) for n_ct in range(1, 700)]
    threshold = ops.tensor_fused_threshold()
    assert all(took[-(-threshold // (k + k_aux)) - 1:])
    assert threshold == (least // (2 if n == 32768 else 1) if least else 49 * 512 // 8)


@pytest.mark.parametrize("n,k,n_ct,rest,least", [
    # up to n = 4096: longer workgroups of more primes, later; ciphertexts in fours later still
    (1024, 2, 8, False, 16), (1024, 3, 7, False, 16), (1024, 3, 8, False, 52), (1024, 4, 7, False, 32), (1024, 4, 8, False, 128), (1024, 6, 9, False, 108), (1024, 6, 12, False, 432),
    (1024, 16, 7, False, 512), (1024, 16, 8, False, 512), (2048, 1, 148, False, 40), (2048, 3, 44, False, 52),
    (2048, 4, 7, False, 40), (2048, 4, 8, False, 128), (2048, 8, 7, False, 256), (2048, 32, 8, False, 512),
    (4096, 6, 7, False, 96), (4096, 6, 8, False, 144), (4096, 9, 9, False, 162), (4096, 8, 16, False, 192), (4096, 10, 8, False, 200), (4096, 12, 32, False, 288),
    (4096, 3, 8, False, 96), (4096, 20, 7, False, 512), (4096, 20, 8, False, 512),
    (1024, 8, 8, True, 8), (2048, 8, 8, True, 20), (4096, 12, 8, True, 48), (8192, 8, 8, True, 96), (16384, 8, 8, True, 68),
    # from n = 8192 on: does the fullest die have a compute unit for each of its workgroups?
    (8192, 8, 32, False, 192), (8192, 8, 33, False, 288), (8192, 10, 24, False, 192), (8192, 10, 25, False, 288), (16384, 16, 16, False, 136), (16384, 16, 17, False, 288),
])
def test_workgroups_from_which_the_one_kernel_relinearisation_is_taken(rules, n, k, n_ct, rest, least):
    assert rules.rule_relin_fused_least(256, n, k, n_ct, rest) == least


@pytest.mark.parametrize("per_unit,n,k,n_ct,whole,takes", [
    # n = 16384: halves of 12 limbs on a die, 32 workgroups a round; 39 and 40 ciphertexts fill the second round, 23 put four into it, 28 ten, 29 sixteen
    (1, 16384, 12, 39, 32, True), (1, 16384, 12, 40, 32, True), (1, 16384, 12, 41, 32, False), (1, 16384, 12, 23, 16, False), (1, 16384, 12, 28, 16, False),
    (1, 16384, 12, 29, 16, True), (1, 16384, 12, 20, 16, True), (1, 16384, 12, 21, 16, False),
    # all 11 limbs on a die: 55 ciphertexts end in the round that 48 begin, 17 put one workgroup into a new one
    (1, 16384, 11, 55, 48, True), (1, 16384, 11, 17, 16, False), (1, 16384, 16, 17, 16, False), (1, 16384, 16, 24, 16, True),
    # other rings count the rest's workgroups
    (2, 8192, 8, 75, 64, False), (2, 8192, 8, 76, 64, True), (2, 8192, 8, 24, 0, True), (2, 8192, 8, 23, 0, False),
])
def test_rest_behind_whole_rounds_of_the_one_kernel_relinearisation(rules, per_unit, n, k, n_ct, whole, takes):
    assert bool(rules.rule_relin_fused_takes_rest(256, per_unit, n, k, n_ct, whole)) == takes


@pytest.mark.parametrize("n,per_units", [(1024, (4, 16, 32)), (2048, (4, 8, 16)), (4096, (2, 4, 8)), (8192, (2, 3)), (16384, (1,))])
def test_work_buffer_holds_every_batch_that_the_separate_kernels_take(rules, n, per_units):
    """Whatever the rules leave to the separate kernels, behind no, one or three whole rounds, fits what is allocated for them."""
    for per_unit in per_units:
        for k in range(1, 17 if n == 16384 else 33):
            fused_round = 256 * per_unit // 8 // k * 8
            most = rules.rule_relin_split_most(n, k, fused_round)
            for whole in (0, fused_round, 3 * fused_round):
                left = [rest for rest in range(1, fused_round) if not rules.rule_relin_fused_takes_rest(256, per_unit, n, k, whole + rest, whole)]
                assert not left or max(left) <= most, (per_unit, k, whole)


@pytest.mark.parametrize("n,k,share", [(8192, 7, 7), (8192, 8, 4), (8192, 9, 9), (8192, 12, 6), (16384, 6, 3), (16384, 16, 8), (4096, 6, 6), (4096, 12, 6)])
def test_one_kernel_relinearisation_halves_the_limbs_of_a_die(rules, n, k, share):
    assert rules.rule_relin_share(n, k) == share
    for n_ct in (1, 3, 8, 37):
        rows = [rules.rule_relin_row(i, share) for i in range(rules.rule_relin_grid(n_ct * k, share))]
        assert sorted(r for r in rows if r < n_ct * k) == list(range(n_ct * k))
        for die in range(8):                                   # a die meets one part of the limbs only
            assert len({r % k // share for r in rows[die::8] if r < n_ct * k}) <= 1
