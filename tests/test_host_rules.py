"""The library's dispatch rules, called as plain functions on the CPU (tests/host_rules.cpp): the sizes at which a rule can go
wrong are too large, or of too large a device, to be run through the entry points."""
import ctypes
import os

import pytest

import emu

_U = ctypes.c_uint32


@pytest.fixture(scope="module")
def rules():
    lib = ctypes.CDLL(emu.build(["-O0"], emu._OUT.replace("libhcnn_emu", "libhcnn_rules"), os.path.join(emu._ROOT, "tests", "host_rules.cpp")))
    lib.rule_mac_matrix_groups.argtypes = [_U] * 7 + [ctypes.c_int32]
    lib.rule_mac_matrix_lds.argtypes, lib.rule_mac_matrix_lds.restype = [_U, ctypes.c_size_t], ctypes.c_size_t
    return lib


# (858993409 terms: 13421773 times 320 words is 2^32 + 64)
@pytest.mark.parametrize("T", [1, 64, 65, 3264, 3265, (1 << 20) - 1, 1 << 20, (1 << 20) + 1, 858993409, 0xffffffff])
@pytest.mark.parametrize("bound", [0, 1, 127])
def test_matrix_form_tables_fit_the_lds_that_a_launch_asks_for(rules, T, bound):
    """A staged group takes 64 offsets and 256 weight words per 64 terms; a row whose tables do not fit stays with the
    vector forms, whatever the bound on its weights."""
    for groups in (1, 2, 4):
        assert rules.rule_mac_matrix_lds(groups, T) == groups * ((T + 63) // 64) * 320 * 4
    for G, F in ((1, 1), (1, 16), (2, 16), (7, 16), (4, 3)):
        form = rules.rule_mac_matrix_groups(256, 1024, 2, 100, G, F, T, bound)
        assert form in (0, 1, 2, 4) and form <= max(G, 1)
        if form:
            assert rules.rule_mac_matrix_lds(form, T) <= 64 * 1024 and T * bound <= 1 << 20
        if T > 3264:
            assert form == 0
