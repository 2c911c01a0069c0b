"""CPU checker for the kernel sources (test helper, not collected by pytest).

Builds paper_1811_00778_amd/csrc/hcnn.cpp with -DHCNN_HOSTEMU (g++, no HIP): the same
kernel phase bodies and the same host orchestration run as loops over blocks and
threads on host memory.  Lets the CPU test-suite compare kernel indexing and
arithmetic with the oracle before anything runs on a GPU.  The product binding never
loads this library.
"""
import ctypes
import os
import subprocess

import numpy as np

from paper_1811_00778_amd import _capi
from paper_1811_00778_amd._ops import OpsMixin

_ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
_SRC_DIR = os.path.join(_ROOT, "paper_1811_00778_amd", "csrc")
_OUT_DIR = os.path.join(_ROOT, "tests", "_build")
# HCNN_EMU_SANITIZE=1: build and load the checker with AddressSanitizer and UndefinedBehaviorSanitizer (host code
# only: this is the one build in which the kernels' indexing runs under a bounds checker).  The sanitizer runtime
# has to be in the process before Python starts, so run it as
#     HCNN_EMU_SANITIZE=1 LD_PRELOAD=$(g++ -print-file-name=libasan.so) ASAN_OPTIONS=detect_leaks=0 \
#         python -m pytest tests/test_emu_parity.py -q
SANITIZE = os.environ.get("HCNN_EMU_SANITIZE", "") not in ("", "0")
_OUT = os.path.join(_OUT_DIR, "libhcnn_emu_san.so" if SANITIZE else "libhcnn_emu.so")
_lib = _lib_shared = _lib_rules = None


def build(defines=(), out=_OUT, source=os.path.join(_SRC_DIR, "hcnn.cpp")) -> str:
    os.makedirs(_OUT_DIR, exist_ok=True)
    srcs = [os.path.join(_SRC_DIR, f) for f in os.listdir(_SRC_DIR)] + [os.path.join(_ROOT, "include", "hcnn.h"), source]
    if os.path.exists(out) and all(os.path.getmtime(s) <= os.path.getmtime(out) for s in srcs):
        return out
    tmp = out + ".tmp.%d" % os.getpid()
    extra = ["-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-fno-omit-frame-pointer"] \
        if SANITIZE else ["-O2"]
    subprocess.check_call(["g++", "-std=c++17"] + extra + ["-DHCNN_HOSTEMU", *defines, "-fPIC", "-shared", "-Wall", "-Wextra",
                           "-Wno-unused-parameter", "-Wno-unknown-pragmas", "-o", tmp,
                           source])
    os.replace(tmp, out)
    return out


def lib():
    global _lib
    if _lib is None:
        _lib = _capi.declare(ctypes.CDLL(build()))
    return _lib


def lib_shared_basis():
    """The checker with the shared-basis relinearisation taken by every ring and basis (the rule of the product waits
    for parameter sets that the oracle is slow at)."""
    global _lib_shared
    if _lib_shared is None:
        _lib_shared = _capi.declare(ctypes.CDLL(build(["-DHCNN_SHARED_ALL"], _OUT.replace(".so", "_shared.so"))))
    return _lib_shared


def rules():
    """The host-side rules of tests/host_rules.cpp."""
    global _lib_rules
    if _lib_rules is None:
        lib = ctypes.CDLL(build(["-O0"], _OUT.replace("libhcnn_emu", "libhcnn_rules"), os.path.join(_ROOT, "tests", "host_rules.cpp")))
        lib.rule_mac_matrix_groups.argtypes = [ctypes.c_uint32] * 7 + [ctypes.c_int32]
        lib.rule_mac_takes_pairs.argtypes = [ctypes.c_uint32] * 6
        lib.rule_mac_pack_groups.argtypes, lib.rule_mac_pack_groups.restype = [ctypes.c_uint32] * 7 + [ctypes.c_int32], ctypes.c_uint32
        lib.rule_mac_matrix_steps.argtypes, lib.rule_mac_matrix_steps.restype = [ctypes.c_uint32] * 6, ctypes.c_uint32
        lib.rule_mac_pack_steps.argtypes, lib.rule_mac_pack_steps.restype = [ctypes.c_uint32] * 7, ctypes.c_uint32
        lib.rule_mac_matrix_lds.argtypes, lib.rule_mac_matrix_lds.restype = [ctypes.c_uint32, ctypes.c_size_t], ctypes.c_size_t
        lib.rule_takes_tensor_fused.argtypes = [ctypes.c_uint32] * 5 + [ctypes.c_size_t]
        lib.rule_tensor_fused_least.argtypes, lib.rule_tensor_fused_least.restype = [ctypes.c_uint32], ctypes.c_size_t
        lib.rule_relin_fused_least.argtypes, lib.rule_relin_fused_least.restype = [ctypes.c_uint32] * 3 + [ctypes.c_size_t, ctypes.c_int], ctypes.c_size_t
        lib.rule_relin_fused_takes_rest.argtypes = [ctypes.c_uint32] * 4 + [ctypes.c_size_t] * 2
        lib.rule_relin_split_most.argtypes, lib.rule_relin_split_most.restype = [ctypes.c_uint32, ctypes.c_uint32, ctypes.c_size_t], ctypes.c_size_t
        lib.rule_splits_tensor_rows.argtypes = [ctypes.c_uint32] * 2 + [ctypes.c_size_t]
        lib.rule_decrypts_by_halves.argtypes = [ctypes.c_uint32] * 3 + [ctypes.c_size_t]
        lib.rule_decrypt_lds.restype = ctypes.c_size_t
        for name in ("rule_relin_share", "rule_relin_grid", "rule_relin_row"):
            getattr(lib, name).argtypes, getattr(lib, name).restype = [ctypes.c_uint32] * 2, ctypes.c_uint32
        lib.rule_tensor_place.argtypes, lib.rule_tensor_place.restype = [ctypes.c_uint32] * 4, ctypes.c_uint32
        lib.rule_shared_basis_min.argtypes, lib.rule_shared_basis_min.restype = [ctypes.c_uint32] * 3, ctypes.c_size_t
        _lib_rules = lib
    return _lib_rules


class device:
    """The checker's device while the block runs: compute units that contexts made in it see, largest allocation granted."""

    def __init__(self, library, units=1, largest=2 ** 64 - 1):
        self.set, self.args = library.hcnn_emu_device, (units, largest)
        self.set.argtypes, self.set.restype = [ctypes.c_uint32, ctypes.c_size_t], None

    def __enter__(self):
        self.set(*self.args)

    def __exit__(self, *_):
        self.set(1, 2 ** 64 - 1)


class EmuContext(OpsMixin):
    def __init__(self, n, q, p, t, library=None):
        self.raw = _capi.RawContext(library or lib(), n, q, p, t, 0)

    def _ptr(self, x):
        return ctypes.c_void_p(x.ctypes.data)

    _NP = {"u32": np.uint32, "i32": np.int32, "u64": np.uint64}

    def _empty(self, shape, dtype_name):
        return np.empty(shape, dtype=self._NP[dtype_name])

    def _check(self, x, dtype_name):
        want = self._NP[dtype_name]
        if not isinstance(x, np.ndarray) or x.dtype != want or not x.flags["C_CONTIGUOUS"]:
            raise TypeError("expected contiguous %s ndarray" % want.__name__)
        if x.ctypes.data % 16:
            raise TypeError("array not 16-byte aligned")


def aligned(a):
    """Copy of a in 16-byte aligned storage (numpy gives 16-byte alignment for fresh allocations)."""
    out = np.empty(a.shape, dtype=a.dtype)
    assert out.ctypes.data % 16 == 0
    out[...] = a
    return out
