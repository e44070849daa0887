"""The rules that choose a kernel by its LDS ask what the device offers (CPU only).

Read through the library's own host functions: with less LDS than a kernel
would request, the rule leaves the call to the general kernels (the launch
would fail); with enough, it takes it.
"""
import ctypes
import glob
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.environ.get("VLASOV_LIB", os.path.join(ROOT, "paper_2110_15867_amd", "libvlasov.so"))
KB = 1024


class DriftAxis(ctypes.Structure):
    _fields_ = [("n", ctypes.c_int), ("nu", ctypes.c_int), ("umax", ctypes.c_double),
                ("du", ctypes.c_double), ("factor", ctypes.c_double)]


class DriftArgs(ctypes.Structure):
    _fields_ = [("x", DriftAxis), ("y", DriftAxis), ("nz", ctypes.c_int), ("nuz", ctypes.c_int),
                ("Nu", ctypes.c_long), ("W", ctypes.c_int), ("zi", ctypes.c_int),
                ("jchunks", ctypes.c_int), ("pair", ctypes.c_int)]


def _rule(name, *argtypes):
    if not os.path.exists(LIB):
        pytest.skip("libvlasov.so not built (run __graft_entry__.build())")
    f = ctypes.CDLL(LIB)[name]
    f.restype, f.argtypes = ctypes.c_bool, argtypes
    return f


# y cells, closing planes of a work-group's threads: 5 planes of S values for
# 64 threads per segment of S cells
@pytest.mark.parametrize("ny,need", [(8, 1 * 8 * 1280), (64, 8 * 8 * 1280), (121, 16 * 8 * 1280),
                                     (128, 16 * 8 * 1280)])
def test_fused_drifts_ask_for_their_lds(ny, need):
    rule = _rule("_ZN6vlasov18drift_yx_supportedERKNS_9DriftArgsEm", ctypes.POINTER(DriftArgs),
                 ctypes.c_size_t)
    a = DriftArgs(DriftAxis(16, 64, 1, 1, 1), DriftAxis(ny, 64, 1, 1, 1), 1, 64, 64 ** 3)
    assert rule(a, 160 * KB)
    assert rule(a, need)
    assert not rule(a, need - 1)


@pytest.mark.parametrize("n,need", [((160, 8, 8), (3 * 8 + 1) * 160 * 16), ((256, 8, 8), (3 * 8 + 1) * 256 * 16),
                                    ((8, 256, 8), (2 * 8 + 1) * 256 * 16),
                                    ((8, 8, 256), ((2 * 8 + 1) * 256 + 16 * 129) * 16)])
def test_field_transforms_ask_for_their_lds(n, need):
    rule = _rule("_ZN6vlasov19field_fft_supportedEPKim", ctypes.POINTER(ctypes.c_int),
                 ctypes.c_size_t)
    mesh = (ctypes.c_int * 3)(*n)
    assert rule(mesh, 160 * KB)
    assert rule(mesh, need)
    assert not rule(mesh, need - 1)
    assert not rule((ctypes.c_int * 3)(257, 8, 8), 160 * KB)


def test_arrays_of_16_byte_accesses_are_declared_so():
    """Dynamic LDS begins behind a kernel's static arrays, at the alignment the
    array is declared with: 16 bytes in every file that reads or writes it by
    groups of four floats."""
    csrc = os.path.join(ROOT, "paper_2110_15867_amd", "csrc")
    seen = 0
    for path in sorted(glob.glob(os.path.join(csrc, "*.h*"))):
        text = open(path).read()
        arrays = re.findall(r"(?:extern )?__shared__ [^;{]*\b(?:lds)\[[^;]*;", text)
        if not arrays or not re.search(r"reinterpret_cast<(?:const )?float(?:4|x4)\*>\((?:lds|line|tile|at)\b", text):
            continue
        seen += 1
        assert all("__align__(16)" in a for a in arrays), (os.path.basename(path), arrays)
    assert seen >= 3        # the kicks, the small meshes' drifts, the line tiles
