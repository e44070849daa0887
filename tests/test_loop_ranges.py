"""The kernels' grid-stride loops end for every size a grid may have (CPU only).

A loop `for (T i = ..; i < n; i += stride)` leaves with i up to a stride above
n, which T must hold: if it wraps instead, the loop runs on with indices
outside its arrays and never ends.  Such sizes take minutes and tens of GB on
the device, so the loops are read from the sources: the type of every counter
that advances by a multiple of blockDim.x, against the largest count it is
compared with.
"""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2110_15867_amd", "csrc")
TYPE_MAX = {"int": 2 ** 31 - 1, "unsigned": 2 ** 32 - 1, "long": 2 ** 63 - 1}
BLOCK = 2 ** 31 - 1          # cells of a velocity block, and of the spatial mesh (dims_of)
LDS = 160 * 1024 // 2        # values of any kind that LDS holds
# The largest value of each bound.  A loop with a bound not named here fails
# the test: name it, with what limits it.
LARGEST = {
    "lpc": BLOCK, "a.nsub": BLOCK, "a.Nu": BLOCK,           # lines, values of a velocity block
    "nv": LDS, "nl": LDS, "nlz": LDS,                       # k_kick_any: blocks in LDS
    "n": LDS, "m * kLines": LDS, "n * kLines": LDS, "total": LDS,   # transforms of lines in LDS
    "2 * kLines * nh": LDS, "2 * kLines * n": LDS,
}
MAX_STRIDE = 1024 * 4 * 8    # threads, values of a vector, loads in flight


def _loops():
    pat = re.compile(r"for \((?:const )?(\w+) (\w+) = [^;]*; *\2 < ([^;]+); *\2 \+= ([^;{]*blockDim[^;{]*)\)")
    for path in sorted(glob.glob(os.path.join(CSRC, "*.h*"))):
        for m in pat.finditer(open(path).read()):
            yield os.path.basename(path), m.group(1), m.group(3).strip()


def test_grid_stride_counters_hold_their_bound_and_a_stride():
    loops = list(_loops())
    assert len(loops) >= 15
    assert ("adjoint.hip", "lpc") in {(f, b) for f, _, b in loops}
    for where, ctype, bound in loops:
        assert bound in LARGEST, (where, bound)
        assert LARGEST[bound] + MAX_STRIDE <= TYPE_MAX[ctype], (where, ctype, bound)
