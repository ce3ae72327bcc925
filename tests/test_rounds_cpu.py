"""The rounds of a sweep are kept as runs of equal depth: a plan of any number of
steps takes no memory for them and launches what the schedule says."""
import ctypes
import subprocess
import sys

import numpy as np
import pytest

from paper_2001_01473_amd import _lib

s5d = pytest.importorskip("paper_2001_01473_amd")


def _rounds(**kw):
    p = s5d.Plan(coeffs=np.full(5, 0.2), ndim=2, radius=1, box=False, **kw)
    fn = _lib.load().s5d_internal_rounds
    fn.restype = ctypes.c_int64
    r, c = ctypes.c_int32(-1), ctypes.c_int32(-1)
    n = fn(p._h, ctypes.c_double(1.0), ctypes.byref(r), ctypes.byref(c))
    p.close()
    return n


@pytest.mark.parametrize("bt", [1, 2, 3, 7, 10])
def test_number_of_rounds(bt):
    for T in list(range(0, 45)) + [1000, 1001]:
        n = _rounds(dtype="f32", interior=(3000, 3000), steps=T, bt=bt, kernel="blocked")
        assert n % 2 == T % 2
        least = -(-T // bt)
        assert least <= n <= least + 1, T


_SNIPPET = r"""
import sys
sys.path[:0] = [%r, %r]
import test_rounds_cpu as t
print(t._rounds(dtype="f32", interior=(300, 300), steps=1 << 45), t._rounds(dtype="f64", interior=(9000, 9000), steps=1 << 45))
"""


def test_any_number_of_steps():
    """(In a process of its own: a list of the rounds would not fit its memory.)"""
    import os
    here = os.path.dirname(os.path.abspath(__file__))
    out = subprocess.run([sys.executable, "-c", _SNIPPET % (os.path.dirname(here), here)], capture_output=True, text=True,
                         timeout=300)
    assert out.returncode == 0, out.stderr[-500:]
    a, b = (int(v) for v in out.stdout.split())
    assert a >= (1 << 45) // 20 and b >= (1 << 45) // 10
