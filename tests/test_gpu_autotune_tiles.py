"""Autotuning a small 2D grid: the baseline it reports is what a plan without
tuning runs, resident tiles included, and they stay on where they are faster."""
import ctypes

import numpy as np
import pytest

import paper_2001_01473_amd as s5d
import stencil_inputs as si
from gpu_util import run_gpu, say
from paper_2001_01473_amd import _lib

pytestmark = pytest.mark.gpu


def _tile(**kw):
    p = s5d.Plan(**kw)
    r, c = ctypes.c_int32(-1), ctypes.c_int32(-1)
    _lib.load().s5d_internal_rounds(p._h, ctypes.c_double(1.0), ctypes.byref(r), ctypes.byref(c))
    p.close()
    return r.value, c.value


@pytest.mark.parametrize("earlier", [False, True], ids=["empty", "streaming entry"])
def test_small_grid_stays_on_tiles(earlier, tmp_path):
    case = si.make_case(si.item_seed(9, 4), 2, 1, False, (512, 512), 100)
    kw = dict(ndim=2, radius=1, box=False, dtype=np.float64, interior=(512, 512), steps=100, coeffs=case.coeffs)
    s5d.tune_cache_clear()
    try:
        want, _ = run_gpu(case.grid, radius=1, box=False, coeffs=case.coeffs, steps=100)
        tile = _tile(**kw)
        assert tile != (0, 0)
        if earlier:  # said to be faster than tiles, and is not
            f = tmp_path / "entry.txt"
            f.write_text("2 0 1 1 0 0 9 9 0 : 9 128 0 32 2 0 : 2.25e-07 : 512 512 1 : 1\n")
            s5d.tune_cache_load(f)
            assert _tile(**kw) == (0, 0)
        say("autotune 512^2", earlier)
        _, rep = s5d.autotune(top_k=3, **kw)
        assert rep["n_measured"] == 3
        assert rep["best_seconds_per_step"] <= rep["default_seconds_per_step"]
        if not earlier:
            assert rep["best_seconds_per_step"] == rep["default_seconds_per_step"]
        assert _tile(**kw) == tile  # over 2 times as fast as the best streaming blocking
        got, _ = run_gpu(case.grid, radius=1, box=False, coeffs=case.coeffs, steps=100)
        np.testing.assert_array_equal(got, want)
    finally:
        s5d.tune_cache_clear()
