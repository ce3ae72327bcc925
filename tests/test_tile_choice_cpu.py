"""Which kernels a sweep takes when the tuning cache holds an entry for it,
checked on the host: an entry that was not timed against resident tiles does
not turn them off, one that was faster than them for its extents does."""
import ctypes

import numpy as np
import pytest

from paper_2001_01473_amd import _lib

s5d = pytest.importorskip("paper_2001_01473_amd")
KW = dict(ndim=2, radius=1, box=False, dtype="f64", steps=100, coeffs=np.full(5, 0.2))


def _tile(interior):
    """(rows, columns) of the resident tile a plan without tuning runs on, (0, 0) if it streams."""
    p = s5d.Plan(interior=interior, **KW)
    r, c = ctypes.c_int32(-1), ctypes.c_int32(-1)
    n = _lib.load().s5d_internal_rounds(p._h, ctypes.c_double(1.0), ctypes.byref(r), ctypes.byref(c))
    p.close()
    assert n > 0
    return r.value, c.value


@pytest.fixture(autouse=True)
def _empty_cache():
    s5d.tune_cache_clear()
    yield
    s5d.tune_cache_clear()


def test_untuned_plans():
    assert _tile((512, 512)) in ((64, 64), (64, 128))
    assert _tile((16384, 16384)) == (0, 0)


def test_model_ranked_entry_keeps_tiles():
    want = _tile((512, 512))
    s5d.autotune(top_k=0, interior=(512, 512), **KW)
    assert _tile((512, 512)) == want


def test_entry_of_an_older_file_keeps_tiles(tmp_path):
    want = _tile((512, 512))
    f = tmp_path / "old.txt"
    f.write_text("2 0 1 1 0 0 9 9 0 : 9 128 0 32 2 0 : 2.25e-06 : 512 512 1\n")
    s5d.tune_cache_load(f)
    assert _tile((512, 512)) == want


def test_entry_measured_faster_than_tiles(tmp_path):
    other = _tile((500, 480))
    assert other != (0, 0)
    f = tmp_path / "new.txt"
    f.write_text("2 0 1 1 0 0 9 9 0 : 9 128 0 32 2 0 : 2.25e-07 : 512 512 1 : 1\n")
    s5d.tune_cache_load(f)
    saved = tmp_path / "saved.txt"
    s5d.tune_cache_save(saved)  # the mark survives a save and a load
    s5d.tune_cache_clear()
    s5d.tune_cache_load(saved)
    assert _tile((512, 512)) == (0, 0)  # the extents it was measured for
    assert _tile((500, 480)) == other   # others of the same bucket
