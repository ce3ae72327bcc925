"""Resident-tile kernels of small 2D grids (default plans), at the edges of
their tiles: bit for bit the plain one-step kernels' result where those exist,
and the oracle's bounds."""
import numpy as np
import pytest

import oracle
import paper_2001_01473_amd as s5d
import stencil_inputs as si
from gpu_util import rel_errors, say, torch

pytestmark = pytest.mark.gpu

DT = {"f32": np.float32, "f64": np.float64, "f32c": np.float32}


def _run(kind, expr, r, box, interior, T, coeffs, grid, **tuning):
    t = torch()
    plan = s5d.Plan(ndim=2, radius=r, box=box, dtype=DT[kind], interior=interior, steps=T, coeffs=coeffs, expr=expr,
                    accum="compensated" if kind == "f32c" else "plain", **tuning)
    x = t.from_numpy(grid).to("cuda:0")
    y = t.full_like(x, float("nan"))  # every interior cell has to be written
    idx = plan.run(x, y)
    t.cuda.synchronize()
    plan.close()
    return (x if idx == 0 else y).cpu().numpy()


# one cell, a row, a column, below / at / above multiples of the tiles' 64
# rows and 64 or 128 columns less the overlap, ragged rows of odd pitch
SIZES = [(1, 1), (1, 200), (150, 1), (47, 63), (48, 112), (49, 113), (64, 128), (131, 257)]


@pytest.mark.parametrize("kind", ["f32", "f64", "f32c"])
@pytest.mark.parametrize("r,box", [(1, False), (2, False), (3, False), (4, False), (1, True), (2, True)])
def test_tiles_equal_direct_kernels(kind, r, box):
    rng = np.random.default_rng(1473)
    c = si.random_coeffs(rng, si.n_points(2, r, box))
    for interior in SIZES:
        grid = rng.random(si.padded_shape(interior, r)).astype(DT[kind])
        for T in (1, 2, 7, 26):
            say("tiles", kind, r, box, interior, T)
            got = _run(kind, "linear", r, box, interior, T, c, grid)
            want = _run(kind, "linear", r, box, interior, T, c, grid, kernel=2)
            np.testing.assert_array_equal(got, want, err_msg="%s T=%d" % (interior, T))
    if kind == "f64":
        ref = oracle.sweep(grid, radius=r, box=box, coeffs=c, steps=T)
        assert max(rel_errors(got, ref)) <= 1e-12
    elif kind == "f32c":
        ref = oracle.sweep(grid, radius=r, box=box, coeffs=c.astype(np.float32), steps=T, accum="compensated")
        np.testing.assert_array_equal(got, ref)


@pytest.mark.parametrize("kind", ["f32", "f64"])
@pytest.mark.parametrize("expr,r,box", [("div", 1, False), ("div", 2, False), ("div", 1, True), ("gradient", 1, False)])
def test_expression_tiles_equal_blocked_kernels(kind, expr, r, box):
    rng = np.random.default_rng(1474)
    u = rng.random(si.n_points(2, r, box))
    c = [0.3, 1.5] if expr == "gradient" else list(u) + [float(u.sum())]
    for interior in SIZES:
        grid = rng.random(si.padded_shape(interior, r)).astype(DT[kind])
        for T in (1, 2, 7, 26):
            say("expression tiles", kind, expr, r, box, interior, T)
            got = _run(kind, expr, r, box, interior, T, c, grid)
            want = _run(kind, expr, r, box, interior, T, c, grid, bt=1)
            np.testing.assert_array_equal(got, want, err_msg="%s T=%d" % (interior, T))
