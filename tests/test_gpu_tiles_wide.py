"""Resident tiles of 64 x 128 cells (two columns a lane), which mid-sized grids
take: every stencil, on ragged grids of several interior tiles, against the
kernels that stream.  The tile a plan runs on is asked for."""
import ctypes

import numpy as np
import pytest

import paper_2001_01473_amd as s5d
import stencil_inputs as si
from gpu_util import say, torch
from paper_2001_01473_amd import _lib

pytestmark = pytest.mark.gpu

DT = {"f32": np.float32, "f64": np.float64, "f32c": np.float32}
SIZES = [(1000, 1101), (1403, 1290), (2051, 1902)]
STENCILS = [("linear", r, False) for r in (1, 2, 3, 4)] + [("linear", 1, True), ("linear", 2, True), ("div", 1, False),
                                                         ("div", 2, False), ("div", 1, True), ("gradient", 1, False)]


def _tile(plan):
    r, c = ctypes.c_int32(-1), ctypes.c_int32(-1)
    _lib.load().s5d_internal_rounds(plan._h, ctypes.c_double(1.0), ctypes.byref(r), ctypes.byref(c))
    return r.value, c.value


@pytest.mark.parametrize("kind", ["f32", "f64", "f32c"])
@pytest.mark.parametrize("expr,r,box", STENCILS)
def test_wide_tiles_equal_streaming_kernels(kind, expr, r, box):
    if kind == "f32c" and expr != "linear":
        pytest.skip("compensated sums are built for the plain stencils")
    if kind == "f32c" and (r == 4 or (r == 2 and box)):
        pytest.skip("the estimate takes the narrow tile or the one-step kernel for these")
    t = torch()
    rng = np.random.default_rng(1493)
    u = rng.random(si.n_points(2, r, box))
    c = [0.3, 1.5] if expr == "gradient" else list(u) + [float(u.sum())] if expr == "div" else list(u / u.sum())
    shapes = set()
    for interior in SIZES:
        for T in (7, 26, 100):
            kw = dict(ndim=2, radius=r, box=box, dtype=DT[kind], interior=interior, steps=T, coeffs=c, expr=expr,
                      accum="compensated" if kind == "f32c" else "plain")
            plan = s5d.Plan(**kw)
            tile = _tile(plan)
            shapes.add(tile)
            if tile != (64, 128):
                plan.close()
                continue
            other = s5d.Plan(**kw, **(dict(kernel=2) if expr == "linear" else dict(bt=1)))
            assert _tile(other) == (0, 0)
            x = t.rand(si.padded_shape(interior, r), dtype=t.float64 if kind == "f64" else t.float32, device="cuda:0")
            say("wide tiles", kind, expr, r, box, interior, T)
            outs = []
            for p in (plan, other):
                a, b = x.clone(), t.full_like(x, float("nan"))
                idx = p.run(a, b)
                t.cuda.synchronize()
                outs.append((a, b)[idx])
                p.close()
            assert t.equal(outs[0], outs[1]), (interior, T)
    assert (64, 128) in shapes, shapes
