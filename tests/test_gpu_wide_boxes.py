"""The coefficients of the 49-point box stay in scalar registers in boundary
waves at every depth: spilled to vector lanes they tripled a step's time."""
import numpy as np
import pytest

import paper_2001_01473_amd as s5d
import stencil_inputs as si
from gpu_util import say, torch

pytestmark = pytest.mark.gpu


def _us_per_step(bt):
    t = torch()
    interior, T = (3000, 4100), 2 * bt
    c = si.random_coeffs(np.random.default_rng(1487), si.n_points(2, 3, True))
    plan = s5d.Plan(ndim=2, radius=3, box=True, dtype="f32", interior=interior, steps=T, coeffs=c, bt=bt, kernel=1)
    x = t.rand(si.padded_shape(interior, 3), device="cuda:0")
    y = t.empty_like(x)
    plan.run(x, y)
    e0, e1 = t.cuda.Event(enable_timing=True), t.cuda.Event(enable_timing=True)
    best = float("inf")
    for _ in range(5):
        e0.record()
        plan.run(x, y)
        e1.record()
        e1.synchronize()
        best = min(best, e0.elapsed_time(e1))
    plan.close()
    return 1e3 * best / T


def test_box2d3r_deep_rounds():
    say("box2d3r f32 b_T = 3")
    base = _us_per_step(3)
    for bt in (4, 5):
        say("box2d3r f32 b_T =", bt)
        us = _us_per_step(bt)
        assert us < 2 * base, "b_T = %d: %.1f us a step, %.1f at b_T = 3" % (bt, us, base)
