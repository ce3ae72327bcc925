"""Which direct kernel a plain 3D star of radius 2..4 takes: marching where it is
the faster one for the grid's shape, and no search at every launch."""
import time

import numpy as np
import pytest

import paper_2001_01473_amd as s5d
import stencil_inputs as si
from gpu_util import run_gpu, say, torch

pytestmark = pytest.mark.gpu

# (interior, type, radius, marches): few planes, one plane, four rows, few tiles,
# of whole lane vectors, where row streaming takes a third to two thirds of the
# time; rows of a few cells and of odd pitch, where marching does
SHAPES = [((4, 512, 512), "f32", 4, False), ((1, 1024, 1024), "f32", 3, False), ((1024, 4, 1024), "f32", 4, False),
          ((64, 64, 512), "f32", 3, False), ((64, 64, 256), "f64", 3, False),
          ((700, 700, 60), "f32", 4, True), ((1024, 1024, 4), "f64", 2, True), ((2000, 26, 56), "f64", 4, True),
          ((420, 512, 483), "f32", 4, True), ((300, 300, 512), "f64", 3, True)]


@pytest.mark.parametrize("interior,dtype,r,marches", SHAPES)
def test_direct_kernel_for_the_shape(interior, dtype, r, marches):
    c = si.random_coeffs(np.random.default_rng(1490), si.n_points(3, r, False))
    plan = s5d.Plan(ndim=3, radius=r, box=False, dtype=dtype, interior=interior, steps=1, coeffs=c, kernel=2)
    q = plan.query()
    plan.close()
    assert (q["tile0"] >= 32) == marches  # rows of a workgroup's tile; row streaming has none


@pytest.mark.parametrize("interior", [(9, 40, 3000), (40, 9, 3000), (3000, 9, 40), (1100, 1000, 1)])
def test_narrow_grids_same_bits(interior):
    r = 2
    rng = np.random.default_rng(1491)
    c = si.random_coeffs(rng, si.n_points(3, r, False))
    g = rng.random(si.padded_shape(interior, r))
    say("narrow", interior)
    got, _ = run_gpu(g, radius=r, box=False, coeffs=c, steps=3, kernel=2)
    want, _ = run_gpu(g, radius=r, box=False, coeffs=c, steps=3, bt=1, kernel=1)
    np.testing.assert_array_equal(got, want)


def test_long_grid_is_not_searched_at_every_launch():
    t = torch()
    interior = (1 << 20, 1, 1)
    c = si.random_coeffs(np.random.default_rng(1492), si.n_points(3, 2, False))
    plan = s5d.Plan(ndim=3, radius=2, box=False, dtype="f32", interior=interior, steps=50, coeffs=c, kernel=2)
    x = t.rand(si.padded_shape(interior, 2), device="cuda:0")
    y = t.empty_like(x)
    say("long grid")
    plan.run(x, y)
    t.cuda.synchronize()
    t0 = time.perf_counter()
    plan.run(x, y)
    host = time.perf_counter() - t0
    t.cuda.synchronize()
    plan.close()
    # 51 launches of some 5 us each; half a million block lengths took over a
    # millisecond at every one
    assert host < 0.02
