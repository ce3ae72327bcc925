"""Marching one-step kernels of 3D stars (grids of 2^20 cells on) at the edges
of their tiles and blocks of planes: the oracle's bits on dyadic inputs, its
bound on random ones, and the blocked kernels' bits at radius 2."""
import numpy as np
import pytest

import oracle
import stencil_inputs as si
from gpu_util import rel_errors, run_gpu, say

pytestmark = pytest.mark.gpu

# rows and columns at and around multiples of the tiles' 26, 28 and 56 rows and
# 56, 120 and 124 columns, odd pitches, plane counts that leave partial blocks
SIZES = [(40, 169, 157), (33, 56, 573), (131, 83, 97)]


@pytest.mark.parametrize("interior", SIZES)
@pytest.mark.parametrize("r", [2, 3, 4])
def test_march_dyadic_bitwise(r, interior):
    case = si.make_dyadic_case(1480 + r, 3, r, False, interior, 2)
    for dtype in (np.float32, np.float64):
        c, g = case.as_dtype(dtype)
        say("march dyadic", r, interior, dtype.__name__)
        got, info = run_gpu(g, radius=r, box=False, coeffs=case.coeffs, steps=2, kernel=2)
        assert info["kernel"] == 2
        want = oracle.sweep(g, radius=r, box=False, coeffs=c, steps=2)
        np.testing.assert_array_equal(got, want)


@pytest.mark.parametrize("r", [2, 3, 4])
def test_march_random(r):
    rng = np.random.default_rng(1484)
    interior = (47, 150, 161)
    c = si.random_coeffs(rng, si.n_points(3, r, False))
    g = rng.random(si.padded_shape(interior, r))
    say("march random", r)
    got, _ = run_gpu(g, radius=r, box=False, coeffs=c, steps=5, kernel=2)
    ref = oracle.sweep(g, radius=r, box=False, coeffs=c, steps=5)
    assert max(rel_errors(got, ref)) <= 1e-12
    if r == 2:
        blocked, _ = run_gpu(g, radius=r, box=False, coeffs=c, steps=5, bt=1, kernel=1)
        np.testing.assert_array_equal(got, blocked)
