"""The divided stencils' quotient over its whole range: one centre weight of one
makes each step the IEEE quotient x / c0, the oracle's bits."""
import numpy as np
import pytest

import oracle
import paper_2001_01473_amd as s5d
import stencil_inputs as si
from gpu_util import say, torch

pytestmark = pytest.mark.gpu

# inside the reciprocal's range, at its ends, below one, negative, far outside
DIVISORS = [118.0, 1.0, 3.0, -7.25, 0.7, 1.3 * 2.0 ** -20, 2.0 ** -21, 2.0 ** 60, 1.1 * 2.0 ** 60, 1e30, 1e-30]


def _values(dtype, shape, seed):
    """Every exponent, subnormals, zeros of both signs, the largest value."""
    rng = np.random.default_rng(seed)
    f = np.finfo(dtype)
    lo, hi = int(np.log2(f.smallest_subnormal)), f.maxexp - 1
    x = np.ldexp(rng.uniform(1, 2, shape), rng.integers(lo, hi + 1, shape)) * rng.choice([-1.0, 1.0], shape)
    x[rng.random(shape) < 0.3] = rng.random()
    with np.errstate(over="ignore", under="ignore"):
        x = np.clip(x, f.min, f.max).astype(dtype)
    flat = x.reshape(-1)
    flat[rng.permutation(flat.size)[:40]] = np.resize(
        np.array([0.0, -0.0, f.max, f.min, f.tiny, f.smallest_subnormal, np.inf, -np.inf, np.nan], dtype), 40)
    return x


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("interior,r,box,tune", [
    ((70, 300), 1, False, dict(bt=1, kernel=1)), ((70, 300), 1, False, dict(bt=3, kernel=1)),
    ((70, 300), 1, False, {}), ((40, 131), 2, False, dict(bt=2, kernel=1)), ((40, 131), 1, True, {}),
    ((9, 40, 130), 1, True, {})], ids=lambda v: str(v).replace(" ", ""))
def test_quotient(interior, r, box, tune, dtype):
    t = torch()
    nd = len(interior)
    n = si.n_points(nd, r, box)
    c = np.zeros(n)
    c[n // 2] = 1.0
    for k, d in enumerate(DIVISORS):
        for T in (1, 3):
            c0 = dtype(d)
            say("quotient", interior, r, box, dtype.__name__, d, T)
            grid = _values(dtype, si.padded_shape(interior, r), 1485 + k)
            plan = s5d.Plan(ndim=nd, radius=r, box=box, dtype=dtype, interior=interior, steps=T,
                            coeffs=list(c) + [float(c0)], expr="div", **tune)
            x = t.from_numpy(grid).to("cuda:0")
            y = t.full_like(x, 0.0)
            idx = plan.run(x, y)
            t.cuda.synchronize()
            got = (x if idx == 0 else y).cpu().numpy()
            plan.close()
            with np.errstate(all="ignore"):
                want = oracle.sweep_div(grid, radius=r, box=box, coeffs=c.astype(dtype), divisor=c0, steps=T)
            np.testing.assert_array_equal(got, want, err_msg="c0 = %g, T = %d" % (d, T))
            np.testing.assert_array_equal(np.signbit(got[got == 0]), np.signbit(want[got == 0]))
