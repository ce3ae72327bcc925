"""Depth, rows per wave and stream blocks that the library chooses for a 3D
grid: the direct kernel's bits alone and in a batch, whatever the extents."""
import numpy as np
import pytest

import paper_2001_01473_amd as s5d
import stencil_inputs as si
from gpu_util import run_gpu, say, torch

pytestmark = pytest.mark.gpu

# one cell and one plane; fewer planes than a block's warm-up; one tile and one
# more column; one turn of the CUs and two; short blocks at b_T = 1
SIZES = [(1, 1, 1), (1, 40, 130), (3, 33, 127), (50, 60, 70), (7, 25, 241), (130, 101, 97), (64, 250, 190)]


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("r,box", [(1, False), (2, False), (1, True)])
def test_default_equals_direct(r, box, dtype):
    t = torch()
    rng = np.random.default_rng(1486)
    c = si.random_coeffs(rng, si.n_points(3, r, box))
    plans, bufs, wants = [], [], []
    for interior in SIZES:
        grid = rng.random(si.padded_shape(interior, r)).astype(dtype)
        for T in (1, 2, 7):
            say("depth3d", r, box, dtype.__name__, interior, T)
            got, info = run_gpu(grid, radius=r, box=box, coeffs=c, steps=T)
            assert info["bt"] <= T
            want, _ = run_gpu(grid, radius=r, box=box, coeffs=c, steps=T, kernel=2)
            np.testing.assert_array_equal(got, want, err_msg="%s T = %d" % (interior, T))
        # the last ones together: stream blocks for a share of the machine
        plans.append(s5d.Plan(ndim=3, radius=r, box=box, dtype=dtype, interior=interior, steps=7, coeffs=c))
        x = t.from_numpy(grid).to("cuda:0")
        bufs.append((x, t.full_like(x, float("nan"))))
        wants.append(want)
    say("depth3d batch", r, box, dtype.__name__)
    batch = s5d.Batch(plans, [x for x, _ in bufs], [y for _, y in bufs])
    idx = batch.run()
    t.cuda.synchronize()
    for k, want in enumerate(wants):
        got = bufs[k][idx[k]].cpu().numpy()
        np.testing.assert_array_equal(got, want, err_msg="batch %s" % (SIZES[k],))
    batch.close()
