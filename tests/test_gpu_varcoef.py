"""Per-cell weights at the edges of their tiles: every depth gives the bits of
depth 1, and the oracle's result within its bounds."""
import numpy as np
import pytest

import oracle
import paper_2001_01473_amd as s5d
import stencil_inputs as si
from gpu_util import rel_errors, say, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("r,box", [(1, False), (2, False), (1, True)])
def test_varcoef_depths_at_tile_edges(r, box, dtype):
    t = torch()
    rng = np.random.default_rng(1475)
    n, T = si.n_points(2, r, box), 9
    # one cell; below, at and above the 128- and 256-column tiles; pitches of
    # every 16-byte phase; several stream blocks
    for interior in ((1, 1), (7, 119), (13, 127), (40, 254), (33, 300), (21, 513)):
        grid = rng.random(si.padded_shape(interior, r)).astype(dtype)
        u = rng.random((n,) + interior)
        fields = (u / u.sum(axis=0)).astype(dtype)
        f = t.from_numpy(fields).to("cuda:0")
        outs = []
        for bt in (1, 2, 3, 4):
            say("varcoef", r, box, dtype.__name__, interior, bt)
            plan = s5d.Plan(ndim=2, radius=r, box=box, dtype=dtype, interior=interior, steps=T, expr="varcoef", bt=bt,
                            stream_chunk=11)
            x = t.from_numpy(grid).to("cuda:0")
            y = t.full_like(x, float("nan"))
            idx = plan.run(x, y, fields=f)
            t.cuda.synchronize()
            outs.append((x if idx == 0 else y).cpu().numpy())
            plan.close()
        for bt, out in zip((2, 3, 4), outs[1:]):
            np.testing.assert_array_equal(out, outs[0], err_msg="%s b_T = %d" % (interior, bt))
        ref = oracle.sweep_varcoef(grid.astype(np.float64), radius=r, box=box, cfield=fields.astype(np.float64), steps=T)
        if dtype == np.float64:
            assert max(rel_errors(outs[0], ref)) <= 1e-12
        else:
            # T steps of at most n roundings of values in [0, 1], weights summing to one within n roundings
            u32 = 2.0 ** -24
            assert np.max(np.abs(outs[0].astype(np.float64) - ref)) <= T * 2 * n * u32
