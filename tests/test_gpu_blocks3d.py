"""3D kernels that a batch and a server launch for larger grids, and the block
lengths of large ones, against single runs and the direct kernel's bits."""
import numpy as np
import pytest

import paper_2001_01473_amd as s5d
import stencil_inputs as si
from gpu_util import run_gpu, say, torch

pytestmark = pytest.mark.gpu

# plain stars of 2^20 cells and more, which march: odd extents and unequal ones
MARCH = [((101, 103, 109), 3), ((47, 150, 161), 4), ((131, 83, 97), 4), ((60, 170, 131), 3)]


def _march_plans(dtype):
    t = torch()
    rng = np.random.default_rng(1494)
    out = []
    for k, (interior, r) in enumerate(MARCH):
        c = si.random_coeffs(rng, si.n_points(3, r, False))
        plan = s5d.Plan(ndim=3, radius=r, box=False, dtype=dtype, interior=interior, steps=3 + k, coeffs=c)
        assert plan.query()["tile0"] >= 32
        x = t.from_numpy(rng.random(si.padded_shape(interior, r)).astype(dtype)).to("cuda:0")
        out.append((plan, x))
    return out


def _alone(plan, x):
    t = torch()
    a, b = x.clone(), t.full_like(x, float("nan"))
    idx = plan.run(a, b)
    t.cuda.synchronize()
    return (a, b)[idx]


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("graph", [False, True])
def test_marching_in_a_batch(dtype, graph):
    t = torch()
    made = _march_plans(dtype)
    want = [_alone(p, x) for p, x in made]
    b0 = [x.clone() for _, x in made]
    b1 = [t.full_like(x, float("nan")) for x in b0]
    batch = s5d.Batch([p for p, _ in made], b0, b1, graph=graph)
    for replay in range(3):
        say("marching batch", dtype.__name__, graph, replay)
        for x, (_, g) in zip(b0, made):
            x.copy_(g)
        idx = batch.run()
        t.cuda.synchronize()
        for i, w in enumerate(want):
            assert t.equal((b0[i], b1[i])[idx[i]], w), (replay, i)
    batch.close()
    for p, _ in made:
        p.close()


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_marching_served(dtype):
    t = torch()
    made = _march_plans(dtype)
    want = [_alone(p, x) for p, x in made]
    server = s5d.Server(hbm_budget_bytes=1 << 30)
    say("marching served", dtype.__name__)
    ids = [server.submit(p, x, keep_result=True) for p, x in made]
    running, queued = server.tick()
    while running or queued:
        running, queued = server.tick()
    server.sync()
    for i, w in zip(ids, want):
        out = t.empty_like(w)
        server.fetch(i, out)
        assert t.equal(out, w)
    server.close()


# T = 1: short blocks, of 4 or 6 planes or by the chooser; over 450 MB a buffer
# the float32 7-point star's blocks of 20 planes
@pytest.mark.parametrize("dtype,r,box,interior,T,chunk", [
    (np.float32, 1, False, (130, 330, 330), 1, 6), (np.float64, 1, False, (130, 330, 330), 1, 4),
    (np.float64, 1, True, (130, 330, 330), 1, None), (np.float64, 2, False, (130, 330, 330), 1, None),
    (np.float32, 1, False, (430, 530, 517), 4, 20)])
def test_blocks_of_large_grids(dtype, r, box, interior, T, chunk):
    t = torch()
    c = si.random_coeffs(np.random.default_rng(1495), si.n_points(3, r, box))
    kw = dict(ndim=3, radius=r, box=box, dtype=dtype, interior=interior, steps=T, coeffs=c)
    plan, direct = s5d.Plan(**kw), s5d.Plan(**kw, kernel=2)
    q = plan.query()
    if chunk is not None:
        assert q["stream_chunk"] == chunk
    elif r == 1:
        assert q["stream_chunk"] < 34  # not the whole turns of deeper rounds
    x = t.rand(si.padded_shape(interior, r), dtype=t.float64 if dtype == np.float64 else t.float32, device="cuda:0")
    say("large blocks", dtype.__name__, r, box, interior, T, q["stream_chunk"])
    assert t.equal(_alone(plan, x), _alone(direct, x))
    plan.close()
    direct.close()
