"""A served request's share of the machine: what it is of the work that the server
holds, whatever has finished, failed or been cancelled before."""
import ctypes

import numpy as np
import pytest

import paper_2001_01473_amd as s5d
import stencil_inputs as si
from gpu_util import say, torch
from paper_2001_01473_amd import _lib

pytestmark = pytest.mark.gpu


def _rounds(plan, share):
    fn = _lib.load().s5d_internal_rounds
    fn.restype = ctypes.c_int64
    r, c = ctypes.c_int32(-1), ctypes.c_int32(-1)
    return fn(plan._h, ctypes.c_double(share), ctypes.byref(r), ctypes.byref(c))


def _plan(n, T):
    return s5d.Plan(ndim=2, radius=1, box=False, dtype="f64", interior=(n, n), steps=T, coeffs=np.full(5, 0.2))


def _drain(server):
    running, queued = server.tick()
    while running or queued:
        running, queued = server.tick()
    server.sync()


def test_share_of_the_held_work():
    t = torch()
    big, small = _plan(2600, 300), _plan(1300, 300)
    share = 1300 ** 2 / (1300 ** 2 + 2600 ** 2)
    assert _rounds(small, 1.0) != _rounds(small, share)  # the sizes tell the shares apart
    grids = {p: t.rand(si.padded_shape((n, n), 1), dtype=t.float64, device="cuda:0") for p, n in ((big, 2600), (small, 1300))}
    server = s5d.Server(hbm_budget_bytes=1 << 30, fail_admit_every=3)
    say("held work: mixed requests")
    ids = [server.submit(p, grids[p]) for p in (big, small, big, small, big)]  # the third fails
    server.tick()
    server.cancel(ids[0])   # running
    late = server.submit(big, grids[big])
    server.cancel(late)     # queued
    _drain(server)
    say("held work: one request after them")
    alone = server.submit(small, grids[small])  # the sixth admission fails, this one is the seventh or earlier
    _drain(server)
    if server.request(alone)["state"] == _lib.REQ_FAILED:
        alone = server.submit(small, grids[small])
        _drain(server)
    assert server.request(alone)["rounds_done"] == _rounds(small, 1.0)
    say("held work: two requests")
    while True:
        pair = [server.submit(p, grids[p]) for p in (small, big)]
        _drain(server)
        if all(server.request(i)["state"] != _lib.REQ_FAILED for i in pair):
            break
    assert server.request(pair[0])["rounds_done"] == _rounds(small, share)
    server.close()
