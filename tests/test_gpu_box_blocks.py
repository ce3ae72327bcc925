"""Stream blocks of the heavy boxes are cut for the waves that pay: one a SIMD for
2D boxes of radius 3 and 4, whatever the kernel's registers let in, and the
workgroups that fit a CU for the 125-point box."""
import pytest

import paper_2001_01473_amd as s5d
import numpy as np
import stencil_inputs as si
from gpu_util import torch

pytestmark = pytest.mark.gpu


def _chosen(rows, tiles, slots, warmup, least):
    """The block length of the chooser's cost: the blocks' work over the slots, and
    a tail of 0.75 blocks."""
    best, h_best = float("inf"), rows
    for n in range(1, max(1, rows // least) + 1):
        h = -(-rows // n)
        per = h + warmup
        cost = max(tiles * -(-rows // h) / slots, 1.0) * per + 0.75 * per
        if cost < best * (1 - 1e-9):
            best, h_best = cost, h
    return h_best


@pytest.mark.parametrize("dtype,r,bt,width", [("f32", 3, 2, 240), ("f32", 4, 1, 248), ("f64", 4, 1, 248), ("f64", 3, 2, 242)])
@pytest.mark.parametrize("interior", [(3000, 4100), (8000, 8000)])
def test_wide_2d_boxes(dtype, r, bt, width, interior):
    cus = torch().cuda.get_device_properties(0).multi_processor_count
    c = si.random_coeffs(np.random.default_rng(1496), si.n_points(2, r, True))
    plan = s5d.Plan(ndim=2, radius=r, box=True, dtype=dtype, interior=interior, steps=2 * bt, coeffs=c)
    q = plan.query()
    plan.close()
    assert (q["bt"], q["cells_per_lane"]) == (bt, 4)
    tiles = -(-interior[1] // width)
    assert q["stream_chunk"] == _chosen(interior[0], tiles, 4 * cus, 2 * bt * r, max(8, bt * r))


def test_125_point_box_one_workgroup():
    cus = torch().cuda.get_device_properties(0).multi_processor_count
    c = si.random_coeffs(np.random.default_rng(1497), 125)
    plan = s5d.Plan(ndim=3, radius=2, box=True, dtype="f32", interior=(256, 256, 256), steps=2, coeffs=c, bt=1,
                    rows_per_wave=4, kernel=1)
    q = plan.query()
    plan.close()
    tiles = -(-256 // 28) * -(-256 // 124)  # 32 rows and 128 columns less the overlap
    assert q["stream_chunk"] == _chosen(256, tiles, cus, 4, 8)
