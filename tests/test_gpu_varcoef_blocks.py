"""Stream blocks of a narrow grid with per-cell weights: as many as there are
waves resident, which LDS limits to two a CU at radius 2, b_T = 4, so that the
launch takes one turn of them."""
import pytest

import paper_2001_01473_amd as s5d
from gpu_util import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("interior", [(6965, 8), (1500, 1500), (200, 5000)])
def test_blocks_fit_the_resident_waves(interior):
    cus = torch().cuda.get_device_properties(0).multi_processor_count
    # LDS of a wave: 9 rows of 256 cells and 7 rows of 9 weights of 256 cells
    waves = (160 * 1024) // ((9 + 7 * 9) * 256 * 4)
    assert waves == 2
    plan = s5d.Plan(ndim=2, radius=2, box=False, dtype="f32", interior=interior, steps=20, expr="varcoef")
    q = plan.query()
    plan.close()
    assert q["bt"] == 4
    tiles = -(-interior[1] // 236)  # 256 columns less an overlap of 10 on either side
    assert tiles * -(-interior[0] // q["stream_chunk"]) <= waves * cus
