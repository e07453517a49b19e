"""Where two steps share a launch (step_pair): which runs take pairs, values
that are not finite in their sensors, and buffers beyond 2 GiB."""
import numpy as np
import pytest

import lbm_inputs
from lbm_inputs import PERIODIC, WALL
from test_gpu_steps import _PAIR, _lid

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lbm():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1507_06767_amd as lbm
    return lbm


def _per_launch(lbm, blk, every):
    st, n = lbm.abi.lbm_get_steps_per_launch(blk.h, every)
    assert st == lbm.LBM_OK
    return n


@pytest.mark.parametrize("q,n,storage,kind,force,every,steps", [
    (19, (64, 64, 64), 1, 0, 0.0, 0, 1),           # 6.9 us a step alone, 9.8 in pairs
    (19, (128, 128, 128), 1, 1, 0.0, 1, 1),        # 52.5, 59.1
    (19, (2048, 32, 32), 1, 0, 0.0, 1, 1),         # 49.5, 55.2
    (19, (2048, 32, 32), 1, 0, 0.0, 0, 1),         # 48.3, 49.5
    (19, (144, 144, 144), 2, 0, 1e-6, 0, 1),       # 70.3, 71.4
    (19, (256, 256, 48), 2, 0, 1e-6, 0, 2),        # 72.1, 65.3
    (19, (256, 256, 48), 1, 1, 0.0, 1, 1),         # 72.8, 82.4
    (19, (204, 100, 84), 2, 0, 1e-6, 0, 1),        # 43.2, 45.0
    (19, (128, 128, 128), 1, 0, 0.0, 0, 2),        # 48.5, 43.8
    (19, (32, 32, 2048), 1, 0, 0.0, 1, 2),         # 86, 54
    (19, (192, 192, 192), 1, 0, 0.0, 1, 2),        # 200, 150
    (19, (24, 24, 24), 0, 0, 0.0, 1, 2),           # 10.5, 9.4
    (9, (256, 256, 1), 1, 0, 0.0, 0, 1),
    (19, (128, 128, 128), 3, 0, 0.0, 0, 1),
])
def test_the_rule_takes_the_shorter_form(lbm, monkeypatch, q, n, storage, kind, force, every, steps):
    """Steps per launch of grids whose two forms differ (us per step measured
    one by one and in pairs)."""
    monkeypatch.delenv("LBM_PAIR", raising=False)
    print(f"\n[case] rule q={q} {n} storage={storage} kind={kind} every={every}", flush=True)
    bc = (WALL,) * 4 + ((PERIODIC,) * 2 if q == 9 else (WALL,) * 2)
    blk = lbm.Blocks(lbm.make_desc(q, n, bc, 0.65, storage=storage, sensor_kind=kind, wall_u=_lid(0.05),
                                   force=(force, 0.0, 0.0)))
    assert _per_launch(lbm, blk, every) == steps
    blk.close()
