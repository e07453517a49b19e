"""Step kernel variants at the sizes where they can go wrong: the float64
block maxima of 3D grids, folded by one atomic maximum per workgroup."""
import numpy as np
import pytest

import lbm_inputs
from lbm_inputs import PERIODIC, WALL

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lbm():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1507_06767_amd as lbm
    return lbm


def _lid(speed):
    w = [[0.0] * 3 for _ in range(6)]
    w[3][0] = speed
    return w


@pytest.mark.parametrize("kind", [0, 1], ids=["l2", "kkn"])
@pytest.mark.parametrize("q,n", [(19, (5, 6, 3)), (19, (65, 9, 17)), (27, (24, 17, 8)), (27, (130, 8, 9))])
def test_float64_block_maxima(lbm, orc, q, n, kind):
    """Partial blocks along every axis, several sensor steps in a row (the
    folded words are cleared in between), one step at a time: block maxima
    within the float64 tolerance of the oracle, 1e-11 relative to
    max(M, 1e-3), and equal flags; then a NaN marks its block alone."""
    print(f"\n[case] f64 block maxima q={q} n={n} kind={kind}", flush=True)
    bc = (WALL,) * 6
    desc = lbm.make_desc(q, n, bc, 0.7, storage=lbm.LBM_F64, sensor_kind=kind, wall_u=_lid(0.04))
    G = orc.Grid(q=q, n=n, bc=bc, wall_u=_lid(0.04), tau=0.7, sensor_kind=kind)
    S = G.equilibrium_state(u=lbm_inputs.velocity_perturbation(n, 0.02, seed=3))
    blk = lbm.Blocks(desc, f0=S)
    for k in range(1, 5):
        blk.step_n(1, 1)
        bm, fl, kk, bad = blk.sensor_flags()
        S, hist = G.run(S, k - 1, 1, 1)
        assert kk == k and not bad
        assert (np.abs(bm - hist[-1][1]) / np.maximum(hist[-1][1], 1e-3)).max() <= 1e-11
        assert (fl == hist[-1][2]).all()
    blk.close()

    desc = lbm.make_desc(q, n, (PERIODIC,) * 6, 0.8, storage=lbm.LBM_F64, sensor_kind=kind)
    G = orc.Grid(q=q, n=n, bc=(PERIODIC,) * 6, tau=0.8, sensor_kind=kind)
    f = G.equilibrium_state()
    f[0, n[2] - 1, n[1] - 1, n[0] - 1] = np.nan          # at rest: it stays in its cell for one step
    blk = lbm.Blocks(desc, f0=f)
    blk.step_n(1, 1)
    bm, fl, _, bad = blk.sensor_flags()
    assert bad and fl[-1, -1, -1] == 2 and np.isnan(bm[-1, -1, -1])
    others = np.ones(fl.shape, bool)
    others[-1, -1, -1] = False
    assert (fl[others] == -1).all()
    blk.close()
