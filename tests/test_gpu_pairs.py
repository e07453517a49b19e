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


def _supported(q, storage, force, smag):
    return not (force and smag) if storage else q == 19 and not force


@pytest.mark.parametrize("q,storage,streaming", [(19, 0, 1), (19, 1, 1), (19, 1, 2), (19, 2, 1), (19, 2, 2),
                                                 (27, 1, 1), (27, 2, 2), (27, 0, 1), (19, 3, 2)])
@pytest.mark.parametrize("case", _PAIR, ids=[c[0] for c in _PAIR])
def test_pairs_are_taken_where_they_exist(lbm, monkeypatch, case, q, storage, streaming):
    """The comparison of pairs with single steps compares the two: with pairs
    switched on every case has 2 steps per launch, those without a pair
    kernel (float64 with a force or on D3Q27, a force with Smagorinsky, 16
    bits) 1; switched off all have 1; none while the sensor is averaged."""
    name, n, bc, wall_u, force, smag, smooth = case
    print(f"\n[case] taken {name} q={q} storage={storage} streaming={streaming}", flush=True)
    exists = storage <= 2 and _supported(q, storage, force, smag)
    for pair, want in (("off", 1), ("on", 2 if exists else 1)):
        monkeypatch.setenv("LBM_PAIR", pair)
        blk = lbm.Blocks(lbm.make_desc(q, n, bc, 0.65, storage=storage, wall_u=wall_u, force=(force, 0.0, 0.0),
                                       smagorinsky=smag, wall_profile=smooth, streaming=streaming))
        assert [_per_launch(lbm, blk, every) for every in (0, 1, 2, 3)] == [want] * 4
        blk.average_begin()
        assert _per_launch(lbm, blk, 1) == 1
        blk.average_end()
        assert _per_launch(lbm, blk, 1) == want
        blk.close()


@pytest.mark.parametrize("value", [float("nan"), float("inf"), -float("inf")], ids=["nan", "inf", "-inf"])
@pytest.mark.parametrize("kind", [0, 1], ids=["l2", "kkn"])
@pytest.mark.parametrize("q,storage,streaming", [(19, 0, 1), (19, 1, 1), (19, 2, 2), (27, 1, 2)])
def test_non_finite_values_through_pairs(lbm, monkeypatch, q, storage, streaming, kind, value):
    """A value that is not finite, in one cell at the far corner, gives the
    same block maxima, flags and cells in pairs as step by step."""
    print(f"\n[case] non-finite q={q} storage={storage} kind={kind} {value}", flush=True)
    n = (41, 36, 30)
    w = [lbm_inputs.velocity_perturbation(n, 0.02, seed=5)]
    runs = []
    for pair in ("off", "on"):
        monkeypatch.setenv("LBM_PAIR", pair)
        blk = lbm.Blocks(lbm.make_desc(q, n, (PERIODIC,) * 4 + (WALL,) * 2, 0.65, storage=storage, sensor_kind=kind,
                                       streaming=streaming))
        assert _per_launch(lbm, blk, 1) == (2 if pair == "on" else 1)
        blk.set_equilibrium(u=w[0])
        f = blk.populations()
        f[3, n[2] - 1, n[1] - 1, n[0] - 1] = value
        blk.set_populations(f)
        got = []
        for every in (1, 2):
            blk.step_n(4, every)
            bm, fl, k, bad = blk.sensor_flags()
            got += [bm, fl.astype(float), blk.populations()]
            assert bad and (fl == 2).any() and k == blk.step
        blk.close()
        runs.append(got)
    for a, b in zip(*runs):
        assert np.array_equal(a, b, equal_nan=True)


@pytest.mark.parametrize("q,n,storage", [(19, (256, 256, 256), 0), (27, (330, 310, 300), 1)])
def test_pairs_in_buffers_beyond_2_gib(lbm, monkeypatch, q, n, storage):
    """Populations of 2.55 and 3.3 GB, whose byte offsets need all 32 bits: the
    bits of single steps, compared on the GPU."""
    import torch
    print(f"\n[case] large buffers q={q} {n} storage={storage}", flush=True)
    lid = _lid(0.05)
    lid[5] = [0.0, 0.03, 0.01]
    runs = []
    for pair in ("off", "on"):
        monkeypatch.setenv("LBM_PAIR", pair)
        blk = lbm.Blocks(lbm.make_desc(q, n, (WALL,) * 6, 0.6, storage=storage, wall_u=lid))
        assert 2 ** 31 < blk._bufs[0].numel() < 2 ** 32
        assert _per_launch(lbm, blk, 1) == (2 if pair == "on" else 1)
        rng = np.random.default_rng(3)
        rho = 1.0 + 0.01 * rng.standard_normal(blk.cells)
        blk.set_equilibrium(rho=rho)
        blk.step_n(8, 1)
        torch.cuda.synchronize()
        plane = n[0] * n[1] * n[2] * (8 if storage == 0 else 4)
        pitch = blk._bufs[0].numel() // q
        state = blk._bufs[0].view(q, pitch)[:, :plane]
        runs.append((state, blk._bufs, *blk.sensor_flags()[:2], np.array(blk.conservation())))
        blk.close()
    assert all(torch.equal(a, b) for a, b in zip(runs[0][0], runs[1][0]))
    for a, b in zip(runs[0][2:], runs[1][2:]):
        assert np.array_equal(a, b)
