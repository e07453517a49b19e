"""Step kernel variants at the sizes where they can go wrong: the float64
block maxima of 3D grids, folded by one atomic maximum per workgroup, two
steps per launch (step_pair) against two launches, and host reads around the
sizes where they change form."""
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


_MOVING = [[0.0, 0.03, 0.01], [0.0, 0.0, 0.0], [0.02, 0.0, 0.01], [0.05, 0.0, -0.02], [0.01, 0.02, 0.0],
           [0.03, -0.01, 0.0]]
_PAIR = [
    # name, n, bc, wall_u, force, smagorinsky, smoothed faces
    ("cavity", (70, 19, 13), (WALL,) * 6, _lid(0.05), 0.0, 0.0, (0,) * 6),
    ("channel", (33, 21, 9), (PERIODIC, PERIODIC, WALL, WALL, PERIODIC, PERIODIC), _lid(0.0), 1e-5, 0.0, (0,) * 6),
    ("box", (20, 17, 18), (PERIODIC,) * 6, _lid(0.0), 0.0, 0.1, (0,) * 6),
    ("walls_x_z", (24, 16, 17), (WALL, WALL, PERIODIC, PERIODIC, WALL, WALL), _MOVING, 0.0, 0.0, (0,) * 6),
    ("all_moving", (41, 36, 30), (WALL,) * 6, _MOVING, 0.0, 0.14, (0, 1, 0, 1, 1, 0)),
    ("narrow", (9, 50, 5), (WALL, WALL, WALL, WALL, PERIODIC, PERIODIC), _MOVING, 1e-5, 0.0, (0,) * 6),
    ("smallest", (4, 4, 4), (PERIODIC,) * 6, _lid(0.0), 0.0, 0.0, (0,) * 6),
    ("tiles", (133, 67, 40), (WALL,) * 6, _lid(0.05), 0.0, 0.0, (0, 0, 0, 1, 0, 0)),
]


@pytest.mark.parametrize("chunk", [0, 6], ids=["eager", "graph"])
@pytest.mark.parametrize("q,storage,streaming", [(19, 0, 1), (19, 1, 1), (19, 1, 2), (19, 2, 1), (19, 2, 2),
                                                 (27, 1, 1), (27, 2, 2)])
@pytest.mark.parametrize("case", _PAIR, ids=[c[0] for c in _PAIR])
def test_pairs_match_single_steps(lbm, monkeypatch, case, q, storage, streaming, chunk):
    """Two steps per launch give the bits of two launches: populations,
    fields, block maxima and flags, over odd and even runs, with the sensor
    at every step and at every third, both sensor kinds, eager and replayed."""
    import torch
    name, n, bc, wall_u, force, smag, smooth = case
    print(f"\n[case] pairs {name} q={q} storage={storage} streaming={streaming} chunk={chunk}", flush=True)
    runs = []
    for pair in ("off", "on"):
        monkeypatch.setenv("LBM_PAIR", pair)
        got = []
        for kind, every in ((0, 1), (1, 3)):
            desc = lbm.make_desc(q, n, bc, 0.65, storage=storage, sensor_kind=kind, wall_u=wall_u,
                                 force=(force, 0.0, 0.0), smagorinsky=smag, wall_profile=smooth, streaming=streaming)
            stream = torch.cuda.Stream()
            blk = lbm.Blocks(desc, stream=stream)
            if chunk:
                blk.use_graphs(chunk)
            blk.set_equilibrium(u=lbm_inputs.velocity_perturbation(n, 0.02, seed=5))
            for k in (7, 2, 13, 6):
                blk.step_n(k, every if k != 13 else 0)
                bm, fl, step, _ = blk.sensor_flags()
                got += [bm, fl, np.array(step), blk.populations(), *blk.macros()]
            blk.close()
        runs.append(got)
    for a, b in zip(*runs):
        assert np.array_equal(a, b), f"{name}: pairs differ"


def test_float64_average_between_pairs(lbm, monkeypatch):
    """A float64 pair folds its second sensor where the averaged maxima are
    returned: runs with averages read in between equal single steps."""
    n = (24, 16, 17)
    runs = []
    for pair in ("off", "on"):
        monkeypatch.setenv("LBM_PAIR", pair)
        desc = lbm.make_desc(19, n, (WALL,) * 6, 0.6, storage=lbm.LBM_F64, wall_u=_lid(0.05))
        blk = lbm.Blocks(desc)
        blk.step_n(4, 1)
        blk.average_begin()
        blk.step_n(5, 1)
        got = [blk.average()[0]]
        blk.average_end()
        for _ in range(3):
            blk.step_n(4, 2)
            got += [blk.sensor_flags()[0], blk.average()[0]]
        blk.close()
        runs.append(got)
    for a, b in zip(*runs):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("n", [(3, 5, 1), (64, 129, 1), (128, 128, 1), (128, 129, 1), (257, 511, 1), (1201, 1103, 1)])
def test_host_reads(lbm, n):
    """Populations and fields come back whole below, at and above the size of
    a small read (16384 cells' fields) and of the ring of the large ones."""
    print(f"\n[case] host reads {n}", flush=True)
    desc = lbm.make_desc(9, n, (PERIODIC,) * 6, 0.8, storage=lbm.LBM_F64)
    f = lbm_inputs.random_populations(9, n, seed=n[0])
    blk = lbm.Blocks(desc, f0=f)
    for _ in range(2):
        assert np.array_equal(blk.populations(), f)
        rho, u = blk.macros()
        c = np.array([(0, 0), (1, 0), (-1, 0), (0, 1), (0, -1), (1, 1), (-1, -1), (1, -1), (-1, 1)], dtype=float)
        assert np.allclose(rho, f.sum(0), rtol=1e-14, atol=0)
        for a in range(2):
            assert np.allclose(u[a] * rho, np.tensordot(c[:, a], f, axes=1), rtol=0, atol=1e-14)
        assert not u[2].any()
    blk.close()


@pytest.mark.parametrize("storage", [0, 1, 2, 3], ids=["f64", "f32", "f32s", "f16s"])
@pytest.mark.parametrize("q,n", [(9, (45, 9, 1)), (19, (8, 8, 8)), (19, (37, 20, 9)), (27, (70, 5, 17))])
def test_state_reads_in_both_slot_orders(lbm, q, n, storage):
    """The in-place scheme's state read before a gather step (the exchanged
    slots, as they lie) and after one (scattered): the populations after k
    steps are the same read with either scheme, and the fields, block means
    and totals are those of the populations.  Bounds: float64 sums of q
    values and, in a block, of up to 512 fields, with one rounding of 2^-53
    per operation."""
    print(f"\n[case] state reads q={q} n={n} storage={storage}", flush=True)
    bc = (PERIODIC,) * 6
    force = (1e-5, 0.0, 0.0)
    f0 = 1.0 + 0.02 * np.random.default_rng(5).standard_normal((q, n[2], n[1], n[0]))
    f0 *= 1.0 / q
    blks = [lbm.Blocks(lbm.make_desc(q, n, bc, 0.8, storage=storage, force=force, streaming=s), f0=f0)
            for s in (lbm.LBM_STREAMING_AUTO if q > 9 and storage == 0 else lbm.LBM_STREAMING_INPLACE,   # (3D float64: ping-pong only)
                      lbm.LBM_STREAMING_PINGPONG)]
    eps = 2.0 ** -53
    for k in range(3):
        f, ref = (b.populations() for b in blks)
        same = storage < 3 or k == 0   # (16 bits: the two kernels round a product and sum differently)
        assert not same or (f == ref).all(), k
        rho, u = blks[0].macros()
        size = np.abs(f).sum(axis=0)
        assert (np.abs(rho - f.sum(axis=0)) <= 2 * q * eps * size).all()
        m = blks[0].block_means()
        bz = 1 if q == 9 else 8
        for kb in range(m.shape[0]):
            for jb in range(m.shape[1]):
                for ib in range(m.shape[2]):
                    at = np.s_[bz * kb:bz * kb + bz, 8 * jb:8 * jb + 8, 8 * ib:8 * ib + 8]
                    want = np.array([(rho[at] - 1.0).mean()] + [u[a][at].mean() for a in range(3)])
                    bound = 2 * 512 * eps * np.array([np.abs(rho[at] - 1.0).mean()] +
                                                     [np.abs(u[a][at]).mean() for a in range(3)]) + 4 * eps
                    assert (np.abs(m[kb, jb, ib] - want) <= bound).all(), (k, kb, jb, ib)
        total = blks[0].conservation()
        cells = n[0] * n[1] * n[2]
        assert abs(total[0] - f.sum()) <= 2 * q * cells * eps * size.sum()
        assert not same or (np.asarray(total) == np.asarray(blks[1].conservation())).all()
        for b in blks:
            b.step_n(1, 0)
    for b in blks:
        b.close()
