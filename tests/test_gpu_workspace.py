"""What the workspace has room for changes where things lie, not the results: scenes whose
particles' cell positions do not fit (P2G forms them from X) against the same scene with
more slots per node, in single calls and batches; split bricks in a workspace that holds
fewer second boxes than bricks, and in one that holds them all."""
import numpy as np
import pytest

import oracle
from paper_2609_27342_amd import workloads as W

from harness import state_errs

pytestmark = pytest.mark.gpu

STEPS = 3
TOL = 1e-5 * STEPS  # FP32 sums of one substep, added up
FIELDS = ("u", "v", "H", "digits")


@pytest.fixture(scope="module")
def tl():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_27342_amd import tlmpm
    tlmpm.lib()
    return tlmpm


def _scene(n_cells, dense, scap, general, full=True):
    """dense: 64 particles per cell instead of 8 (the same particles on a coarser grid)."""
    extra = dict(material=1, viscosity=5.0, yield_stress=300.0) if general else {}
    s = W.box_scene(n_cells=tuple(n * (2 if dense else 1) for n in n_cells), seed=61, floor_on=0,
                    gravity=[0.0, 0.0, -9.81], slot_capacity=scap, **extra)
    if full:  # whole bricks from the origin on
        s["params"].update(dx=0.02 if dense else 0.01, origin=[0.0] * 3, cells=list(n_cells))
    return s


def _start(s, g, codes):
    n = s["X"].shape[0]
    rng = np.random.default_rng(62)
    F = (np.eye(3)[None] + 0.03 * rng.normal(size=(n, 3, 3))).astype(np.float32)
    v = (rng.normal(size=(n, 3)) * 0.1).astype(np.float32)
    dig = np.zeros((n, 4), np.uint8)
    if codes > 1:
        dig[:, 0] = np.where(s["X"][:, 0] > np.median(s["X"][:, 0]), 1, 2)
    g.write(v=v, F=F, digits=dig)
    return v, F, dig


# a full brick of 8 per cell with one slot: 6144 bytes of positions against 6000; of 64 per
# cell with two slots 49152 against 12000 (with 16 slots both fit: 96000)
@pytest.mark.parametrize("general", [False, True])
@pytest.mark.parametrize("n_cells,dense,scap,codes", [((8, 8, 8), False, 1, 1), ((4, 4, 4), True, 1, 1),
                                                      ((4, 4, 4), True, 2, 2), ((8, 4, 5), True, 2, 2)])
def test_positions_that_do_not_fit(tl, n_cells, dense, scap, codes, general):
    out = []
    for slots in (scap, 16):
        s = _scene(n_cells, dense, slots, general)
        print(f"[case] positions {n_cells} dense={dense} slots={slots} general={general} n={s['X'].shape[0]}",
              flush=True)
        g = tl.Scene(s)
        v, F, dig = _start(s, g, codes)
        for _ in range(STEPS):
            g.step([])
        assert g.status() == 0
        out.append(g.read(FIELDS))
    for f in FIELDS:
        assert np.array_equal(out[0][f], out[1][f]), f
    if not general:
        o = oracle.OracleScene(s)
        o.set(v=v, F=F.reshape(-1, 9), digits=dig)
        for _ in range(STEPS):
            o.step([])
        e = state_errs(out[0], o.get(), s["X"], s["params"])
        assert max(e) < TOL, e


def test_positions_that_do_not_fit_in_a_batch(tl):
    scenes = [_scene((4, 4, 4), True, scap, False) for scap in (2, 16, 2)]
    print("[case] positions in a batch", flush=True)
    gs = [tl.Scene(s) for s in scenes]
    for s, g in zip(scenes, gs):
        _start(s, g, 2)
    with tl.Batch(gs) as b:
        b.step([[]] * 3, STEPS)
    out = [g.read(FIELDS) for g in gs]
    for g in gs:
        assert g.status() == 0
    for f in FIELDS:
        assert np.array_equal(out[0][f], out[1][f]) and np.array_equal(out[0][f], out[2][f]), f


@pytest.mark.parametrize("n_cells", [(8, 7, 6), (17, 8, 8)])
def test_split_bricks_in_any_order(tl, n_cells):
    """Every mixed brick split (their second boxes lie in the order in which they became
    mixed) against none split and the oracle."""
    s = _scene(n_cells, False, 8, False, full=False)
    n = s["X"].shape[0]
    rng = np.random.default_rng(63)
    dig = np.zeros((n, 4), np.uint8)
    band = np.abs(s["X"][:, 0] - np.median(s["X"][:, 0])) < 0.011  # some cells of random codes
    dig[:, 0] = np.where(band, rng.integers(0, 3, n), np.where(s["X"][:, 0] > np.median(s["X"][:, 0]), 1, 2))
    v = (rng.normal(size=(n, 3)) * 0.1).astype(np.float32)
    print(f"[case] split bricks {n_cells} n={n}", flush=True)
    out = []
    try:
        for div in (1, 2, None):
            if div is None:
                tl.set_tuning(split_cap=0)
            else:
                tl.set_tuning(split_lo=0, split_hi=1 << 30, split_div=div, split_cap=1 << 30)
            g = tl.Scene(s)
            g.write(v=v, digits=dig)
            for _ in range(STEPS):
                g.step([])
            assert g.status() == 0
            out.append(g.read(FIELDS))
    finally:
        tl.set_tuning(None)
    o = oracle.OracleScene(s)
    o.set(v=v, digits=dig)
    for _ in range(STEPS):
        o.step([])
    b = o.get()
    for a in out:
        e = state_errs(a, b, s["X"], s["params"])
        assert max(e) < TOL, e
