"""The quadratic stencil's sums per side key against the oracle: bricks of one to six keys
(a pass per key; the node kernels look up the first four at once), more keys in a brick than
slots at a node, and particles on the half planes of cells, whose outer nodes have zero
weight."""
import numpy as np
import pytest

import oracle
from paper_2609_27342_amd import workloads as W

from harness import state_errs

pytestmark = pytest.mark.gpu

STEPS = 2
TOL = 1e-5 * STEPS  # FP32 sums of one substep, added up

CODES = np.array([[0, 0], [1, 0], [2, 0], [0, 1], [0, 2], [1, 2]], np.uint8)


@pytest.fixture(scope="module")
def tl():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_27342_amd import tlmpm
    tlmpm.lib()
    return tlmpm


def _check(tl, s, code, seed):
    n = s["X"].shape[0]
    rng = np.random.default_rng(seed)
    F = (np.eye(3)[None] + 0.03 * rng.normal(size=(n, 3, 3))).astype(np.float32)
    v = (rng.normal(size=(n, 3)) * 0.1).astype(np.float32)
    dig = np.zeros((n, 4), np.uint8)
    dig[:, :2] = CODES[code]
    g = tl.Scene(s)
    g.write(v=v, F=F, digits=dig)
    o = oracle.OracleScene(s)
    o.set(v=v, F=F.reshape(n, 9), digits=dig)
    for _ in range(STEPS):
        g.step([])
        o.step([])
    assert g.status() == 0
    a, b = g.read(("u", "v", "H")), o.get()
    eu, ev, eH = state_errs(a, b, s["X"], s["params"])
    assert eu < TOL and ev < TOL and eH < TOL, (eu, ev, eH)


@pytest.mark.parametrize("material", [0, 1])
@pytest.mark.parametrize("n_codes", [1, 2, 4, 6])
def test_keys_per_brick(tl, n_codes, material):
    extra = dict(material=1, viscosity=5.0, yield_stress=300.0) if material else {}
    s = W.box_scene(n_cells=(9, 4, 6), seed=51, floor_on=0, stencil=1, slot_capacity=8, gravity=[0.0, 0.0, -9.81],
                    **extra)
    code = np.random.default_rng([52, n_codes]).integers(0, n_codes, s["X"].shape[0])
    print(f"[case] quadratic keys per brick {n_codes} material={material} n={code.size}", flush=True)
    _check(tl, s, code, 53)


def test_more_keys_than_slots(tl):
    """Three layers of one brick, two cells apart: three keys, two at any node."""
    s = W.box_scene(n_cells=(8, 7, 5), seed=54, floor_on=0, stencil=1, slot_capacity=2)
    q = (s["X"][:, 0].astype(np.float64) - s["params"]["origin"][0]) / s["params"]["dx"]
    layer = np.select([(q > 4) & (q < 4.5), (q > 6) & (q < 6.5), (q > 7.5) & (q < 8)], [0, 1, 3], -1)
    keep = layer >= 0
    for f in ("X", "vol0", "mass", "E"):
        s[f] = np.ascontiguousarray(s[f][keep])
    assert set(layer[keep]) == {0, 1, 3}
    print(f"[case] quadratic more keys than slots n={keep.sum()}", flush=True)
    _check(tl, s, layer[keep], 55)


@pytest.mark.parametrize("n_codes", [1, 3])
@pytest.mark.parametrize("planes", [1, 3])
def test_particles_on_half_planes(tl, planes, n_codes):
    dx = 2.0 ** -7
    s = W.box_scene(n_cells=(6, 5, 4), dx=dx, seed=56, floor_on=0, stencil=1, slot_capacity=8)
    X = s["X"].astype(np.float64)
    rng = np.random.default_rng([57, planes])
    some = rng.random(X.shape[0]) < 0.3
    for a in range(planes):
        X[some, a] = (np.floor(X[some, a] / dx) + 0.5) * dx
    s["X"] = X.astype(np.float32)
    print(f"[case] quadratic half planes {planes} codes={n_codes} n={X.shape[0]}", flush=True)
    _check(tl, s, rng.integers(0, n_codes, X.shape[0]), 58)


@pytest.mark.parametrize("scap", [1, 2])
def test_sums_without_a_slot_are_reported(tl, scap):
    """Bricks of one key each that meet at nodes with room for one key less: besides the full
    slot list, the sums left without a slot are reported."""
    s = W.box_scene(n_cells=(12, 4, 4), seed=59, floor_on=0, stencil=1, slot_capacity=scap)
    brick = np.floor((s["X"][:, 0].astype(np.float64) - s["params"]["origin"][0]) / s["params"]["dx"]).astype(int) // 4
    code = brick if scap == 1 else brick + (brick == 1) * (s["X"][:, 1] > 0.02)
    n = code.size
    dig = np.zeros((n, 4), np.uint8)
    dig[:, :2] = CODES[code]
    print(f"[case] quadratic sums without a slot scap={scap} n={n}", flush=True)
    g = tl.Scene(s)
    g.write(digits=dig)
    g.step([])
    status, text = g.status_detail()
    assert status == tl.E_SLOT_OVERFLOW
    bits = int(text.rsplit(" ", 1)[1])
    assert bits == 2 + 8  # TL_ST_SLOT and TL_ST_LOOKUP
