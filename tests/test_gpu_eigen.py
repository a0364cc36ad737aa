"""Fixed-corotated stress and plastic projection at strains where an eigen-decomposition by
rotations can go wrong: none, rotations only (equal eigenvalues), one or two stretched axes,
nearly equal eigenvalues, tiny off-diagonals, and large general strains, against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2609_27342_amd import workloads as W

from harness import state_errs

pytestmark = pytest.mark.gpu

STEPS = 2
TOL = 1e-5 * STEPS  # FP32 sums of one substep, added up


@pytest.fixture(scope="module")
def tl():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_27342_amd import tlmpm
    tlmpm.lib()
    return tlmpm


def _rotations(rng, n):
    q = rng.normal(size=(n, 4))
    q /= np.linalg.norm(q, axis=1)[:, None]
    w, x, y, z = q.T
    return np.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                     2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                     2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], 1).reshape(n, 3, 3)


def _F(kind, n, rng):
    I = np.broadcast_to(np.eye(3), (n, 3, 3))
    if kind == "none":
        return I
    if kind == "rotated":
        return _rotations(rng, n)
    if kind == "general":
        return I + 0.1 * rng.normal(size=(n, 3, 3))
    s = 1.0 + 0.2 * rng.random((n, 3))
    if kind == "one axis":
        s[:, 1:] = 1.0
    if kind == "two axes":
        s[:, 1] = s[:, 0]
    if kind == "nearly equal":
        s = s[:, :1] + 1e-6 * rng.random((n, 3))
    F = np.einsum("ni,ij->nij", s, np.eye(3))
    if kind == "tiny":
        F = F + 10.0 ** rng.uniform(-30, -6, (n, 1, 1)) * rng.normal(size=(n, 3, 3))
    if kind in ("two axes", "nearly equal"):
        R = _rotations(rng, n)
        F = np.matmul(np.matmul(R, F), R.transpose(0, 2, 1))
    return F


@pytest.mark.parametrize("yield_stress", [0.0, 3e4])
@pytest.mark.parametrize("kind", ["none", "rotated", "one axis", "two axes", "nearly equal", "tiny", "general"])
def test_strains(tl, kind, yield_stress):
    s = W.box_scene(n_cells=(4, 5, 3), seed=61, E=1e6, floor_on=0, material=1, yield_stress=yield_stress,
                    gravity=[0.0, 0.0, -9.81])
    n = s["X"].shape[0]
    rng = np.random.default_rng([62, len(kind)])
    # the same strain in all particles of a call would cancel: each has its own
    F = _F(kind, n, rng).astype(np.float32)
    v = (rng.normal(size=(n, 3)) * 0.1).astype(np.float32)
    print(f"[case] strains {kind} yield={yield_stress} n={n}", flush=True)
    g = tl.Scene(s)
    g.write(v=v, F=F)
    o = oracle.OracleScene(s)
    o.set(v=v, F=F.reshape(n, 9).astype(np.float64))
    for _ in range(STEPS):
        g.step([])
        o.step([])
    assert g.status() == 0
    a, b = g.read(("u", "v", "H")), o.get()
    eu, ev, eH = state_errs(a, b, s["X"], s["params"])
    print(f"[strains] {kind} u {eu:.1e} v {ev:.1e} H {eH:.1e}", flush=True)
    assert eu < TOL and ev < TOL and eH < TOL, (eu, ev, eH)
