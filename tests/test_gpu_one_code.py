"""P2G and G2P of bricks whose neighbourhood holds one side code (no slot tables) and of
bricks with several, against the oracle at the sizes where the two meet: bodies of one
cell, of exactly one brick, just beyond a brick's edge; 8 and 64 particles per cell
(one round and several); no digits, one digit everywhere, two codes meeting at a brick
face, inside a brick and in single cells."""
import numpy as np
import pytest

import oracle
from paper_2609_27342_amd import workloads as W

from harness import state_errs

pytestmark = pytest.mark.gpu

STEPS = 2
# one substep of the transfers agrees to 1e-5 (FP32 sums of up to 64 terms); the errors
# of the substeps add up
TOL = 1e-5 * STEPS


@pytest.fixture(scope="module")
def tl():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_27342_amd import tlmpm
    tlmpm.lib()
    return tlmpm


def _scene(n_cells, dense, seed):
    s = W.box_scene(n_cells=tuple(n * (2 if dense else 1) for n in n_cells), seed=seed, floor_on=0,
                    gravity=[0.0, 0.0, -9.81], slot_capacity=8)
    if dense:  # the same particles on a grid twice as coarse: 64 per cell
        s["params"].update(dx=0.02, origin=[-0.02] * 3, cells=[n + 2 for n in n_cells])
    return s


def _digits(kind, X, dx, rng):
    d = np.zeros((X.shape[0], 4), np.uint8)
    if kind == "one":
        d[:, 1] = 2
    elif kind == "face":  # two compatible codes meet at the face between two bricks
        d[X[:, 0] > 3 * dx, 0] = 1
    elif kind == "inside":  # two conflicting codes meet inside a brick
        d[:, 0] = np.where(X[:, 0] > 1.5 * dx, 1, 2)
    elif kind == "cells":  # several codes in the cells of one corner
        corner = np.all(X < 2 * dx, axis=1)
        d[corner, 0] = rng.integers(0, 3, size=corner.sum())
    return d


@pytest.mark.parametrize("kind", ["none", "one", "face", "inside", "cells"])
@pytest.mark.parametrize("n_cells,dense", [((1, 1, 1), False), ((2, 3, 2), True), ((3, 3, 3), False),
                                           ((4, 5, 9), False), ((13, 4, 3), False), ((5, 4, 4), True)])
def test_one_code_and_several(tl, n_cells, dense, kind):
    rng = np.random.default_rng([31, *n_cells])
    s = _scene(n_cells, dense, 31)
    n, dx = s["X"].shape[0], s["params"]["dx"]
    dig = _digits(kind, s["X"].astype(np.float64), dx, rng)
    F = (np.eye(3)[None] + 0.03 * rng.normal(size=(n, 3, 3))).astype(np.float32)
    v = (rng.normal(size=(n, 3)) * 0.1).astype(np.float32)
    print(f"[case] one code n_cells={n_cells} dense={dense} {kind} n={n}", flush=True)
    g = tl.Scene(s)
    g.write(v=v, F=F, digits=dig)
    o = oracle.OracleScene(s)
    o.set(v=v, F=F.reshape(n, 9), digits=dig)
    for _ in range(STEPS):
        g.step([])
        o.step([])
    if dense and kind == "cells":
        # 64 particles of three codes need more than the 8 same-code groups a cell may have
        assert g.status() == tl.E_SLOT_OVERFLOW
        return
    assert g.status() == 0
    a, b = g.read(("u", "v", "F", "H", "digits")), o.get()
    assert np.array_equal(a["digits"], dig)
    eu, ev, eH = state_errs(a, b, s["X"], s["params"])
    assert eu < TOL and ev < TOL and eH < TOL, (eu, ev, eH)


@pytest.mark.parametrize("kind", ["none", "inside"])
@pytest.mark.parametrize("planes", [1, 2, 3])
def test_particles_on_grid_planes(tl, planes, kind):
    """Particles exactly on grid planes (zero weights along 1 to 3 axes: those corners
    take no part in any sum or gradient), mixed with ordinary ones; dx is a power of two,
    so that the positions are exact."""
    dx = 2.0 ** -7
    s = W.box_scene(n_cells=(6, 5, 4), dx=dx, seed=33, floor_on=0, slot_capacity=8)
    X = s["X"].astype(np.float64)
    n = X.shape[0]
    rng = np.random.default_rng([34, planes])
    some = rng.random(n) < 0.3
    for a in range(planes):  # to the lower plane of the particle's cell
        X[some, a] = np.floor(X[some, a] / dx) * dx
    s["X"] = X.astype(np.float32)
    dig = _digits(kind, X, dx, rng)
    F = (np.eye(3)[None] + 0.03 * rng.normal(size=(n, 3, 3))).astype(np.float32)
    v = (rng.normal(size=(n, 3)) * 0.1).astype(np.float32)
    print(f"[case] on grid planes {planes} {kind} n={n}", flush=True)
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


@pytest.mark.parametrize("n_codes", [1, 2, 4, 5, 7])
def test_slot_tables(tl, n_codes):
    """Slots per node against a count of the distinct codes of its 8 cells: up to the four
    that are kept in registers, and beyond; in both tables, unchanged and rewritten."""
    s = _scene((6, 5, 9), False, 35)
    rng = np.random.default_rng([36, n_codes])
    X, p = s["X"].astype(np.float64), s["params"]
    n = X.shape[0]
    cell = np.floor((X - np.asarray(p["origin"], np.float64)) / p["dx"]).astype(int)
    codes = np.array([[a, b, 0, 0] for a in range(3) for b in range(3)], np.uint8)[:n_codes]

    def expected(dig):
        seen = {}
        for c, k in zip(cell, dig[:, 0].astype(int) * 3 + dig[:, 1]):
            for d in np.ndindex(2, 2, 2):
                seen.setdefault(tuple(c + d), set()).add(k)
        return np.bincount([len(v) for v in seen.values()], minlength=17)[1:17]

    print(f"[case] slot tables codes={n_codes} n={n}", flush=True)
    g = tl.Scene(s)
    for every in (1.0, 0.3, 0.0):  # all particles of mixed codes, some, none
        dig = codes[np.where(rng.random(n) < every, rng.integers(0, n_codes, n), 0)]
        g.write(digits=dig)
        for _ in range(3):
            assert list(g.slot_histogram()[1:]) == list(expected(dig))
            g.step([])
        assert g.status() == 0
