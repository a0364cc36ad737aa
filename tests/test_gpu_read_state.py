"""State copies to the host (arranged in the caller's order on the device): what was written
comes back bit for bit, in one piece and in several (a few bricks with very many
particles each, whose staging area holds only a part), and with 15 digits."""
import numpy as np
import pytest

from paper_2609_27342_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tl():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_27342_amd import tlmpm
    tlmpm.lib()
    return tlmpm


def _scene(coarse, cuts, scap, seed):
    s = W.box_scene(n_cells=(18, 11, 7), seed=seed, floor_on=0, max_cuts=cuts, slot_capacity=scap)
    if coarse > 1:  # the same particles on a grid `coarse` times coarser
        dx = 0.01 * coarse
        s["params"].update(dx=dx, origin=[-dx] * 3, cells=[-(-n // coarse) + 2 for n in (18, 11, 7)])
    return s


@pytest.mark.parametrize("coarse,cuts,scap", [(1, 4, 8), (1, 15, 16), (6, 4, 1), (18, 1, 1)])
def test_written_state_reads_back(tl, coarse, cuts, scap):
    s = _scene(coarse, cuts, scap, 41)
    n = s["X"].shape[0]
    rng = np.random.default_rng(42)
    u = (rng.normal(size=(n, 3)) * 1e-3).astype(np.float32)
    v = rng.normal(size=(n, 3)).astype(np.float32)
    H = (0.01 * rng.normal(size=(n, 3, 3))).astype(np.float32)
    D = rng.random(n).astype(np.float32)
    dig = np.zeros((n, cuts), np.uint8)
    dig[:, cuts - 1] = np.where(s["X"][:, 0] < 0.06, 1, 2) if scap > 1 else 2
    print(f"[case] read back coarse={coarse} cuts={cuts} n={n}", flush=True)
    g = tl.Scene(s)
    g.write(u=u, v=v, H=H, D=D, digits=dig)
    a = g.read(("X", "u", "v", "F", "code", "D", "digits", "H"))
    assert np.array_equal(a["X"], s["X"]) and np.array_equal(a["u"], u) and np.array_equal(a["v"], v)
    assert np.array_equal(a["H"], H) and np.array_equal(a["D"], D) and np.array_equal(a["digits"], dig)
    assert np.array_equal(a["F"], H + np.eye(3, dtype=np.float32))
    assert np.array_equal(a["code"], dig.astype(np.uint64) @ (np.uint64(3) ** np.arange(cuts, dtype=np.uint64)))
    b = g.read(("v", "digits"))  # fields by themselves
    assert np.array_equal(b["v"], v) and np.array_equal(b["digits"], dig)
