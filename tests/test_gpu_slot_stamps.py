"""The slot tables' two buffers over substeps that label, pause, label elsewhere, and after
digits are written or labels assigned between substeps: a scene stepped without reads, whose
tables change buffers and copy what changed since a buffer was last built, against its twin
that is read after every substep (a read applies the pending F update, and tables are then
rebuilt in place), and against a count of the digits around every node."""
import numpy as np
import pytest

from paper_2609_27342_amd import workloads as W

pytestmark = pytest.mark.gpu

FIELDS = ("u", "v", "H", "digits")


@pytest.fixture(scope="module")
def tl():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_27342_amd import tlmpm
    tlmpm.lib()
    return tlmpm


def _scene(contact, seed=71, n_cells=(13, 9, 10)):
    s = W.box_scene(n_cells=n_cells, seed=seed, floor_on=0, slot_capacity=16, material_contact=contact)
    s["v0"] = (np.random.default_rng(seed).normal(size=s["X"].shape) * 0.05).astype(np.float32)
    return s


def _blade(cut, n, at, z, new=False):
    """A descending blade: behind its edge at height z, 2 cm to either side of n x = at."""
    p = np.asarray(n, np.float64) * at
    return W.blade(cut, (p[0], p[1], z), n, (0, 0, -1), (0, 0, -20.0), 1.0, 0.02, 0.3, 0.005, new_cut=new)


def _label(cut, n, at, z, new=False):
    return [W.tool(_blade(cut, n, at, z, new), contact=False, cutting=False)]


class Expected:
    """Nodes by number of distinct codes in their 8 cells."""

    def __init__(self, s):
        p = s["params"]
        c = np.floor((s["X"].astype(np.float64) - np.asarray(p["origin"])) / p["dx"]).astype(np.int64)
        dims = np.asarray(p["cells"]) + 1
        self.nodes = np.concatenate([np.ravel_multi_index((c + d).T, dims) for d in np.ndindex(2, 2, 2)])

    def __call__(self, digits):
        code = digits.astype(np.int64) @ 3 ** np.arange(digits.shape[1])
        pairs = np.unique(self.nodes * 3 ** digits.shape[1] + np.tile(code, 8))
        return list(np.bincount(np.unique(pairs // 3 ** digits.shape[1], return_counts=True)[1], minlength=17)[1:17])


X, Y = (1, 0, 0), (0, 1, 0)


def _schedule():
    """(what, argument) of each substep; every blade takes in a new layer of particles (5 mm)"""
    at = []
    for j in range(5):
        at.append(("step", _label(0, X, 0.062, 0.096 - 0.005 * j, j == 0)))
    at += [("step", [])] * 3
    for j in range(4):
        at.append(("step", _label(1, Y, 0.045, 0.096 - 0.005 * j, j == 0)))
    at.append(("assign", _blade(0, X, 0.062, 0.066)))
    at.append(("step", []))
    at.append(("assign", _blade(1, Y, 0.045, 0.071)))
    at.append(("assign", _blade(0, X, 0.062, 0.056)))
    at.append(("step", _label(1, Y, 0.045, 0.061)))
    at.append(("step", []))
    at.append(("write", None))
    for j in range(4):
        at.append(("step", _label(2, X, 0.025, 0.096 - 0.005 * j, j == 0)))
    at += [("step", [])] * 2
    for j in range(3):
        at.append(("step", _label(0, X, 0.062, 0.051 - 0.005 * j)))
    return at


def _do(g, what, arg, dig):
    if what == "step":
        g.step(arg)
    elif what == "assign":
        g.assign_labels([arg])
    else:
        g.write(digits=dig)


@pytest.mark.parametrize("one_stream", [0, 2048])
@pytest.mark.parametrize("contact", [0, 1])
def test_buffers_follow_the_digits(tl, contact, one_stream):
    s = _scene(contact)
    n, K = s["X"].shape[0], s["params"]["max_cuts"]
    expected = Expected(s)
    dig = np.zeros((n, K), np.uint8)
    dig[:, 3] = np.where(s["X"][:, 2] > 0.05, 1, 2)
    print(f"[case] slot buffers contact={contact} one_stream={one_stream} n={n}", flush=True)
    try:
        tl.set_tuning(one_stream_bricks=one_stream)
        a, b = tl.Scene(s), tl.Scene(s)
    finally:
        tl.set_tuning(None)
    seen, changes = None, 0
    for j, (what, arg) in enumerate(_schedule()):
        _do(a, what, arg, dig)
        _do(b, what, arg, dig)
        d = b.read(("digits",))["digits"]
        changes += seen is not None and not np.array_equal(seen, d)
        seen = d
        want = expected(d)
        assert a.slot_histogram()[1:] == want, (j, what)
        assert b.slot_histogram()[1:] == want, (j, what)
    assert changes >= 18 and sum(want[2:]) > 0  # it kept labelling; some nodes hold three codes or more
    assert a.status() == 0 and b.status() == 0
    sa, sb = a.read(FIELDS), b.read(FIELDS)
    for f in FIELDS:
        assert np.array_equal(sa[f], sb[f]), f


@pytest.mark.parametrize("first", [0, 1])
def test_batch_of_scenes_with_different_buffers(tl, first):
    """Members with a pending update in either buffer, and with none: the common buffer is
    built from each member's own, then steps of the batch label and pause."""
    before = [3, 4, 4, 0, 1]  # substeps that label (the buffer changes in each)
    pause = [0, 1, 0, 0, 2]
    read = [False, False, True, False, True]  # applies the pending update
    scenes = [_scene(1, 72 + i, (9 + i, 6, 10)) for i in range(5)]
    print(f"[case] slot buffers of a batch, first {first}", flush=True)

    def prepare(i):
        g = tl.Scene(scenes[i])
        for j in range(before[i]):
            g.step(_label(0, X, 0.042, 0.096 - 0.005 * j, j == 0))
        for _ in range(pause[i]):
            g.step([])
        if read[i]:
            g.read(("u",))
        return g

    after = [_label(1, Y, 0.035, 0.096 - 0.005 * j, j == 0) for j in range(3)] + [[]] * 2 + \
            [_label(0, X, 0.042, 0.066 - 0.005 * j) for j in range(3)]
    gs = [prepare(i) for i in range(5)]
    with tl.Batch(gs[first:] + gs[:first]) as b:  # (the first one's buffer becomes the common one)
        for tools in after:
            b.step([tools] * 5, 1)
    for i, g in enumerate(gs):
        h = g.slot_histogram()[1:]
        alone = prepare(i)
        for tools in after:
            alone.step(tools)
            alone.read(("u",))
        assert g.status() == 0 and alone.status() == 0
        x, y = g.read(FIELDS), alone.read(FIELDS)
        for f in FIELDS:
            assert np.array_equal(x[f], y[f]), (i, f)
        assert h == Expected(scenes[i])(x["digits"]) == alone.slot_histogram()[1:], i
        assert sum(h[1:]) > 0
