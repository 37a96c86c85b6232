"""GPU test of the voxel-centre evaluation where its row intervals and its
launch shape change path: faces nearly parallel to x (their crossing is left
to the exact integers), crossings exactly on voxel centres (ties), one or two
items per wave by the size of the call."""
import numpy as np
import pytest

import oracle
import synth
from conftest import synth_problem
from parity import assert_parity, to_host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2303_04873_amd as morea  # noqa: E402

DIMS = (40, 22, 18)
UNIT = 2.0 ** -10


def vertices(kind, rs, n):
    """n tets [n][4][3] of a kind, snapped coordinates."""
    box = np.array(DIMS) - 1.0
    v = rs.uniform(0, 1, (n, 4, 3)) * box
    if kind == "grid":                        # vertices on voxel centres: ties
        v = np.round(v)
    elif kind == "near grid":                 # one unit off
        v = np.round(v) + rs.integers(-1, 2, v.shape) * UNIT
    elif kind == "slivers along x":           # faces within a few units of parallel to x
        v[:, 1:3] = v[:, :1] + rs.integers(-3, 4, (n, 2, 3)) * UNIT
        v[:, 1, 0] += np.where(v[:, 0, 0] > 20, -18, 18)
        v[:, 2, 2] += np.where(v[:, 0, 2] > 9, -7, 7)
    elif kind == "planes through centres":    # a face in an x = const or y = const voxel plane
        v[:, :3, 0] = np.round(v[:, :1, 0])
        v[::2, 1:, 1] = np.round(v[::2, 1:2, 1])
    return np.round(v / UNIT) * UNIT


@pytest.mark.parametrize("kind", ["grid", "near grid", "slivers along x", "planes through centres", "uniform"])
def test_row_intervals(kind):
    """Counts and flags exact, objectives within the parity bar, on 300
    unrelated tets and their images under small moves."""
    rs = np.random.default_rng(len(kind))
    v = vertices(kind, rs, 900)
    d = np.linalg.det(v[:, 1:] - v[:, :1])
    v = v[np.abs(d) > 1e-4][:300]
    assert len(v) == 300
    pts = v.reshape(-1, 3).astype(np.float32)
    tets = np.arange(len(pts), dtype=np.int32).reshape(-1, 4)
    img = [(rs.uniform(0, 1, DIMS[::-1]) * (rs.uniform(0, 1, DIMS[::-1]) > 0.3)).astype(np.float32) for _ in range(2)]
    el = np.ones(len(tets), np.float32)
    prob = morea.Problem(DIMS, img[0], img[1], tets, pts, el, [], [], radius=2.0, max_population=2)
    op = oracle.Problem(DIMS, img[0], img[1], tets, pts, el, [], [], 2.0)
    moved = pts + rs.integers(-2000, 2001, pts.shape) * np.float32(UNIT)
    cands = np.stack([np.stack([pts.T, moved.T]), np.stack([moved.T, pts.T])]).astype(np.float32)
    out = prob.eval_full(torch.from_numpy(np.ascontiguousarray(cands)).cuda())
    assert_parity(to_host(out), op.evaluate(cands), what=kind)


@pytest.mark.parametrize("config,pop", [(1, 13), (2, 6)])
def test_candidates_do_not_depend_on_items_per_wave(config, pop):
    """`pop` candidates run one item per wave, one more two items: the same
    bits (5,120 items of small tets, 20,480 of large ones lie between)."""
    p = synth_problem(config)
    pts = torch.from_numpy(np.ascontiguousarray(synth.make_population(p)[:pop + 1])).cuda()
    prob = morea.Problem.from_synth(p, max_population=pop + 1)
    limit = 20480 if np.prod(p.dims) >= 256 * p.n_tets else 5120
    assert pop * p.n_tets <= limit < (pop + 1) * p.n_tets
    one = to_host(prob.eval_full(pts[:pop].contiguous()))
    two = to_host(prob.eval_full(pts))
    for k in one:
        np.testing.assert_array_equal(one[k], two[k][:pop])
