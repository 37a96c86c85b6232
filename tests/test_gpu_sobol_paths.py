"""GPU test of the Sobol-sampled estimator's sample paths against the oracle:
tets inside the image's border cells, tets that leave them, and tets so thin
that points fall exactly on grid planes, where a corner with weight 0 must not
count as foreground."""
import numpy as np
import pytest

import oracle
import synth
from parity import assert_parity, to_host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2303_04873_amd as morea  # noqa: E402

DIMS = (20, 18, 16)
TETS = np.array([[0, 1, 2, 3]], np.int32)


def images(seed):
    rs = np.random.default_rng(seed)
    shape = DIMS[::-1]
    return [(rs.uniform(0, 1, shape) * (rs.uniform(0, 1, shape) > 0.5)).astype(np.float32) for _ in range(2)]


def thin(axis, plane):
    """Three vertices on a grid plane, the fourth 2^-10 above it."""
    p = np.array([[3.25, 2.5, 4.0], [15.5, 3.75, 5.25], [5.0, 14.25, 3.5], [6.5, 7.25, 11.0]])
    p[:3, axis] = plane
    p[3, axis] = plane + 2.0 ** -10
    return p


WIDE = np.array([[2.0, 3.0, 2.5], [16.5, 4.0, 3.0], [5.0, 13.5, 4.0], [7.0, 8.0, 12.0]])
CASES = {
    "inside": (WIDE, WIDE + 0.3, 3.0),
    "border cells": (WIDE * 0 + [[-0.9, -0.5, -0.5], [19.9, 0, 0], [0, 17.9, 0], [0, 0, 15.9]], WIDE, 1.0),
    "leaves the border": (WIDE - [[4.0, 0, 0]], WIDE + [[0, 6.0, 0]], 1.0),
    "thin x": (thin(0, 5.0), WIDE, 1e8),
    "thin y": (thin(1, 6.0), thin(0, 9.0), 1e8),
    "thin z": (WIDE, thin(2, 7.0), 1e8),
    "outer planes": (thin(2, 15.0), thin(1, 17.0), 1e8),
}


@pytest.mark.parametrize("storage", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("case", sorted(CASES))
def test_sample_paths(case, storage):
    """Counts and flags equal, objectives within the parity bound (the oracle
    interpolates the same points in FP64); two guidance sets near the tets."""
    S, T, rate = CASES[case]
    img_s, img_t = images(5)
    rs = np.random.default_rng(6)
    sets = [[rs.uniform(1, 14, (9, 3)).astype(np.float32) for _ in range(2)] for _ in range(2)]
    el = np.ones(1, np.float32)
    pts = WIDE.astype(np.float32)
    args = (TETS, pts, el, sets[0], sets[1])
    prob = morea.Problem(DIMS, img_s, img_t, *args, radius=3.0, storage=storage, max_population=1)
    quant = [img_s, img_t] if storage == "f32" else [oracle.quantize(i, storage) for i in (img_s, img_t)]
    op = oracle.Problem(DIMS, quant[0], quant[1], *args, 3.0)
    cand = np.stack([np.asarray(S, np.float32).T, np.asarray(T, np.float32).T])[None]
    out = prob.eval_sobol(torch.from_numpy(np.ascontiguousarray(cand)).cuda(), rate=rate, seed=3)
    ref = op.evaluate_sobol(cand, rate=rate, seed=3)
    assert ref["counts"].min() > 100
    assert_parity(to_host(out), ref, what=case)


@pytest.mark.parametrize("pop", [1, 11, 12, 13, 40])
def test_candidates_do_not_depend_on_their_block(pop):
    """A population large enough for staged images (12 candidates a block, the
    last block partly filled) scores each candidate as it scores alone, up to
    the order of FP32 sums; a candidate far off, one partly outside and an
    invalid one leave their block's others alone."""
    n, cells = 40, 4
    pts, tets, fixed = synth.kuhn_grid((n, n, n), (cells, cells, cells))
    rs = np.random.default_rng(4)
    img = [(rs.uniform(0, 1, (n, n, n)) * (rs.uniform(0, 1, (n, n, n)) > 0.3)).astype(np.float32) for _ in range(2)]
    sets = [[rs.uniform(4, n - 5, (40, 3)).astype(np.float32)] for _ in range(2)]
    prob = morea.Problem((n, n, n), img[0], img[1], tets, pts, np.ones(len(tets), np.float32), sets[0], sets[1],
                         radius=4.0, max_population=pop)
    cands = np.stack([np.stack([(pts + np.where(fixed, 0, rs.normal(0, 0.4, pts.shape))).T for _ in range(2)])
                      for _ in range(pop)]).astype(np.float32)
    if pop >= 13:
        cands[3] += 9.0                  # partly outside
        cands[5, 1] *= 0.5               # other tets than its block's
        cands[7, 0, 1, 20] = np.nan
    t = torch.from_numpy(np.ascontiguousarray(cands)).cuda()
    out = to_host(prob.eval_sobol(t, rate=2.5, seed=6))
    for k in range(pop):
        one = to_host(prob.eval_sobol(t[k:k + 1].contiguous(), rate=2.5, seed=6))
        np.testing.assert_array_equal(out["counts"][k], one["counts"][0])
        np.testing.assert_array_equal(out["flags"][k], one["flags"][0])
        np.testing.assert_allclose(out["obj"][k], one["obj"][0], rtol=2e-6)
