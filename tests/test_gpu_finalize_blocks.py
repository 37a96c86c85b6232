"""GPU test of the per-candidate reduction's block, which follows the mesh's
tets and points (64, 256 or 1,024 threads): against the oracle on both sides of
each line, and bit for bit against the same mesh with points that no tet uses,
which takes the largest block."""
import numpy as np
import pytest

import oracle
from parity import assert_parity, to_host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2303_04873_amd as morea  # noqa: E402

DIMS = (26, 22, 20)


@pytest.mark.parametrize("n_tets,n_pts", [(1, 4), (63, 42), (64, 42), (65, 42), (64, 43), (255, 170), (256, 170),
                                          (257, 170), (256, 171)])
def test_blocks_give_the_same_sums(n_tets, n_pts):
    rs = np.random.default_rng(n_tets + n_pts)
    pts = (rs.uniform(0.5, 1, (n_pts, 3)) * (np.array(DIMS) - 2)).astype(np.float32)
    tets = []
    while len(tets) < n_tets:
        t = rs.choice(n_pts, 4, replace=False)
        v = pts[t].astype(np.float64)
        if abs(np.linalg.det(v[1:] - v[0])) > 1:
            tets.append(t)
    tets = np.array(tets, np.int32)
    img = [(rs.uniform(0, 1, DIMS[::-1]) * (rs.uniform(0, 1, DIMS[::-1]) > 0.3)).astype(np.float32) for _ in range(2)]
    sets = [[rs.uniform(10, 18, (30, 3)).astype(np.float32)] for _ in range(2)]
    el = rs.uniform(0.5, 2, n_tets).astype(np.float32)
    cands = np.stack([np.stack([pts.T, (pts + rs.normal(0, 0.4, pts.shape)).T]) for _ in range(5)]).astype(np.float32)
    cands[3, 1, 2, n_pts - 1] = np.inf
    outs, caches = [], []
    for extra in (0, 500):
        more = np.full((extra, 3), 1.0, np.float32)
        wide = np.concatenate([cands, np.broadcast_to(more.T, (5, 2, 3, extra))], axis=3)
        prob = morea.Problem(DIMS, img[0], img[1], tets, np.concatenate([pts, more]), el, sets[0], sets[1], radius=3.0,
                             max_population=5)
        caches.append(prob.new_cache(5))
        outs.append(to_host(prob.eval_full(torch.from_numpy(np.ascontiguousarray(wide)).cuda(), cache=caches[-1])))
    assert_parity(outs[0], oracle.Problem(DIMS, img[0], img[1], tets, pts, el, sets[0], sets[1], 3.0).evaluate(cands),
                  what="oracle")
    for k in outs[0]:
        np.testing.assert_array_equal(outs[0][k], outs[1][k], err_msg=k)
    assert torch.equal(caches[0], caches[1])
