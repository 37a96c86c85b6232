"""GPU test at the far end of the largest volumes (1024 x 1024 x 512 voxels,
the limit of 2^29), where the byte offset of an FP32 voxel passes 2^31: tets
there score as the oracle scores them in a small grid, the rest of the large
one being zero like the small one's surroundings."""
import numpy as np
import pytest

import oracle
from parity import assert_parity, to_host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2303_04873_amd as morea  # noqa: E402


def test_byte_offsets_beyond_2_31():
    n, first = 14, 498                                   # voxels 498 .. 511 of each axis
    rs = np.random.default_rng(12)
    small = [(rs.uniform(0, 1, (n, n, n)) * (rs.uniform(0, 1, (n, n, n)) > 0.4)).astype(np.float32) for _ in range(2)]
    dims = (1024, 1024, 512)
    assert ((first + n) * 1026 * 1026 * 4) > 1 << 31
    big = []
    for img in small:
        v = np.zeros(dims[::-1], np.float32)
        v[first:, first:first + n, first:first + n] = img
        big.append(v)
    pts = np.array([[1.5, 1.25, 1.75], [11.75, 2.0, 1.5], [2.25, 11.5, 2.0], [3.0, 3.5, 12.5], [12.25, 12.0, 12.25]],
                   np.float32)
    tets = np.array([[0, 1, 2, 3], [1, 2, 3, 4]], np.int32)
    el = np.ones(2, np.float32)
    moved = (np.round((pts + rs.normal(0, 0.3, pts.shape)).clip(1, 12.7) * 1024) / 1024).astype(np.float32)
    cands = np.stack([np.stack([pts.T, moved.T]), np.stack([moved.T, pts.T])]).astype(np.float32)
    prob = morea.Problem(dims, big[0], big[1], tets, pts + first, el, [], [], radius=1.0, max_population=2)
    op = oracle.Problem((n, n, n), small[0], small[1], tets, pts, el, [], [], 1.0)
    out = prob.eval_full(torch.from_numpy(np.ascontiguousarray(cands + first)).cuda())
    assert_parity(to_host(out), op.evaluate(cands), what="far end")
