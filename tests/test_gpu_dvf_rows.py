"""GPU test of the DVF rasterizer's rows and batches where they can go wrong:
thin and one-voxel grids, rows longer than a batch, tets of many parts and
wider than 64 voxels (int64 planes), folded meshes with centres in several
tets and in none.  Against the oracle: coverage exact, displacements within
FP32 rounding of its exact barycentric images (2e-6 voxel + 1e-6 relative)."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2303_04873_amd as morea  # noqa: E402


@pytest.mark.parametrize("dims,mesh,move", [
    ((1, 1, 1), (2, 2, 2), 0.0), ((3, 1, 70), (2, 2, 2), 0.4), ((130, 5, 3), (2, 2, 2), 0.5),
    ((200, 9, 7), (3, 2, 2), 2.0), ((64, 64, 64), (2, 2, 2), 1.0), ((66, 67, 65), (2, 2, 2), 30.0),
    ((33, 31, 29), (4, 5, 3), 6.0), ((40, 24, 16), (6, 4, 3), 9.0)])
def test_rows_batches_and_parts(dims, mesh, move):
    pts, tets, fixed = synth.kuhn_grid(dims, mesh)
    rs = np.random.default_rng(sum(dims))
    flat = np.full(dims[::-1], 0.5, np.float32)
    args = (dims, flat, flat, tets, pts, np.ones(len(tets), np.float32))
    prob, op = morea.Problem(*args, max_population=1), oracle.Problem(*args, [], [], 1.0)
    covered = set()
    for k in range(2):
        S, T = (pts + (0.0 if k else 1.0) * np.where(fixed, 0.3, 1.0) * rs.normal(0, move, pts.shape)
                for _ in range(2))
        cand = np.ascontiguousarray(np.stack([S.T, T.T]), dtype=np.float32)
        out = prob.rasterize_dvf(torch.from_numpy(cand).cuda())
        fwd, inv, cover = op.dvf(cand)
        np.testing.assert_array_equal(out["cover"].cpu().numpy(), cover)
        np.testing.assert_allclose(out["fwd"].cpu().numpy(), fwd, rtol=1e-6, atol=2e-6)
        np.testing.assert_allclose(out["inv"].cpu().numpy(), inv, rtol=1e-6, atol=2e-6)
        covered |= set(np.unique(cover).tolist())
    if 6.0 <= move < 20.0:
        assert {0, 1, 2} <= covered
