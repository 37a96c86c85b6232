"""GPU test of the pre-screen around its tiles: 64 offspring a wave in two
network tiles of 32, runs of 1 to 8 tets by the amount of work, and slabs of
the offspring's coordinates."""
import numpy as np
import pytest

import synth
from conftest import oracle_problem, synth_problem
from oracle import surrogate_inputs
from test_gpu_surrogate import random_theta

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2303_04873_amd as morea  # noqa: E402

COLUMN_BYTES = 256 << 20


@pytest.fixture(scope="module")
def c1():
    p = synth_problem(1)
    prob = morea.Problem.from_synth(p, max_population=8)
    s = morea.Surrogate(prob, max_rows=1024, seed=3)
    s.set_params(random_theta(9, scale=0.5))
    parents, _ = synth.make_offspring(p, n_parents=5, per_parent=1, seed=7)
    cache = prob.new_cache(5)
    dp = torch.from_numpy(parents).cuda()
    prob.eval_full(dp, cache=cache)
    return p, prob, s, dp, cache


def offspring(p, dp, pop, seed):
    rs = np.random.default_rng(seed)
    of = rs.integers(0, len(dp), pop).astype(np.int32)
    pts = dp.cpu().numpy()[of] + rs.normal(0, 0.3, (pop,) + tuple(dp.shape[1:])).astype(np.float32)
    return torch.from_numpy(pts.astype(np.float32)).cuda(), torch.from_numpy(of).cuda()


@pytest.mark.parametrize("pop", [1, 31, 33, 63, 64, 65, 200, 1000])
def test_scores_equal_row_predictions(c1, pop):
    """Each score against the weighted row predictions over explicit feature
    rows: the network's outputs differ by the FP32 order of its sums (1e-5 of
    the change per tet), so 1e-4 of a score; invalid parents score +inf and
    leave the other lanes of their wave alone."""
    p, prob, s, dp, cache = c1
    do, of = offspring(p, dp, pop, pop)
    score = s.prescreen(do, dp, cache, of).cpu().numpy()
    feats = s.features(do, dp, cache, of)
    y = s.predict_rows(feats.reshape(-1, s.n_features).contiguous()).cpu().numpy().astype(np.float64).reshape(pop, -1)
    op = oracle_problem(1)
    rec = op.evaluate(dp.cpu().numpy(), records=True)["records"]
    want = surrogate_inputs.score(op, do.cpu().numpy(), rec, of.cpu().numpy(),
                                  y * s.h_scale / surrogate_inputs.h_scale(op))
    np.testing.assert_allclose(score, want, rtol=1e-4, atol=1e-6)
    bad = of.clone()
    bad[0::3] = -1
    bad[64:128] = len(dp)
    got = s.prescreen(do, dp, cache, bad).cpu().numpy()
    lost = (bad.cpu().numpy() < 0) | (bad.cpu().numpy() >= len(dp))
    assert np.all(np.isposinf(got[lost]))
    np.testing.assert_array_equal(got[~lost], score[~lost])


def test_slabs_of_coordinates_give_the_same_scores(c1):
    """More offspring than one slab of coordinates holds, 40 of them repeated:
    equal offspring score equal to the bit wherever they lie."""
    p, prob, s, dp, cache = c1
    n_points = dp.shape[-1]
    pop = COLUMN_BYTES // (36 * n_points) + 129
    do, of = offspring(p, dp, 40, 3)
    idx = torch.arange(pop, device="cuda") % 40
    score = s.prescreen(do[idx].contiguous(), dp, cache, of[idx].contiguous())
    assert torch.isfinite(score).all()
    assert torch.equal(score, score[:40][idx])
