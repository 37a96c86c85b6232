"""GPU test of populations whose per-candidate reduction takes more threads
than one axis of a launch holds (2^22 candidates of 1,024 threads)."""
import numpy as np
import pytest

from parity import to_host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2303_04873_amd as morea  # noqa: E402

DISTINCT = 7


@pytest.mark.parametrize("pop", [(1 << 21) - 1, 1 << 21, (1 << 22) + 3])
def test_repeated_candidates_score_alike(pop):
    """A mesh of one tet; `pop` candidates repeat seven, whose outputs alone
    they equal to the bit, with both estimators; so do their caches."""
    rs = np.random.default_rng(3)
    img = [rs.uniform(0, 1, (6, 6, 6)).astype(np.float32) for _ in range(2)]
    pts = np.array([[0.5, 0.25, 0.5], [4.5, 0.5, 1.0], [1.0, 4.25, 0.5], [1.5, 1.0, 4.75]], np.float32)
    prob = morea.Problem((6, 6, 6), img[0], img[1], np.array([[0, 1, 2, 3]], np.int32), pts, np.ones(1, np.float32),
                         [], [], radius=1.0, max_population=pop)
    few = np.stack([np.stack([(pts + rs.normal(0, 0.3, pts.shape)).T for _ in range(2)]) for _ in range(DISTINCT)])
    few[3, 0, 1, 2] = np.nan
    few = torch.from_numpy(np.ascontiguousarray(few.astype(np.float32))).cuda()
    idx = torch.arange(pop, device="cuda") % DISTINCT
    many = few[idx].contiguous()
    for run in (prob.eval_full, lambda t: prob.eval_sobol(t, rate=3.0, seed=2)):
        alone = to_host(run(few))
        out = run(many)
        for k, v in out.items():
            want = torch.from_numpy(alone[k]).cuda()[idx]
            assert torch.equal(torch.nan_to_num(v.float(), nan=-7.0), torch.nan_to_num(want.float(), nan=-7.0)), k
    caches = []
    for t in (few, many):
        caches.append(prob.new_cache(len(t)))
        prob.eval_full(t, cache=caches[-1])
    for first, size in ((0, 48), (48, 64)):           # two records a candidate, then its totals
        part = [c.view(torch.uint8)[first * n:(first + size) * n].view(n, size)
                for c, n in zip(caches, (DISTINCT, pop))]
        assert torch.equal(part[1], part[0][idx])
