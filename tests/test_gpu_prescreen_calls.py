"""GPU test of the pre-screen's sums: an offspring's score has the same bits
whatever the size of the call it is in, hence the length of the runs of tets
(8, 4, 2 or 1), also where the last eight tets are incomplete."""
import numpy as np
import pytest

import synth
from test_gpu_surrogate import random_theta

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2303_04873_amd as morea  # noqa: E402

ITEMS = 4096                 # work items that a call's runs are made short for


def run_length(n_tets, pop):
    run = 1
    while run < 8 and 2 * run * ITEMS <= n_tets * -(-pop // 64):
        run *= 2
    return run


@pytest.mark.parametrize("cells", [(4, 4, 4), (3, 3, 2), (5, 4, 5)])
def test_scores_do_not_depend_on_the_call(cells):
    n = 24
    pts, tets, fixed = synth.kuhn_grid((n, n, n), cells)
    rs = np.random.default_rng(len(tets))
    img = [(rs.uniform(0, 1, (n, n, n)) * (rs.uniform(0, 1, (n, n, n)) > 0.3)).astype(np.float32) for _ in range(2)]
    prob = morea.Problem((n, n, n), img[0], img[1], tets, pts, np.ones(len(tets), np.float32), [], [], radius=1.0,
                         max_population=6)
    s = morea.Surrogate(prob, max_rows=64, seed=3)
    s.set_params(random_theta(9, scale=0.5))
    par = [np.stack([pts.T, (pts + np.where(fixed, 0, rs.normal(0, 0.4, pts.shape))).T]) for _ in range(6)]
    par = torch.from_numpy(np.ascontiguousarray(np.stack(par), np.float32)).cuda()
    cache = prob.new_cache(6)
    prob.eval_full(par, cache=cache)
    pops = [1]
    for run in (2, 4, 8):                        # the smallest and the largest call of each length
        least = -(-run * ITEMS // len(tets)) * 64 - 63
        pops += [least - 1, least]
    assert [run_length(len(tets), p) for p in pops] == [1, 1, 2, 2, 4, 4, 8]
    pop = pops[-1]
    of = torch.from_numpy(rs.integers(0, 6, pop).astype(np.int32)).cuda()
    move = torch.randn((pop,) + tuple(par.shape[1:]), generator=torch.Generator().manual_seed(1)).cuda()
    off = (par[of.long()] + 0.3 * move).contiguous()
    whole = s.prescreen(off, par, cache, of)
    assert torch.isfinite(whole).all()
    for p in pops[:-1]:
        for first in (0, pop - p):
            part = s.prescreen(off[first:first + p].contiguous(), par, cache, of[first:first + p].contiguous())
            assert torch.equal(part, whole[first:first + p]), (p, first)
