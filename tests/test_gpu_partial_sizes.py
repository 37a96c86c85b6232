"""GPU test of partial evaluation's list sizes: the one-block preparation (up
to 1,024 evaluations) and the four launches beyond it, one item per wave and
two, the untuned form and the set ones.  An evaluation's outputs depend on
nothing else in its call, so every split of a list gives the same bits as the
whole; the whole's first evaluations are compared with the oracle."""
import numpy as np
import pytest

import synth
from conftest import oracle_problem, synth_problem
from parity import assert_parity, to_host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2303_04873_amd as morea  # noqa: E402

N = 2600


@pytest.fixture(scope="module")
def lists():
    """1,500 groups (more than a pass of the one block) of 1 to 3 points and
    2,600 evaluations of them, some with a parent or group out of range."""
    p = synth_problem(1)
    rs = np.random.default_rng(8)
    sizes = rs.integers(1, 4, 1500)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    pts = np.concatenate([rs.choice(p.n_points, k, replace=False) for k in sizes]).astype(np.int32)
    parents = synth.make_population(p, pop=9, seed=3, perturb_source=True, fold_fraction=0.25)
    prob = morea.Problem.from_synth(p, max_population=9)
    prob.set_groups(off, pts)
    prob.reserve_partial(N)
    par = torch.from_numpy(parents).cuda()
    cache = prob.new_cache(9)
    prob.eval_full(par, cache=cache)
    ep = rs.integers(0, 9, N).astype(np.int32)
    eg = rs.integers(0, 1500, N).astype(np.int32)
    ep[[5, 700, 2599]] = [9, -1, 50]
    eg[[6, 1024]] = [-1, 1500]
    rows = np.where((eg >= 0) & (eg < 1500), sizes[np.clip(eg, 0, 1499)], 0)
    start = np.concatenate([[0], np.cumsum(rows)])
    new = np.empty((start[-1], 2, 3), np.float32)
    for e in range(N):
        if rows[e]:
            idx = pts[off[eg[e]]:off[eg[e] + 1]]
            base = parents[np.clip(ep[e], 0, 8)][:, :, idx].transpose(2, 0, 1)
            new[start[e]:start[e + 1]] = base + rs.normal(0, 0.5, base.shape)
    dev = tuple(torch.from_numpy(a).cuda() for a in (ep, eg, new))
    out = prob.eval_partial(par, cache, *dev)
    torch.cuda.synchronize()
    want = to_host(out)
    kids, idx = [], [e for e in range(40) if e not in (5, 6)]
    for e in idx:
        child = parents[ep[e]].copy()
        child[:, :, pts[off[eg[e]]:off[eg[e] + 1]]] = new[start[e]:start[e + 1]].transpose(1, 2, 0)
        kids.append(child)
    assert_parity(want, oracle_problem(1).evaluate(np.stack(kids)), idx=idx, what="whole list")
    assert all(want["flags"][e] == 4 and np.isnan(want["obj"][e]).all() for e in (5, 6, 700, 1024, 2599))
    return prob, par, cache, dev, start, want


@pytest.mark.parametrize("shape", [None, (0, 0), (256, 8)])
@pytest.mark.parametrize("count", [1, 64, 65, 1023, 1024, 1025, 1600])
def test_parts_equal_the_whole(lists, count, shape):
    prob, par, cache, (ep, eg, new), start, want = lists
    if shape is not None:
        prob.set_partial_shape(*shape)
    for e0 in (0, N - count):
        part = (ep[e0:e0 + count].clone(), eg[e0:e0 + count].clone(), new[start[e0]:start[e0 + count]].clone())
        if part[2].numel() == 0:
            part = part[:2] + (new[:1].clone(),)
        out = prob.eval_partial(par, cache, *part)
        torch.cuda.synchronize()
        for k, v in to_host(out).items():
            np.testing.assert_array_equal(v, want[k][e0:e0 + count], err_msg=k)
