"""GPU test of partial evaluation's launch forms: the shape that is reported
is the one that runs, so that setting it back changes nothing; the untuned
form (on problems where no shape is ever set), the grid and the persistent
one give the same bits with every storage, for even groups (grid by default)
and for uneven ones (persistent by default), and for lists of any length."""
import numpy as np
import pytest

import synth
from conftest import synth_problem
from parity import to_host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2303_04873_amd as morea  # noqa: E402


class Lists:
    """Evaluations (parent, group) of 6 parents of the 32^3 phantom."""

    def __init__(self, off, pts, ep, eg, storage="f32"):
        p = synth_problem(1)
        parents = synth.make_population(p, pop=6, seed=4, perturb_source=True, fold_fraction=0.25)
        rs = np.random.default_rng(len(ep))
        new = [parents[a][:, :, pts[off[g]:off[g + 1]]].transpose(2, 0, 1) for a, g in zip(ep, eg)]
        new = np.concatenate([v + rs.normal(0, 0.5, v.shape) for v in new]).astype(np.float32)
        self.prob = morea.Problem.from_synth(p, storage=storage, max_population=6)
        self.prob.set_groups(off, pts)
        self.prob.reserve_partial(len(ep))
        self.par = torch.from_numpy(parents).cuda()
        self.cache = self.prob.new_cache(6)
        self.prob.eval_full(self.par, cache=self.cache)
        self.rows = np.concatenate([[0], np.cumsum(np.diff(off)[eg])])
        self.args = tuple(torch.from_numpy(np.ascontiguousarray(a)).cuda()
                          for a in (ep.astype(np.int32), eg.astype(np.int32), new))

    def run(self, first=0, last=None):
        ep, eg, new = self.args
        last = len(ep) if last is None else last
        out = self.prob.eval_partial(self.par, self.cache, ep[first:last].clone(), eg[first:last].clone(),
                                     new[self.rows[first]:self.rows[last]].clone())
        torch.cuda.synchronize()
        return to_host(out)


def groups_of(kind):
    p = synth_problem(1)
    if kind == "even":
        return synth.make_groups(p, n_groups=8)
    # one group over most of the mesh and 300 of the point with the fewest tets
    tets_of = np.bincount(p.tets.ravel(), minlength=p.n_points)
    few, big = int(np.argmin(tets_of)), np.arange(min(p.n_points, 127))
    dep = int(np.isin(p.tets, big).any(axis=1).sum())
    assert dep > 64 * -(-(dep + 300 * int(tets_of[few])) // 301)
    off = np.concatenate([[0], len(big) + np.arange(301)])
    return off.astype(np.int32), np.concatenate([big, np.full(300, few)]).astype(np.int32)


def same(a, b, what):
    for k in a:
        np.testing.assert_array_equal(a[k], b[k], err_msg=f"{what} {k}")


@pytest.mark.parametrize("storage", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("kind", ["even", "uneven"])
def test_reported_shape_is_the_one_that_runs(kind, storage):
    off, pts = groups_of(kind)
    rs = np.random.default_rng(2)
    n = 150
    eg = rs.integers(0, len(off) - 1, n)
    eg[:3] = 0
    lists = Lists(off, pts, rs.integers(0, 6, n), eg, storage)
    prob = lists.prob
    shape = prob.partial_shape()
    assert (shape == (0, 0)) == (kind == "even")
    untuned = lists.run()
    prob.set_partial_shape(*shape)
    assert prob.partial_shape() == shape
    captures = morea.morea_partial_graphs(prob.handle)[1]
    same(lists.run(), untuned, "set back")
    assert morea.morea_partial_graphs(prob.handle)[1] - captures <= 1
    for other in [(0, 0), (256, 8), (5, 2)]:
        prob.set_partial_shape(*other)
        assert prob.partial_shape() == other
        same(lists.run(), untuned, f"shape {other}")


def test_shape_before_and_after_a_reservation():
    off, pts = groups_of("even")
    prob = morea.Problem.from_synth(synth_problem(1), max_population=1)
    assert prob.partial_shape() == (0, -1)
    prob.set_groups(off, pts)
    prob.reserve_partial(10)
    assert prob.partial_shape() == (0, 0)
    prob.set_groups(*groups_of("uneven"))
    prob.reserve_partial(10)
    blocks, chunk = prob.partial_shape()
    assert blocks > 0 and chunk == 8


@pytest.mark.parametrize("count", [1, 64, 65, 1023, 1024, 1025, 1600])
def test_untuned_parts_equal_the_whole(count):
    """No shape is ever set on these problems: the default dispatch at the
    edges of the one-block preparation and of one or two items a wave."""
    rs = np.random.default_rng(9)
    p = synth_problem(1)
    sizes = rs.integers(1, 4, 200)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    pts = np.concatenate([rs.choice(p.n_points, k, replace=False) for k in sizes]).astype(np.int32)
    n = 2600
    lists = Lists(off, pts, rs.integers(0, 6, n), rs.integers(0, 200, n))
    assert lists.prob.partial_shape() == (0, 0)
    whole = lists.run()
    for first in (0, n - count):
        part = lists.run(first, first + count)
        same(part, {k: v[first:first + count] for k, v in whole.items()}, f"{first}")


def test_grid_form_with_a_wide_bound():
    """2,400 evaluations with 2,000 items of two tets on average, but one group
    of 30,000: the grid covers 72 million items, whose waves fit a launch at
    two items each only."""
    rs = np.random.default_rng(11)
    n_tets, n_pts, n = 30000, 400, 2400
    pts = rs.uniform(1, 30, (n_pts, 3)).astype(np.float32)
    tets = np.stack([np.concatenate([[0], 2 + rs.choice(n_pts - 2, 3, replace=False)]) for _ in range(n_tets)])
    tets[0, 3] = 1                                    # the only tet of point 1
    v = pts[tets].astype(np.float64)
    tets = tets[np.abs(np.linalg.det(v[:, 1:] - v[:, :1])) > 1e-2].astype(np.int32)
    assert (tets == 1).sum() == 1
    dep = len(tets)
    img = [rs.uniform(0, 1, (32, 32, 32)).astype(np.float32) for _ in range(2)]
    prob = morea.Problem((32, 32, 32), img[0], img[1], tets, pts, np.ones(dep, np.float32), [], [], radius=1.0,
                         max_population=2)
    groups = np.ones(dep, np.int32)                   # point 1, but the first: point 0
    groups[0] = 0
    prob.set_groups(np.arange(dep + 1, dtype=np.int32), groups)
    prob.reserve_partial(n)
    assert prob.partial_shape() != (0, 0)             # uneven
    assert 1 << 26 <= n * dep < 1 << 27 and 2 * n <= 5120
    par = torch.from_numpy(np.stack([np.stack([pts.T, pts.T + np.float32(0.25)])] * 2)).cuda().contiguous()
    cache = prob.new_cache(2)
    prob.eval_full(par, cache=cache)
    ep = torch.from_numpy(rs.integers(0, 2, n).astype(np.int32)).cuda()
    eg = torch.from_numpy(np.where(np.arange(n) == 1200, 0, 5).astype(np.int32)).cuda()
    new = torch.from_numpy(rs.uniform(1, 30, (n, 2, 3)).astype(np.float32)).cuda()
    outs = []
    for shape in [(0, 0), (256, 8)]:
        prob.set_partial_shape(*shape)
        outs.append(to_host(prob.eval_partial(par, cache, ep, eg, new)))
    same(outs[0], outs[1], "grid and persistent")
