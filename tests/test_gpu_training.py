"""GPU test of the surrogate's training kernels at batch sizes around their
tiles: 32 rows a wave, 128 a block's step, 32,768 a step of all 256 blocks."""
import numpy as np
import pytest

from conftest import synth_problem
from oracle import mlp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2303_04873_amd as morea  # noqa: E402

MAX_ROWS = 65536


@pytest.fixture(scope="module")
def surrogate():
    prob = morea.Problem.from_synth(synth_problem(1), max_population=1)
    return morea.Surrogate(prob, max_rows=MAX_ROWS, seed=3)


@pytest.mark.parametrize("rows", [1, 31, 32, 33, 127, 128, 129, 1000])
def test_gradients_and_step_at_tile_edges(surrogate, rows):
    """Every gradient entry against FP64 backpropagation with the kernels'
    BF16 rounding points.  Bound: FP32 accumulation (1e-4 of the entry's L1
    mass) plus two BF16 rounding flips of single terms (2^-7 of the largest
    term).  The first Adam step moves a parameter by lr g / (|g| + 1e-8),
    which FP32 rounding changes by less than 1e-5 of lr and one rounding of
    the parameter (2^-23 of it)."""
    s = surrogate
    rs = np.random.default_rng(rows)
    theta = np.concatenate([rs.normal(0, 0.3, 128 * 23), rs.normal(0, 0.1, 128), rs.normal(0, 0.12, 128 * 128),
                            rs.normal(0, 0.1, 257)]).astype(np.float32)
    s.set_params(theta)
    X = rs.normal(0, 1, (rows, mlp.N_IN)).astype(np.float32)
    t = rs.normal(0, 1, rows).astype(np.float32)
    dX, dt = torch.from_numpy(X).cuda(), torch.from_numpy(t).cuda()
    g, loss = s.gradients(dX, dt)
    g = g.cpu().numpy().astype(np.float64)
    lref = mlp.loss(theta, X, t, rnd=mlp.bf16)
    assert abs(loss.item() - lref) <= 1e-5 * lref
    rb = mlp.bf16
    p = mlp.unpack(theta)
    y, (Xb, z1, h1, z2, h2) = mlp.forward(theta, X, rb)
    dy = 2.0 * (y - t) / rows
    dz2 = np.outer(dy, p["w3"]) * (z2 > 0)
    dz2b = rb(dz2)
    dz1 = (dz2b @ rb(p["W2"])) * (h1 > 0)
    dz1b = rb(dz1)
    mass = [(np.abs(dz1b).T @ np.abs(Xb), np.abs(dz1b).max(0)[:, None] * np.abs(Xb).max(0)[None]),
            (np.abs(dz1).sum(0), np.abs(dz1).max(0)),
            (np.abs(dz2b).T @ np.abs(h1), np.abs(dz2b).max(0)[:, None] * np.abs(h1).max(0)[None]),
            (np.abs(dz2).sum(0), np.abs(dz2).max(0)),
            (np.abs(h2).T @ np.abs(dy), np.abs(h2).max(0) * np.abs(dy).max()),
            (np.array([np.abs(dy).sum()]), np.array([np.abs(dy).max()]))]
    l1, big = (np.concatenate([m[k].reshape(-1) for m in mass]) for k in (0, 1))
    ref = mlp.gradient(theta, X, t, rnd=rb)
    bad = np.abs(g - ref) > 1e-4 * l1 + 2.0 ** -7 * big + 1e-12
    assert not bad.any(), (rows, np.flatnonzero(bad)[:5], g[bad][:5], ref[bad][:5])

    fresh = morea.Surrogate(s.problem, max_rows=rows, seed=1)
    fresh.set_params(theta)
    out = torch.empty(1, device="cuda")
    fresh.train_step(dX, dt, 1e-3, loss_out=out)
    assert out.item() == loss.item()
    want = theta - 1e-3 * g / (np.abs(g) + 1e-8)
    assert np.all(np.abs(fresh.get_params() - want) <= 1e-8 + 2.0 ** -23 * np.abs(theta))


def test_gradients_of_a_batch_of_many_steps(surrogate):
    """65,536 rows (two steps of every block) against the sum of 64 batches of
    1,024, whose sizes are covered above.  A batch's terms are those of its
    parts times 1/64, exactly (BF16 rounding commutes with powers of two), so
    only the order of the FP32 sums differs: 1e-4 of the entry's L1 mass.  (A
    comparison with the FP64 reference does not bound a batch this large: an
    h1 on a BF16 rounding boundary can move a z2 across zero, which switches
    one row's whole term.)"""
    s = surrogate
    rs = np.random.default_rng(77)
    theta = np.concatenate([rs.normal(0, 0.3, 128 * 23), rs.normal(0, 0.1, 128), rs.normal(0, 0.12, 128 * 128),
                            rs.normal(0, 0.1, 257)]).astype(np.float32)
    s.set_params(theta)
    X = rs.normal(0, 1, (MAX_ROWS, mlp.N_IN)).astype(np.float32)
    t = rs.normal(0, 1, MAX_ROWS).astype(np.float32)
    dX, dt = torch.from_numpy(X).cuda(), torch.from_numpy(t).cuda()
    g, loss = s.gradients(dX, dt)
    parts = [s.gradients(dX[k:k + 1024], dt[k:k + 1024]) for k in range(0, MAX_ROWS, 1024)]
    want = torch.stack([p[0] for p in parts]).double().mean(0).cpu().numpy()
    assert abs(loss.item() - np.mean([p[1].item() for p in parts])) <= 1e-6 * loss.item()
    p = mlp.unpack(theta)
    y, (Xb, _, h1, z2, h2) = mlp.forward(theta, X, mlp.bf16)
    dy = np.abs(2.0 * (y - t) / MAX_ROWS)
    dz2 = np.outer(dy, np.abs(p["w3"])) * (z2 > 0)
    dz1 = np.abs((np.outer(2.0 * (y - t) / MAX_ROWS, p["w3"]) * (z2 > 0)) @ p["W2"]) * (h1 > 0)
    l1 = np.concatenate([m.reshape(-1) for m in (dz1.T @ np.abs(Xb), dz1.sum(0), dz2.T @ h1, dz2.sum(0),
                                                 h2.T @ dy, dy.sum()[None])])
    bad = np.abs(g.cpu().numpy() - want) > 1e-4 * l1 + 1e-12
    assert not bad.any(), np.flatnonzero(bad)[:5]
