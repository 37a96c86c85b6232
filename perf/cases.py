"""Measured workloads of the library, each through its public entry points.

A case is a dict of plain values; ``kind`` names the call:

  evaluate   full evaluation of a population (Problem.eval_full), with or without the per-tet cache
  sobol      the random-sampling estimator on a population (Problem.eval_sobol)
  partial    partial evaluations of every (parent, point group) pair (Problem.eval_partial)
  mixing     one colour of a generation: distributions, sampled children, their partial evaluations
  gradients  loss and gradients of one surrogate training batch (Surrogate.gradients)
  prescreen  scores of a batch of offspring (Surrogate.prescreen)
  dvf        forward and inverse deformation fields of one candidate (Problem.rasterize_dvf)
  archive    selection and clusters of a population, then offers to the elitist archive

Inputs are drawn on the GPU from the seed: phantom image pairs of smooth ellipsoids with exact
background, warped into each other with one organ missing in the target; the Kuhn mesh over the grid;
guidance points on the organ surfaces; populations around the grid (source) and the warped grid
(target).  ``exact`` evaluates the definitions in 64 bits with plain torch operations.
"""
import math

import numpy as np
import torch

import paper_2303_04873_amd as morea

DEV = "cuda"
ONE = 1024            # fixed-point units per voxel: coordinates are snapped to 2^-10 voxel
N_FEATURES, HIDDEN = 23, 128


# ------------------------------------------------------------------------------------ cases

def listed():
    g128 = dict(nx=128, ny=128, nz=96, mx=10, my=10, mz=8, storage="f32", sigma=0.5)
    g32 = dict(nx=32, ny=32, nz=32, mx=5, my=5, mz=5, storage="f32", sigma=0.5)
    g192 = dict(nx=192, ny=192, nz=128, mx=14, my=14, mz=10, sigma=0.5)
    return [
        # a small phantom's population: launches and latency count
        dict(g32, name="evaluate_32_pop16", kind="evaluate", pop=16, cache=False),
        # the benchmark's population; the cache is kept as the optimizer does
        dict(g128, name="evaluate_128_pop512", kind="evaluate", pop=512, cache=True),
        # the larger image pair, stored in 16 bits to halve its memory
        dict(g192, name="evaluate_192_bf16_pop256", kind="evaluate", pop=256, cache=False, storage="bf16"),
        # a cropped pair whose sides fit no tile, a few candidates
        dict(name="evaluate_97x113x71_f16_pop37", kind="evaluate", nx=97, ny=113, nz=71, mx=8, my=9, mz=6,
             storage="f16", sigma=0.5, pop=37, cache=True),
        # a batch of uneven partial evaluations: every parent with every point group
        dict(g128, name="partial_128_512x64", kind="partial", pop=512, groups=64, gmin=4, gmax=48),
        # the same call on a small problem with few children
        dict(g32, name="partial_32_16x8", kind="partial", pop=16, groups=8, gmin=2, gmax=8),
        # one colour of an optimizer generation: estimate, sample, evaluate the children
        dict(g128, name="mixing_128_pop512", kind="mixing", pop=512, clusters=10, members=36),
        # the estimator with random points
        dict(g128, name="sobol_128_pop128", kind="sobol", pop=128, rate=1.0),
        # one training batch of the surrogate
        dict(name="gradients_65536", kind="gradients", rows=65536),
        # a batch of offspring ranked before the exact evaluation
        dict(g128, name="prescreen_128_4096", kind="prescreen", pop=512, per_parent=8),
        # the fields of a finished registration
        dict(g128, name="dvf_128", kind="dvf"),
        # the bookkeeping of two generations: eight offers of a population
        dict(name="archive_512x8", kind="archive", pop=512, batches=8, capacity=2000, clusters=10, points=800),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["evaluate", "evaluate", "partial", "partial", "mixing", "sobol", "gradients", "prescreen",
                       "dvf", "archive"])
    if kind == "gradients":
        return dict(kind=kind, rows=_log_int(rng, 1000, 200000))
    if kind == "archive":
        pop = _log_int(rng, 24, 900)
        return dict(kind=kind, pop=pop, batches=rng.randint(1, 8), capacity=_log_int(rng, 50, 2000),
                    clusters=rng.randint(1, 10), points=_log_int(rng, 100, 1000))
    nx = _log_int(rng, 24, 150)
    ny, nz = (max(16, int(nx * rng.uniform(0.6, 1.1))) for _ in range(2))
    cell = rng.uniform(8.0, 16.0)
    c = dict(kind=kind, nx=nx, ny=ny, nz=nz, storage=rng.choice(["f32", "f32", "bf16", "f16"]),
             sigma=round(rng.uniform(0.2, 0.7), 2))
    c.update(mx=max(3, round(nx / cell) + 1), my=max(3, round(ny / cell) + 1), mz=max(3, round(nz / cell) + 1))
    most = max(8, min(700, int(7e8 / (nx * ny * nz))))
    if kind == "evaluate":
        c.update(pop=_log_int(rng, 4, most), cache=rng.random() < 0.5)
    elif kind == "sobol":
        c.update(pop=_log_int(rng, 4, max(8, most // 4)), rate=round(rng.uniform(0.25, 1.5), 2))
    elif kind == "partial":
        c.update(pop=_log_int(rng, 4, min(200, most)), groups=_log_int(rng, 4, 64), gmin=rng.randint(1, 4),
                 gmax=rng.randint(5, 48))
    elif kind == "mixing":
        c.update(pop=_log_int(rng, 24, max(32, most)), clusters=rng.randint(1, 10), members=rng.randint(8, 24))
    elif kind == "prescreen":
        tets = 6 * (c["mx"] - 1) * (c["my"] - 1) * (c["mz"] - 1)
        c.update(pop=_log_int(rng, 4, max(8, min(most // 2, int(1.4e7 / (8 * tets))))), per_parent=rng.randint(1, 8))
    return c


# ----------------------------------------------------------------------------------- inputs

def _generator(seed):
    return torch.Generator(device=DEV).manual_seed(1000003 * (seed % (1 << 40)) + 17)


def _mesh(c):
    """Grid points [n][3], 6 Kuhn tets per cell, and the coordinates pinned to the box faces."""
    shape, dims = (c["mx"], c["my"], c["mz"]), (c["nx"], c["ny"], c["nz"])
    ax = [-0.5 + np.arange(p) * (n / (p - 1)) for p, n in zip(shape, dims)]
    k, j, i = np.meshgrid(*(np.arange(p) for p in shape[::-1]), indexing="ij")
    ijk = np.stack([i.ravel(), j.ravel(), k.ravel()], -1)
    points = np.stack([ax[a][ijk[:, a]] for a in range(3)], -1)
    step = np.array([1, shape[0], shape[0] * shape[1]])
    cell = ijk[(ijk < np.array(shape) - 1).all(1)] @ step
    perms = [(0, 1, 2), (0, 2, 1), (1, 0, 2), (1, 2, 0), (2, 0, 1), (2, 1, 0)]
    corners = np.array([np.concatenate([[0], np.cumsum(step[list(p)])]) for p in perms])
    tets = (cell[:, None, None] + corners[None]).reshape(-1, 4).astype(np.int32)
    fixed = (ijk == 0) | (ijk == np.array(shape) - 1)
    return points.astype(np.float32), tets, fixed, ijk


def _registration(c, seed):
    """Image pair, mesh, guidance sets and a true displacement of one synthetic registration."""
    rng = np.random.default_rng([seed, 1])
    gen = _generator(seed)
    n = np.array([c["nx"], c["ny"], c["nz"]], dtype=np.float64)
    centres, semi = rng.uniform(0.3 * n, 0.7 * n, (6, 3)), rng.uniform(0.12 * n, 0.25 * n, (6, 3))
    values = rng.uniform(0.2, 0.9, 6)
    bumps, weights = rng.uniform(0.2 * n, 0.8 * n, (4, 3)), rng.normal(size=(4, 3))
    width = n.mean() / 4
    z, y, x = torch.meshgrid(*(torch.arange(int(m), device=DEV, dtype=torch.float64) for m in n[::-1]),
                             indexing="ij")
    grid = torch.stack([x, y, z], -1)

    def shift(p, w):
        u = torch.zeros_like(p)
        for b, v in zip(bumps, w):
            r2 = (p - torch.tensor(b, device=DEV)).square().sum(-1, keepdim=True)
            u += torch.tensor(v, device=DEV) * torch.exp(-r2 / (2 * width * width))
        return u

    weights *= 0.094 * n[0] / float(shift(grid[::4, ::4, ::4], weights).norm(dim=-1).max())

    def organs(p, which):
        out = torch.zeros(p.shape[:-1], device=DEV, dtype=torch.float64)
        for k in which:
            rho = ((p - torch.tensor(centres[k], device=DEV)) / torch.tensor(semi[k], device=DEV)).norm(dim=-1)
            t = (((1 - rho) * float(np.cbrt(semi[k].prod())) + 1) * 0.5).clamp(0, 1)
            out = torch.maximum(out, values[k] * t * t * (3 - 2 * t))
        return out

    back = grid.clone()
    for _ in range(12):
        back = grid - shift(back, weights)
    images = []
    for clean in (organs(grid, range(6)), organs(back, range(5))):
        noise = torch.randn(clean.shape, generator=gen, device=DEV)
        images.append(torch.where(clean > 0, (clean + 0.02 * noise).clamp(0, 1), 0).float().contiguous())
    points, tets, fixed, ijk = _mesh(c)
    ref = torch.tensor(points, device=DEV, dtype=torch.float64)
    move = shift(ref, weights)
    move[torch.tensor(fixed, device=DEV)] = 0
    sets_s, sets_t = [], []
    for k in range(5):
        d = rng.normal(size=(40, 3))
        s = torch.tensor(centres[k] + d / np.linalg.norm(d, axis=1, keepdims=True) * semi[k], device=DEV)
        sets_s.append(s.float().cpu().numpy())
        sets_t.append((s + shift(s, weights)).float().cpu().numpy())
    el = rng.choice([0.5, 1.0, 10.0], len(tets), p=[0.2, 0.7, 0.1]).astype(np.float32)
    return dict(images=images, points=points, tets=tets, fixed=fixed, ijk=ijk, elasticity=el, sets=(sets_s, sets_t),
                radius=max(0.8, 0.025 * c["nx"]), ref=ref, target=(ref + move).float().double(), gen=gen, rng=rng)


def _population(r, pop, sigma, source=True, folds=True):
    """Candidates [pop][2][3][n_points]; every 16th has one point pushed through a face of its tet."""
    free = torch.tensor(~r["fixed"].T, device=DEV)
    base = torch.stack([r["ref"].T, r["target"].T])
    noise = torch.randn((pop, 2, 3, len(r["points"])), generator=r["gen"], device=DEV) * sigma * free
    if not source:
        noise[:, 0] = 0
    pts = (base + noise).float()
    interior = np.flatnonzero(~r["fixed"].any(1))
    for c in range(0, pop if folds and interior.size else 0, 16):
        v, m = int(r["rng"].choice(interior)), int(r["rng"].integers(2))
        tet = r["tets"][int(r["rng"].choice(np.flatnonzero((r["tets"] == v).any(1))))]
        face = pts[c, m][:, torch.tensor(tet[tet != v].astype(np.int64), device=DEV)].mean(1)
        pts[c, m, :, v] = face + 0.3 * (face - pts[c, m, :, v])
    return pts.contiguous()


def _groups(r, c):
    """Point groups grown breadth-first over the mesh's edges (CSR)."""
    shape = (c["mx"], c["my"], c["mz"])
    near = [d for d in np.ndindex(3, 3, 3) if any(v != 1 for v in d)]
    near = [np.array(d) - 1 for d in near]
    near = [d for d in near if d.min() >= 0 or d.max() <= 0]
    off, pts = [0], []
    for _ in range(c["groups"]):
        size = min(int(r["rng"].integers(c["gmin"], c["gmax"] + 1)), len(r["points"]))
        queue = [int(r["rng"].integers(len(r["points"])))]
        seen = set(queue)
        for v in queue:
            if len(queue) >= size:
                break
            for d in near:
                q = r["ijk"][v] + d
                w = int(q[0] + shape[0] * (q[1] + shape[1] * q[2]))
                if (q >= 0).all() and (q < shape).all() and w not in seen:
                    seen.add(w)
                    queue.append(w)
        pts += queue[:size]
        off.append(len(pts))
    return np.array(off, np.int32), np.array(pts, np.int32)


def _elements(r, c):
    """Pairs of points along x that cover the mesh, and one colour of them whose tets are disjoint."""
    ijk, row = r["ijk"], c["mx"]
    first = np.flatnonzero((ijk[:, 0] % 2 == 0) & (ijk[:, 0] + 1 < row))
    colour = np.flatnonzero((ijk[first] % np.array([4, 2, 2]) == 0).all(1))
    return np.stack([first, first + 1], 1).astype(np.int32), colour.astype(np.int32)


def _inputs(c, seed):
    """Everything that a case reads, as tensors and arrays; the same for the same seed."""
    kind = c["kind"]
    if kind == "gradients":
        gen, n = _generator(seed), c["rows"]
        x = torch.randn((n, N_FEATURES), generator=gen, device=DEV)
        x[:, 12:15] *= 0.4
        x[:, 15:] = x[:, 15:].abs() * 0.3
        w = torch.randn(N_FEATURES, generator=gen, device=DEV) * 0.1
        y = torch.tanh(x @ w) * x[:, 22] + 0.5 * x[:, 13] + 0.02 * torch.randn(n, generator=gen, device=DEV)
        return dict(feats=x.contiguous(), targets=y.contiguous(), params=_params(seed))
    if kind == "archive":
        return _objectives(c, seed)
    r = _registration(c, seed)
    if kind in ("evaluate", "sobol"):
        r["pts"] = _population(r, c["pop"], c["sigma"])
    elif kind == "dvf":
        r["pts"] = _population(r, 1, 2 * c["sigma"], folds=seed % 2 == 0)
    elif kind == "partial":
        r["pts"] = _population(r, c["pop"], c["sigma"])
        off, gp = _groups(r, c)
        r["groups"] = off, gp
        r["ep"] = torch.arange(c["pop"], device=DEV, dtype=torch.int32).repeat_interleave(len(off) - 1)
        r["eg"] = torch.arange(len(off) - 1, device=DEV, dtype=torch.int32).repeat(c["pop"])
        old = r["pts"][:, :, :, torch.tensor(gp.astype(np.int64), device=DEV)].permute(0, 3, 1, 2)
        free = torch.tensor(~r["fixed"][gp], device=DEV)[None, :, None, :]
        noise = torch.randn(old.shape, generator=r["gen"], device=DEV) * 0.5 * free
        r["new"] = (old + noise).reshape(-1, 2, 3).contiguous()
    elif kind == "mixing":
        r["pts"] = _population(r, c["pop"], c["sigma"])
        r["elements"], colour = _elements(r, c)
        r["eg"] = torch.tensor(colour, device=DEV).repeat(c["pop"])
        r["ep"] = torch.arange(c["pop"], device=DEV, dtype=torch.int32).repeat_interleave(len(colour))
        cluster = torch.randint(c["clusters"], (c["pop"],), generator=r["gen"], device=DEV, dtype=torch.int32)
        r["ec"] = cluster[r["ep"].long()].contiguous()
        members = [np.sort(r["rng"].choice(c["pop"], min(c["members"], c["pop"]), replace=False))
                   for _ in range(c["clusters"])]
        r["off"] = torch.tensor(np.cumsum([0] + [len(m) for m in members]), device=DEV, dtype=torch.int32)
        r["members"] = torch.tensor(np.concatenate(members), device=DEV, dtype=torch.int32)
        r["z"] = torch.randn((2 * len(r["ep"]), 2, 3), generator=r["gen"], device=DEV)
        r["pinned"] = torch.tensor(r["fixed"] @ np.array([1, 2, 4]), device=DEV, dtype=torch.uint8)
    else:
        r["parents"] = _population(r, c["pop"], c["sigma"], source=False, folds=False)
        r["of"] = torch.arange(c["pop"], device=DEV, dtype=torch.int32).repeat_interleave(c["per_parent"])
        r["pts"] = r["parents"][r["of"].long()].clone()
        noise = torch.randn(r["pts"][:, 1].shape, generator=r["gen"], device=DEV) * 0.5
        r["pts"][:, 1] += noise * torch.tensor(~r["fixed"].T, device=DEV)
        r["params"] = _params(seed)
    return r


def _params(seed):
    """Network parameters: W1, b1, W2, b2, w3, b3."""
    rng = np.random.default_rng([seed, 2])
    parts = [rng.normal(0, (2 / N_FEATURES) ** 0.5, HIDDEN * N_FEATURES), rng.normal(0, 0.05, HIDDEN),
             rng.normal(0, (2 / HIDDEN) ** 0.5, HIDDEN * HIDDEN), rng.normal(0, 0.05, HIDDEN),
             rng.normal(0, 0.05, HIDDEN), rng.normal(0, 0.05, 1)]
    return np.concatenate(parts).astype(np.float32)


def _objectives(c, seed):
    """Objective vectors near a trade-off surface that improves from batch to batch; a few folded."""
    gen = _generator(seed)
    batches = []
    for b in range(c["batches"]):
        u = torch.rand((c["pop"], 3), generator=gen, device=DEV).clamp_min(1e-6)
        u = u / u.norm(dim=1, keepdim=True)
        d = 1 - u * (0.8 + 0.01 * b) + 0.02 * torch.rand((c["pop"], 1), generator=gen, device=DEV)
        obj = d * torch.tensor([0.04, 0.6, 1e-3], device=DEV)
        folded = torch.rand(c["pop"], generator=gen, device=DEV) < 0.03
        batches.append(dict(obj=obj.float().contiguous(), flags=folded.to(torch.uint8),
                            severity=torch.where(folded, 10 * u[:, 0], 0).contiguous()))
    pts = torch.rand((c["pop"], 2, 3, c["points"]), generator=gen, device=DEV) * 100
    return dict(batches=batches, pts=pts)


def _stored(r, c):
    kind = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[c["storage"]]
    return [im.to(kind).double() for im in r["images"]]


def _problem(r, c, pop):
    a, b = (im.cpu().numpy() for im in r["images"])
    return morea.Problem((c["nx"], c["ny"], c["nz"]), a, b, r["tets"], r["points"], r["elasticity"], *r["sets"],
                         radius=r["radius"], storage=c["storage"], max_population=pop)


def prepare(case, seed):
    c, kind = case, case["kind"]
    s = dict(kind=kind, case=c, **_inputs(c, seed))
    if kind == "gradients":
        pts, tets, _, _ = _mesh(dict(nx=8, ny=8, nz=8, mx=2, my=2, mz=2))
        flat = np.full((8, 8, 8), 0.5, np.float32)
        s["problem"] = morea.Problem((8, 8, 8), flat, flat, tets, pts, np.ones(len(tets), np.float32))
        s["surrogate"] = morea.Surrogate(s["problem"], max_rows=c["rows"])
        s["surrogate"].set_params(s["params"])
        return s
    if kind == "archive":
        s["archive"] = morea.Archive(c["capacity"], n_points=c["points"])
        return s
    prob = s["problem"] = _problem(s, c, len(s["pts"]))
    if kind in ("evaluate", "sobol"):
        s["out"] = prob.outputs(c["pop"])
        s["cache"] = prob.new_cache(c["pop"]) if c.get("cache") else None
    elif kind in ("partial", "mixing"):
        off, gp = s["groups"] if kind == "partial" else (
            np.arange(0, s["elements"].size + 1, 2, dtype=np.int32), s["elements"].reshape(-1))
        prob.set_groups(off, gp)
        prob.reserve_partial(len(s["ep"]))
        s["cache"] = prob.new_cache(c["pop"])
        prob.eval_full(s["pts"], cache=s["cache"])
        s["out"] = prob.outputs(len(s["ep"]))
        if kind == "mixing":
            s["work"] = prob.mixing_workspace(c["clusters"])
            s["new"] = torch.empty_like(s["z"])
    elif kind == "prescreen":
        s["cache"] = prob.new_cache(c["pop"])
        prob.eval_full(s["parents"], cache=s["cache"])
        s["surrogate"] = morea.Surrogate(prob, max_rows=1024)
        s["surrogate"].set_params(s["params"])
        s["score"] = torch.empty(len(s["pts"]), device=DEV)
    elif kind == "dvf":
        shape = (c["nz"], c["ny"], c["nx"])
        s["out"] = dict(fwd=torch.empty(shape + (3,), device=DEV), inv=torch.empty(shape + (3,), device=DEV),
                        cover=torch.empty((2,) + shape, dtype=torch.int32, device=DEV),
                        work=torch.empty((2,) + shape, dtype=torch.int32, device=DEV))
    return s


# -------------------------------------------------------------------------------------- run

def run(state):
    s, kind = state, state["kind"]
    if kind == "gradients":
        grads, loss = s["surrogate"].gradients(s["feats"], s["targets"])
        return dict(grads=grads, loss=loss)
    if kind == "archive":
        first, c, arc = s["batches"][0], s["case"], s["archive"]
        sel = morea.select_clusters(first, round(0.35 * c["pop"]), c["clusters"])
        arc.clear()
        entered = [arc.update(b, pts=s["pts"]) for b in s["batches"]]
        n_sel = torch.arange(c["pop"], device=DEV) < sel["n_selected"]
        n_mem = torch.arange(sel["clu_members"].numel(), device=DEV) < sel["clu_off"][-1]
        held = arc.stamp >= 0
        return dict(selection=sel["selection"] * n_sel, n_selected=sel["n_selected"], offsets=sel["clu_off"],
                    members=sel["clu_members"] * n_mem, cluster_of=sel["cluster_of"],
                    inserted=[e[0] for e in entered], slots=[e[1] for e in entered], obj=arc.obj, stamp=arc.stamp,
                    pts=torch.where(held[:, None, None, None], arc.pts, 0.0), state=arc.state, best=arc.best)
    prob = s["problem"]
    if kind == "evaluate":
        prob.eval_full(s["pts"], cache=s["cache"], out=s["out"])
        return s["out"] if s["cache"] is None else dict(s["out"], **_cache_views(s["cache"], s["case"], prob.n_tets))
    if kind == "sobol":
        return prob.eval_sobol(s["pts"], rate=s["case"]["rate"], seed=7, out=s["out"])
    if kind == "mixing":
        k = s["case"]["clusters"]
        prob.estimate_distributions(s["pts"], s["off"], s["members"], s["work"], pinned=s["pinned"])
        prob.sample_partial(s["pts"], s["work"], k, s["ep"], s["eg"], s["ec"], s["z"], pinned=s["pinned"],
                            out=s["new"])
    if kind in ("partial", "mixing"):
        prob.eval_partial(s["pts"], s["cache"], s["ep"], s["eg"], s["new"], out=s["out"])
        return s["out"] if kind == "partial" else dict(s["out"], new=s["new"])
    if kind == "prescreen":
        return s["surrogate"].prescreen(s["pts"], s["parents"], s["cache"], s["of"], score=s["score"])
    out = prob.rasterize_dvf(s["pts"][0], out=s["out"])
    return dict(fwd=out["fwd"], inv=out["inv"], cover=out["cover"])


def _cache_views(cache, c, n_tets):
    """The fields of the cache's records [pop][n_tets][2], read in place."""
    n = c["pop"] * n_tets * 2
    f = cache[:24 * n].view(torch.float32).view(c["pop"], n_tets, 2, 6)
    i = cache[:24 * n].view(torch.int32).view(c["pop"], n_tets, 2, 6)
    return dict(rec_h=f[..., 0], rec_g=f[..., 1], rec_n=i[..., 2], rec_mag=f[..., 3], rec_vol=f[..., 4],
                rec_bits=i[..., 5])


# ------------------------------------------------------------------------------------- work

def work(case):
    """Bytes: each input read and each output written once.  Operations: 60 per voxel sample (map,
    trilinear read, h, sums), 240 per random point, the dense layers of the surrogate, 50 per field value."""
    c, kind = case, case["kind"]
    net = 2 * (N_FEATURES * HIDDEN + HIDDEN * HIDDEN + HIDDEN)
    if kind == "gradients":
        return dict(bytes=4 * c["rows"] * (N_FEATURES + 1) + 8 * 19713, flops=3 * net * c["rows"])
    if kind == "archive":
        pts = 24 * c["points"]
        kept = min(c["capacity"], c["pop"] * c["batches"])
        return dict(bytes=c["batches"] * c["pop"] * 22 + 2 * pts * kept + 16 * c["capacity"],
                    flops=8 * c["batches"] * c["pop"] * (c["pop"] + kept))
    voxels, tets = c["nx"] * c["ny"] * c["nz"], 6 * (c["mx"] - 1) * (c["my"] - 1) * (c["mz"] - 1)
    points = c["mx"] * c["my"] * c["mz"]
    images = 2 * voxels * (4 if c["storage"] == "f32" else 2)
    if kind == "dvf":
        return dict(bytes=24 * points + 2 * voxels * 16, flops=50 * 2 * voxels)
    cand = 24 * points
    if kind in ("evaluate", "sobol"):
        ops = 60 if kind == "evaluate" else 240 * c["rate"]
        rec = 48 * tets * c["pop"] if c.get("cache") else 0
        return dict(bytes=images + c["pop"] * (cand + 25) + rec, flops=ops * 2 * voxels * c["pop"])
    if kind == "prescreen":
        n = c["pop"] * c["per_parent"]
        return dict(bytes=images + (n + c["pop"]) * cand + 48 * tets * c["pop"] + 4 * n,
                    flops=n * tets * (net + 26 * 2 * 20))
    per = tets / points
    if kind == "mixing":
        evals = c["pop"] * max(1, points // 16)
        share = min(1.0, 36 / tets)
        size = 2
    else:
        evals, size = c["pop"] * c["groups"], (c["gmin"] + c["gmax"]) / 2
        share = min(1.0, 3 * size * per / tets)
    return dict(bytes=images + c["pop"] * (cand + 48 * tets) + evals * (33 + 24 * size),
                flops=60 * 2 * voxels * share * evals)


# ------------------------------------------------------------------------------------ exact

FACES = [(1, 2, 3), (0, 2, 3), (0, 3, 1), (0, 1, 2)]


def _cross(u, w):
    return torch.stack([u[..., 1] * w[..., 2] - u[..., 2] * w[..., 1], u[..., 2] * w[..., 0] - u[..., 0] * w[..., 2],
                        u[..., 0] * w[..., 1] - u[..., 1] * w[..., 0]], -1)


def _det(v):
    return (_cross(v[:, 1] - v[:, 0], v[:, 2] - v[:, 0]) * (v[:, 3] - v[:, 0])).sum(-1)


def _spread(counts):
    """For items with these counts: the item of every unit and the unit's place in its item."""
    item = torch.arange(len(counts), device=DEV).repeat_interleave(counts)
    return item, torch.arange(len(item), device=DEV) - (counts.cumsum(0) - counts)[item]


def _voxels(own, dims):
    """Voxel centres of tets own [m][4][3] (fixed point): tet, voxel [n][3] and barycentrics 1..3 in 64 bits."""
    d = _det(own)
    normal, base, lex = [], [], []
    for i, (b, u, w) in enumerate(FACES):
        n = _cross(own[:, u] - own[:, b], own[:, w] - own[:, b])
        n = n * torch.sign((n * (own[:, i] - own[:, b])).sum(-1, keepdim=True))
        x, y, z = n.unbind(-1)
        lex.append(((x > 0) | ((x == 0) & ((y > 0) | ((y == 0) & (z > 0))))).long())
        normal.append(n)
        base.append(own[:, b])
    top = torch.tensor(dims, device=DEV) - 1
    lo = (-torch.div(-own.amin(1), ONE, rounding_mode="floor")).clamp_min(0)
    hi = torch.minimum(torch.div(own.amax(1), ONE, rounding_mode="floor"), top)
    size = torch.where((d != 0)[:, None], hi - lo + 1, 0).clamp_min(0)
    t, r = _spread(torch.where((size > 0).all(1), size[:, 1] * size[:, 2], 0))
    ny = size[t, 1]
    p = torch.stack([lo[t, 0], lo[t, 1] + r % ny, lo[t, 2] + torch.div(r, ny, rounding_mode="floor")], -1)
    js, je = torch.zeros_like(t), size[t, 0] - 1
    at = []
    for i in range(4):
        n = normal[i][t]
        b = (n * (p * ONE - base[i][t])).sum(-1)
        at.append(b)
        b, a = b + lex[i][t], n[:, 0] * ONE
        m = a.abs().clamp_min(1)
        js = torch.where(a > 0, torch.maximum(js, torch.div(-b, m, rounding_mode="floor") + 1), js)
        je = torch.where(a < 0, torch.minimum(je, -torch.div(-b, m, rounding_mode="floor") - 1), je)
        je = torch.where((a == 0) & (b <= 0), -1, je)
    row, j = _spread((je - js + 1).clamp_min(0))
    j, t = j + js[row], t[row]
    p = p[row]
    p[:, 0] += j
    bary = [(at[i][row] + normal[i][t, 0] * ONE * j).double() / d[t].abs() for i in (1, 2, 3)]
    return t, p, bary


def _corners(q, dims):
    """Padded corner indices (one border voxel on each side) and fractions of points q [n][3]."""
    k = q.floor()
    f = q - k
    k = k.long() + 1
    ax = [(k[:, a].clamp(0, dims[a] + 1), (k[:, a] + 1).clamp(0, dims[a] + 1)) for a in range(3)]
    px, pxy = dims[0] + 2, (dims[0] + 2) * (dims[1] + 2)
    return [ax[2][z] * pxy + ax[1][y] * px + ax[0][x] for z in (0, 1) for y in (0, 1) for x in (0, 1)], f


def _lerp(v, f):
    x = [v[2 * i] + f[:, 0] * (v[2 * i + 1] - v[2 * i]) for i in range(4)]
    y = [x[0] + f[:, 1] * (x[1] - x[0]), x[2] + f[:, 1] * (x[3] - x[2])]
    return y[0] + f[:, 2] * (y[1] - y[0])


def _image_at(img, q, dims):
    """Trilinear value (zero outside) and whether a supported corner is positive."""
    idx, f = _corners(q, dims)
    v = [img[i] for i in idx]
    on = f > 0
    fg = torch.zeros_like(on[:, 0])
    for i, x in enumerate(v):
        ok = x > 0
        for a, bit in ((0, i & 1), (1, i & 2), (2, i & 4)):
            ok = ok & on[:, a] if bit else ok
        fg |= ok
    return torch.where(fg, _lerp(v, f), 0.0), fg


def _pair_term(a, fa, b, fb):
    return torch.where(fa & fb, (a - b).square(), (fa != fb).double())


class _Exact:
    """The definitions on one problem, in 64 bits."""

    def __init__(self, c, r):
        self.dims = (c["nx"], c["ny"], c["nz"])
        pad = torch.nn.functional.pad
        self.plain = _stored(r, c)
        self.img = [pad(v, (1,) * 6).reshape(-1) for v in self.plain]
        self.tets = torch.tensor(r["tets"].astype(np.int64), device=DEV)
        self.ref = torch.sign(_det(self.fix(torch.tensor(r["points"], device=DEV))[self.tets]))
        self.el = torch.tensor(r["elasticity"], device=DEV).double()
        self.radius = float(np.float32(r["radius"]))
        z, y, x = torch.meshgrid(*(torch.arange(n, device=DEV, dtype=torch.float64) for n in self.dims[::-1]),
                                 indexing="ij")
        self.maps, self.band, self.near, self.weight = [], [], [], []
        for sets in r["sets"]:
            total, vols = sum(len(s) for s in sets), []
            for s in sets:
                best = torch.full(x.shape, math.inf, device=DEV, dtype=torch.float64)
                for px, py, pz in (self.fix(torch.tensor(s)).double() / ONE).tolist():
                    best = torch.minimum(best, (x - px).square() + (y - py).square() + (z - pz).square())
                vols.append(best.sqrt().float())
            self.weight.append([len(s) / total for s in sets])
            v = torch.stack(vols)
            edge = pad(v[None], (1,) * 6, mode="replicate")[0].double()
            self.maps.append(edge.reshape(len(vols), -1))
            self.band.append(v.reshape(len(vols), -1).double() < self.radius)
            low = -torch.nn.functional.max_pool3d(-edge.amin(0)[None, None], 3, 1, 1)
            self.near.append(low.reshape(-1) < self.radius)

    @staticmethod
    def fix(x):
        return torch.round(x.double() * ONE).long()

    def verts(self, pts, cand, tet):
        """Fixed-point vertices [m][2][4][3] of (candidate, tet) pairs."""
        v = self.tets[tet]
        rows = pts.transpose(2, 3)                      # [pop][mesh][point][axis]
        return self.fix(torch.stack([rows[cand[:, None], m, v] for m in range(2)], 1))

    def guidance(self, d, t, q, dist):
        """Per set: the tets and terms of samples whose own distance dist(set) is inside the band."""
        idx, f = _corners(torch.minimum(q.clamp_min(0), torch.tensor(self.dims, device=DEV) - 1.0), self.dims)
        for s, w in enumerate(self.weight[d]):
            dn = dist(s)
            dq = _lerp([self.maps[1 - d][s][i] for i in idx], f)
            term = w * (self.radius - dn) / self.radius * (dn - dq).square()
            yield t, torch.where(dn < self.radius, term, 0.0)

    def centres(self, d, own, oth):
        """Sums of h and guidance and the counts over the voxel centres of own."""
        t, p, bary = _voxels(own, self.dims)
        o = oth.double() / ONE
        q = o[t, 0]
        for i in range(3):
            q = q + bary[i][:, None] * (o[t, i + 1] - o[t, 0])
        # a point on a grid plane (where both meshes share a coordinate) carries no weight beyond it
        q = torch.where((q - q.round()).abs() < 1e-9, q.round(), q)
        h = torch.zeros(len(own), device=DEV, dtype=torch.float64)
        g, n = torch.zeros_like(h), torch.zeros(len(own), device=DEV, dtype=torch.long)
        nx, ny, _ = self.dims
        a = self.img[d][((p[:, 2] + 1) * (ny + 2) + p[:, 1] + 1) * (nx + 2) + p[:, 0] + 1]
        h.index_add_(0, t, _pair_term(a, a > 0, *_image_at(self.img[1 - d], q, self.dims)))
        n.index_add_(0, t, torch.ones_like(t))
        flat = (p[:, 2] * ny + p[:, 1]) * nx + p[:, 0]
        k = self.band[d].any(0)[flat].nonzero()[:, 0]
        own_at = ((p[k, 2] + 1) * (ny + 2) + p[k, 1] + 1) * (nx + 2) + p[k, 0] + 1
        for u, term in self.guidance(d, t[k], q[k], lambda s: self.maps[d][s][own_at]):
            g.index_add_(0, u, term)
        return h, g, n

    def sobol(self, d, own, oth, rate):
        """The same over the random points of the sampling estimator (seed 7)."""
        m = len(own)
        count = torch.floor(_det(own).abs().double() * (rate / 6442450944.0) + 0.5).long().clamp_max(1 << 20)
        hsh = _mix(torch.full((m,), _signed(7 + GOLDEN * (d + 1)), device=DEV))
        for i in range(12):
            hsh = _mix(hsh + _signed(GOLDEN) + (own.reshape(m, 12)[:, i] & 0xffffffff))
        words = [_mix(hsh + _signed(GOLDEN)), _mix(hsh + _signed(2 * GOLDEN))]
        shift = [words[0] & 0xffffffff, _lshr(words[0], 32), words[1] & 0xffffffff, _lshr(words[1], 32)]
        t, n = _spread(count)
        e = []
        for j in range(4):
            u = shift[j][t]
            for b in range(20):
                u = u ^ (-((n >> b) & 1) & DIRECTIONS[j][b])
            e.append(-torch.log((2 * (u >> 9) + 1).double() * 2.0 ** -24))
        total = sum(e)
        pq = []
        for v in (own.double() / ONE, oth.double() / ONE):
            x = v[t, 0]
            for i in range(3):
                x = x + (e[i + 1] / total)[:, None] * (v[t, i + 1] - v[t, 0])
            pq.append(x)
        p, q = pq
        h = torch.zeros(m, device=DEV, dtype=torch.float64)
        g = torch.zeros_like(h)
        h.index_add_(0, t, _pair_term(*_image_at(self.img[d], p, self.dims), *_image_at(self.img[1 - d], q, self.dims)))
        p = torch.minimum(p.clamp_min(0), torch.tensor(self.dims, device=DEV) - 1.0)
        k = self.near[d][_corners(p, self.dims)[0][0]].nonzero()[:, 0]
        idx, f = _corners(p[k], self.dims)
        for u, term in self.guidance(d, t[k], q[k], lambda s: _lerp([self.maps[d][s][i] for i in idx], f)):
            g.index_add_(0, u, term)
        return h, g, count

    def items(self, pts, cand, tet, sums=None, chunk=100000):
        """Records of (candidate, tet) items: h, g, n, vol [m][2] and mag [m]."""
        sums = sums or self.centres
        out = dict(h=[], g=[], n=[], vol=[], mag=[], viol=[])
        for at in range(0, len(tet), chunk):
            k, t = cand[at:at + chunk], tet[at:at + chunk]
            v = self.verts(pts, k, t)
            part = [sums(d, v[:, d], v[:, 1 - d]) for d in range(2)]
            for name, i in (("h", 0), ("g", 1), ("n", 2)):
                out[name].append(torch.stack([part[0][i], part[1][i]], 1))
            det = torch.stack([_det(v[:, 0]), _det(v[:, 1])], 1)
            viol = torch.sign(det) != self.ref[t][:, None]
            out["viol"].append(viol)
            out["vol"].append(torch.where(viol, det.abs().double() / 6442450944.0, 0.0))
            x = v.double() / ONE
            ends = torch.cat([x, x.mean(2, keepdim=True)], 2)
            ends = torch.stack([(ends[:, :, i] - ends[:, :, j]).norm(dim=-1) for j in range(5) for i in range(j)], -1)
            out["mag"].append(self.el[t] * (ends[:, 0] - ends[:, 1]).square().sum(-1))
        return {k: torch.cat(v) for k, v in out.items()}

    def population(self, pts, sums=None):
        """Records of every (candidate, tet), [pop][n_tets] first."""
        pop, m = len(pts), len(self.tets)
        at = torch.arange(m * pop, device=DEV)
        rec = self.items(pts, at % pop, torch.div(at, pop, rounding_mode="floor"), sums)
        return {k: v.reshape(m, pop, *v.shape[1:]).transpose(0, 1) for k, v in rec.items()}

    def objectives(self, h, mag, g, n, vol):
        obj = torch.stack([h / n, mag / (10.0 * len(self.tets)), g / n], -1)
        return dict(obj=obj, severity=vol, flags=None, counts=None)


GOLDEN = 0x9e3779b97f4a7c15


def _signed(x):
    x &= (1 << 64) - 1
    return x - (1 << 64) if x >> 63 else x


def _lshr(x, k):
    return (x >> k) & ((1 << (64 - k)) - 1)


def _mix(z):
    z = (z ^ _lshr(z, 30)) * _signed(0xbf58476d1ce4e5b9)
    z = (z ^ _lshr(z, 27)) * _signed(0x94d049bb133111eb)
    return z ^ _lshr(z, 31)


def _directions():
    """Direction numbers of four Sobol dimensions: 1, x + 1, x^2 + x + 1, x^3 + x + 1."""
    out = [[0x80000000 >> b for b in range(32)]]
    for poly, deg, first in ((0x3, 1, (1,)), (0x7, 2, (1, 3)), (0xb, 3, (1, 3, 1))):
        m = list(first)
        for k in range(deg, 32):
            x = m[k - deg]
            for i in range(1, deg + 1):
                if (poly >> (deg - i)) & 1:
                    x ^= m[k - i] << i
            m.append(x)
        out.append([(m[b] << (31 - b)) & 0xffffffff for b in range(32)])
    return out


DIRECTIONS = _directions()


def _exact_evaluate(c, r):
    e = _Exact(c, r)
    sums = None if c["kind"] == "evaluate" else lambda d, a, b: e.sobol(d, a, b, c["rate"])
    rec = e.population(r["pts"], sums)
    out = e.objectives(rec["h"].sum((1, 2)), rec["mag"].sum(1), rec["g"].sum((1, 2)), rec["n"].sum((1, 2)),
                       rec["vol"].sum((1, 2)))
    if c.get("cache"):
        mag = torch.stack([rec["mag"], torch.zeros_like(rec["mag"])], -1)
        out.update(rec_h=rec["h"], rec_g=rec["g"], rec_n=None, rec_mag=mag, rec_vol=rec["vol"], rec_bits=None)
    return out


def _exact_samples(c, r):
    """New coordinates of the mixing case: normal distributions per (cluster, element)."""
    el = torch.tensor(r["elements"].astype(np.int64), device=DEV)[r["eg"].long()]
    x = r["pts"].double().permute(0, 3, 1, 2)                       # [pop][point][mesh][axis]
    new = x[r["ep"].long()[:, None], el].reshape(len(el), 12)       # the parents' values
    z = r["z"].double().reshape(len(el), 12)
    fixed = torch.tensor(r["fixed"], device=DEV)
    off = r["off"].tolist()
    for k in range(c["clusters"]):
        mem = x[r["members"][off[k]:off[k + 1]].long()]
        for e in torch.unique(r["eg"]).tolist():
            pair = r["elements"][e].astype(np.int64)
            free = (~fixed[torch.tensor(pair, device=DEV)])[:, None, :].expand(2, 2, 3).reshape(12).nonzero()[:, 0]
            v = mem[:, torch.tensor(pair, device=DEV)].reshape(len(mem), 12)[:, free]
            mean = v.mean(0)
            cov = (v - mean).T @ (v - mean) / len(v)
            if len(v) <= len(free):
                return None          # a singular covariance: no factor to compare with
            low = torch.linalg.cholesky(cov)
            at = ((r["eg"] == e) & (r["ec"] == k)).nonzero()[:, 0]
            new[at[:, None], free] = mean + z[at[:, None], free] @ low.T
    return new.reshape(-1, 2, 3)


def _exact_partial(c, r):
    if c["kind"] == "mixing":
        new64 = _exact_samples(c, r)
        if new64 is None:
            return None
        new, groups = new64.float(), [g.astype(np.int64) for g in r["elements"]]
    else:
        off, gp = r["groups"]
        new64, new, groups = None, r["new"], [gp[a:b].astype(np.int64) for a, b in zip(off, off[1:])]
    e = _Exact(c, r)
    parent = e.population(r["pts"])
    total = {k: v.sum(tuple(range(1, v.dim()))) for k, v in parent.items()}
    ep, eg = r["ep"].long(), r["eg"].long()
    sizes = torch.tensor([len(g) for g in groups], device=DEV)
    first = sizes[eg].cumsum(0) - sizes[eg]
    out = {k: torch.empty(len(ep), device=DEV, dtype=torch.float64) for k in ("h", "mag", "g", "n", "vol")}
    for g in torch.unique(eg).tolist():
        at = (eg == g).nonzero()[:, 0]
        pts = torch.tensor(groups[g], device=DEV)
        child = r["pts"][ep[at]].clone()
        rows = new[first[at][:, None] + torch.arange(len(pts), device=DEV)]
        child[:, :, :, pts] = rows.permute(0, 2, 3, 1)
        dep = torch.isin(e.tets, pts).any(1).nonzero()[:, 0]
        k = torch.arange(len(at) * len(dep), device=DEV)
        rec = e.items(child, torch.div(k, len(dep), rounding_mode="floor"), dep[k % len(dep)])
        for name in out:
            fresh = rec[name].reshape(len(at), -1).sum(1)
            old = parent[name][ep[at]][:, dep].reshape(len(at), -1).sum(1)
            out[name][at] = (total[name][ep[at]] + (fresh - old)).double()
    res = e.objectives(out["h"], out["mag"], out["g"], out["n"], out["vol"])
    return res if new64 is None else dict(res, new=new64)


def _exact_dvf(c, r):
    e = _Exact(c, r)
    tet = torch.arange(len(e.tets), device=DEV)
    v = e.verts(r["pts"], torch.zeros_like(tet), tet)
    nx, ny, nz = e.dims
    out = dict(cover=None)
    for d, name in ((0, "fwd"), (1, "inv")):
        t, p, bary = _voxels(v[:, d], e.dims)
        o = v[:, 1 - d].double() / ONE
        q = o[t, 0]
        for i in range(3):
            q = q + bary[i][:, None] * (o[t, i + 1] - o[t, 0])
        flat = (p[:, 2] * ny + p[:, 1]) * nx + p[:, 0]
        owner = torch.full((nx * ny * nz,), len(tet), device=DEV).scatter_reduce(0, flat, t, "amin")
        k = (owner[flat] == t).nonzero()[:, 0]
        field = torch.zeros((nx * ny * nz, 3), device=DEV, dtype=torch.float64)
        field[flat[k]] = q[k] - p[k]
        out[name] = field.reshape(nz, ny, nx, 3)
    return out


def _network(params):
    cut = np.cumsum([HIDDEN * N_FEATURES, HIDDEN, HIDDEN * HIDDEN, HIDDEN, HIDDEN])
    w1, b1, w2, b2, w3, b3 = (torch.tensor(p, device=DEV).double() for p in np.split(params, cut))
    return w1.reshape(HIDDEN, N_FEATURES), b1, w2.reshape(HIDDEN, HIDDEN), b2, w3, b3


def _predict(net, x):
    w1, b1, w2, b2, w3, b3 = net
    return torch.relu(torch.relu(x @ w1.T + b1) @ w2.T + b2) @ w3 + b3


def _exact_gradients(r):
    net = [p.requires_grad_() for p in _network(r["params"])]
    loss = (_predict(net, r["feats"].double()) - r["targets"].double()).square().mean()
    grads = torch.autograd.grad(loss, net)
    return dict(grads=torch.cat([g.reshape(-1) for g in grads]), loss=loss.detach().reshape(1))


def _halton(j, base):
    v, f = 0.0, 1.0 / base
    while j:
        v += f * (j % base)
        j, f = j // base, f / base
    return v


def _exact_prescreen(c, r):
    e = _Exact(c, r)
    parents = e.population(r["parents"])
    term = parents["h"].sum(2) / parents["n"].sum(2).clamp_min(1)
    scale = (e.plain[0] - e.plain[1]).square().mean()
    # statistics of each reference tet's voxels
    ref = e.fix(torch.tensor(r["points"], device=DEV))[e.tets]
    t, p, _ = _voxels(ref, e.dims)
    a, b = (im[p[:, 2], p[:, 1], p[:, 0]] for im in e.plain)
    cols = torch.stack([torch.ones_like(a), a, a * a, a > 0, b, b * b, b > 0, (a - b).square()], 1)
    s = torch.zeros((len(e.tets), 8), device=DEV, dtype=torch.float64).index_add_(0, t, cols)
    s = s / s[:, :1].clamp_min(1)
    dev = [(s[:, k + 1] - s[:, k].square()).clamp_min(0).sqrt() for k in (1, 4)]
    stats = torch.stack([s[:, 1], dev[0], s[:, 3], s[:, 4], dev[1], s[:, 6], s[:, 7] / scale], 1)
    # the point sets behind the estimated changes: vertices, edge midpoints, interior points
    sets = [np.eye(4), np.array([(np.eye(4)[i] + np.eye(4)[j]) / 2 for i in range(4) for j in range(i)])]
    u = np.sort([[_halton(j, b) for b in (2, 3, 5)] for j in range(1, 17)], axis=1)
    sets.append(np.stack([u[:, 0], u[:, 1] - u[:, 0], u[:, 2] - u[:, 1], 1 - u[:, 2]], 1))
    bary = torch.tensor(np.concatenate(sets), device=DEV)
    top = torch.tensor(e.dims, device=DEV) - 1.0

    def means(v):                                     # v [m][2][n_tets][4][3]
        x = [torch.minimum((bary @ v[:, k]).clamp_min(0), top).reshape(-1, 3) for k in range(2)]
        val = []
        for k in range(2):
            idx, f = _corners(x[k], e.dims)
            val.append(_lerp([e.img[k][i] for i in idx], f))
        h = (val[0] - val[1]).square().reshape(len(v), -1, 26)
        return torch.stack([h[..., :4].mean(-1), h[..., 4:10].mean(-1), h[..., 10:].mean(-1)], -1)

    def geometry(pts):
        return pts.double().transpose(2, 3)[:, :, e.tets]

    net = _network(r["params"])
    base = torch.cat([means(geometry(r["parents"][k:k + 32])) for k in range(0, c["pop"], 32)])
    scores = []
    for k in range(0, len(r["pts"]), 32):
        v, of = geometry(r["pts"][k:k + 32]), r["of"][k:k + 32].long()
        moves = (v[:, 1] - geometry(r["parents"][of])[:, 1]).flatten(2) * 2
        x = torch.cat([moves, (means(v) - base[of]) / scale, stats.expand(len(v), -1, -1),
                       (term[of] / scale)[..., None]], -1)
        edge = v[..., 1:, :] - v[..., :1, :]
        w = ((_cross(edge[..., 0, :], edge[..., 1, :]) * edge[..., 2, :]).sum(-1).abs() / 6).sum(1)
        scores.append((w * (term[of] + scale * _predict(net, x))).sum(1) / w.sum(1))
    return torch.cat(scores)


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "archive":
        return None                                   # copies of inputs and whole numbers
    r = _inputs(c, seed)
    if kind == "gradients":
        return _exact_gradients(r)
    if kind in ("evaluate", "sobol"):
        return _exact_evaluate(c, r)
    if kind in ("partial", "mixing"):
        return _exact_partial(c, r)
    return _exact_dvf(c, r) if kind == "dvf" else _exact_prescreen(c, r)
