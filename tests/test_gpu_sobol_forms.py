"""GPU test of the Sobol estimator's two forms (images staged in LDS for a
block of candidates, or read where they are): a candidate's outputs have the
same bits in both, alone (never staged) and in its population, whatever the
storage, also in a block that has waves to spare and beside candidates that
are invalid or partly outside; and in both forms points on grid planes leave
corners of weight 0 out of the foreground."""
import numpy as np
import pytest

import oracle
import synth
from parity import assert_parity, to_host
from test_gpu_sobol_paths import CASES, DIMS, TETS, WIDE, images

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2303_04873_amd as morea  # noqa: E402


def same_bits(out, k, one, what):
    for key in one:
        np.testing.assert_array_equal(out[key][k], one[key][0], err_msg=f"{what} {key}")


@pytest.mark.parametrize("storage", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("case", sorted(CASES))
def test_paths_in_both_forms(case, storage):
    """A block of 12 copies of each case beside the same candidate alone, which
    is compared with the oracle."""
    S, T, rate = CASES[case]
    rate = max(rate, 12.0)                      # 216 voxels: 12 candidates are staged from 408 samples
    img_s, img_t = images(5)
    rs = np.random.default_rng(6)
    sets = [[rs.uniform(1, 14, (9, 3)).astype(np.float32) for _ in range(2)] for _ in range(2)]
    args = (TETS, WIDE.astype(np.float32), np.ones(1, np.float32), sets[0], sets[1])
    prob = morea.Problem(DIMS, img_s, img_t, *args, radius=3.0, storage=storage, max_population=12)
    quant = [img_s, img_t] if storage == "f32" else [oracle.quantize(i, storage) for i in (img_s, img_t)]
    op = oracle.Problem(DIMS, quant[0], quant[1], *args, 3.0)
    cand = np.stack([np.asarray(S, np.float32).T, np.asarray(T, np.float32).T])[None]
    one = to_host(prob.eval_sobol(torch.from_numpy(np.ascontiguousarray(cand)).cuda(), rate=rate, seed=3))
    assert_parity(one, op.evaluate_sobol(cand, rate=rate, seed=3), what=case)
    out = to_host(prob.eval_sobol(torch.from_numpy(np.repeat(cand, 12, 0)).cuda(), rate=rate, seed=3))
    for k in range(12):
        same_bits(out, k, one, case)


@pytest.mark.parametrize("storage", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("pop,last", [(12, 12), (23, 11), (35, 11)])
def test_population_and_alone_give_the_same_bits(pop, last, storage):
    """Blocks of 12 candidates a tet; 23 and 35 leave a wave to spare in the
    last, which also holds an invalid candidate and one partly outside."""
    n, cells = 40, 4
    per = -(-pop // -(-pop // 12))
    assert per == 12 and pop - (pop - 1) // per * per == last
    pts, tets, fixed = synth.kuhn_grid((n, n, n), (cells, cells, cells))
    rs = np.random.default_rng(pop)
    img = [(rs.uniform(0, 1, (n, n, n)) * (rs.uniform(0, 1, (n, n, n)) > 0.3)).astype(np.float32) for _ in range(2)]
    sets = [[rs.uniform(4, n - 5, (40, 3)).astype(np.float32)] for _ in range(2)]
    prob = morea.Problem((n, n, n), img[0], img[1], tets, pts, np.ones(len(tets), np.float32), sets[0], sets[1],
                         radius=4.0, storage=storage, max_population=pop)
    cands = np.stack([np.stack([(pts + np.where(fixed, 0, rs.normal(0, 0.4, pts.shape))).T for _ in range(2)])
                      for _ in range(pop)]).astype(np.float32)
    cands[pop - 2, 0, 1, 20] = np.nan
    cands[pop - 4] += 1.5
    if pop > 12:
        cands[pop - 1, 1] += 0.75
    t = torch.from_numpy(np.ascontiguousarray(cands)).cuda()
    out = to_host(prob.eval_sobol(t, rate=4.0, seed=6))
    assert out["counts"][0].min() > 1e5
    for k in range(pop):
        same_bits(out, k, to_host(prob.eval_sobol(t[k:k + 1].contiguous(), rate=4.0, seed=6)), f"candidate {k}")
