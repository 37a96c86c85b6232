"""GPU tests of the selection and of the archive update at the sizes where
their kernels change shape: populations around powers of two (several threads
a solution, one, a full block), selections from one solution to all, several
clusters a pass and one; archives of one slot, around 1,024 slots (the slots
of a thread) and at the limit of 4,096 candidates, with and without thinning.
Everything equals the reference exactly."""
import numpy as np
import pytest

from test_gpu_archive import grid_offers, plane_offers, run_sequence
from test_gpu_select import check

pytestmark = pytest.mark.gpu

pytest.importorskip("torch")


@pytest.mark.parametrize("n,size,k", [(1, 1, 1), (2, 2, 5), (63, 20, 3), (64, 64, 64), (65, 1, 4), (511, 200, 1),
                                      (512, 179, 10), (513, 513, 7), (1000, 512, 9), (1024, 1024, 3)])
def test_selection_sizes(n, size, k):
    rs = np.random.default_rng(n)
    for grid in (4, 1000):                      # many equal vectors, then few
        obj = rs.integers(0, grid, (n, 3)).astype(np.float32)
        fl = rs.choice(np.array([0, 0, 0, 0, 0, 0, 1, 2, 4], np.uint8), n)
        sv = np.where(fl & 3, rs.integers(1, 4, n), 0).astype(np.float32)
        check(obj, fl, sv, size, k, gmax=None if grid == 4 else 0.8 * grid)


@pytest.mark.parametrize("cap,offers", [(1, 7), (2, 300), (64, 64), (1023, 1024), (1024, 1), (1025, 900),
                                        (3072, 1024), (4095, 1)])
def test_archive_sizes(cap, offers):
    rs = np.random.default_rng(cap)
    batches = [plane_offers(rs, offers), grid_offers(rs, offers, 6), plane_offers(rs, offers)]
    if cap == 3072:                             # fill it, so that the last batch has to be thinned
        batches = [plane_offers(rs, offers) for _ in range(4)]
    _, ref = run_sequence(cap, batches, [None] * len(batches))
    assert len(ref.members()) <= cap
