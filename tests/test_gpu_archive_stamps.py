"""GPU test of the archive update on members that a caller stored with equal
insertion stamps (two archives put together, a restarted counter): equal stamps
are ordered by slot, also where the boxes are thinned."""
import numpy as np
import pytest

from oracle import archive as ar
from test_gpu_archive import check, dev, plane_offers

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2303_04873_amd as morea  # noqa: E402


@pytest.mark.parametrize("stamps", ["all equal", "pairs", "restarted counter"])
@pytest.mark.parametrize("cap,offers", [(40, 30), (1500, 700)])
def test_equal_stamps(cap, offers, stamps):
    rs = np.random.default_rng(cap)
    a, ref = morea.Archive(cap), ar.Archive(cap)
    obj, _, _ = plane_offers(rs, cap)
    ref.obj[:] = obj
    order = rs.permutation(cap)
    ref.stamp[:] = {"all equal": order * 0 + 3, "pairs": order // 2, "restarted counter": order}[stamps]
    ref.next_stamp = 0 if stamps == "restarted counter" else cap
    a.obj.copy_(dev(ref.obj))
    a.stamp.copy_(dev(ref.stamp.astype(np.int32)))
    a.state.copy_(dev(np.array([cap, ref.next_stamp, 0, 0], np.int32)))
    for k in range(3):
        obj, flags, sev = plane_offers(rs, offers)
        ins, slot = a.update(dict(obj=dev(obj), flags=dev(flags), severity=dev(sev)))
        ins_ref, slot_ref = ar.update(ref, obj, flags, sev)
        assert ref.levels > 0
        check(a, ref, ins, slot, ins_ref, slot_ref, f"{stamps} {k}")
