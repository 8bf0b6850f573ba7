"""Batch members whose geometry a caller set, by rows, by waves per SIMD or by the
autotuner, keep it (at least 8 rows); only members that nobody tuned take the
longer segments of a large batch."""
import pytest

from paper_2110_12448_amd import pfiso
from paper_2110_12448_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("how", ["nobody", "rows", "waves", "default-waves", "autotuner"])
@pytest.mark.parametrize("members,rows", [(2, 8), (8, 20), (20, 32)])  # 16, 64, 160 rows per SIMD
def test_members_keep_their_geometry(members, rows, how):
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    nx, ny = 61, 4100 * cus // 256
    pr = wl.problem(2, (nx, ny), noise=0.0)
    ss = [pfiso.Solver(pr, precision=pfiso.PF_F32) for _ in range(members)]
    b = pfiso.Batch(ss)
    segs = [-(-ny // rows)] * members
    assert b.launch_waves() == 2 * sum(segs)
    default = ss[0].geometry()[0]
    if how != "nobody":
        s = ss[1]
        if how == "autotuner":
            s.autotune(1)
        else:
            s.tune({"rows": 11, "waves": -1, "default-waves": default}[how])
        k = s.geometry()[0]
        alone = -(-ny // k) if k > 0 else -k * 4 * cus // 2
        segs[1] = -(-ny // max(8, -(-ny // alone)))
    b.step(2)
    assert b.launch_waves() == 2 * sum(segs)
    b.close()
    for s in ss:
        s.close()
