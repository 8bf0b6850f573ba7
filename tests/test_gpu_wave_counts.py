"""The waves that serving admits by are those the library launches: solves on
their own, batches of every size, and a served batch under a cap."""
import pytest

from paper_2110_12448_amd import pfiso, serve
from paper_2110_12448_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _cus():
    import torch
    return torch.cuda.get_device_properties(0).multi_processor_count


@pytest.mark.parametrize("precision", [pfiso.PF_F32, pfiso.PF_F64])
@pytest.mark.parametrize("shape", [(64, 64), (300, 57), (1024, 1024), (1024, 2048), (9000, 21),
                                   (24, 32, 17), (33, 29, 6), (97, 131, 90), (128, 128, 128)])
def test_solve_on_its_own(shape, precision):
    pr = wl.problem(len(shape), shape, noise=0.0)
    s = pfiso.Solver(pr, precision=precision)
    assert serve.estimated_waves(pr, cus=_cus(), precision=precision) == s.launch_waves()
    s.close()


@pytest.mark.parametrize("members", [1, 6, 24])   # 8 to 200 strip rows per SIMD
def test_batch(members):
    prs = [wl.problem(2, (512 + 61 * (i % 3), 900 - 37 * (i % 4)), noise=0.0)
           for i in range(members)]
    ss = [pfiso.Solver(pr, precision=pfiso.PF_F32) for pr in prs]
    b = pfiso.Batch(ss)
    load = sum(serve.strip_rows(pr) for pr in prs) / (4.0 * _cus())
    want = sum(serve.estimated_waves(pr, batched=True, cus=_cus(), load=load) for pr in prs)
    assert want == b.launch_waves()
    b.close()
    for s in ss:
        s.close()


def test_admission_counts_the_rows_of_the_whole_batch(monkeypatch):
    """24 solves of 512^2 under a cap of 8200 waves: 13 of them run 7488 waves in
    8-row segments, 14 and more 234 each in 20-row ones, so all 24 are admitted
    (8-row counts would stop at 15)."""
    if _cus() != 256:
        pytest.skip("the counts are those of 256 compute units")
    pr = wl.problem(2, (512, 512), noise=0.0)
    sizes = []

    class Batch(pfiso.Batch):
        def __init__(self, solvers, graph_steps=0):
            super().__init__(solvers, graph_steps=graph_steps)
            sizes.append((len(self.solvers), self.launch_waves()))

    monkeypatch.setattr(pfiso, "Batch", Batch)
    srv = serve.Server(8 << 30, max_waves=8200)
    res = srv.run([serve.Request(i, 0.0, pr, 4) for i in range(24)], realtime=False)
    assert len(res) == 24 and sizes == [(24, 24 * 9 * 26)]
