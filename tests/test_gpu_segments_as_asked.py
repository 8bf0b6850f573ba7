"""2D launch geometry: a strip gets the segments that were asked for, also where
their number is no multiple of the four that share a workgroup, and the fields
are bit for bit those of independent segments."""
import numpy as np
import pytest

from paper_2110_12448_amd import pfiso
from paper_2110_12448_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _run(pr, precision, tune, steps=9):
    s = pfiso.Solver(pr, precision=precision)
    s.tune(tune)
    waves = s.launch_waves()
    s.step(steps)
    _, U, psi, _ = s.read_fields()
    s.close()
    return waves, psi, U


# 1 to 3 segments above the groups of four, none, and fewer than four segments;
# wide lattices where a few waves per SIMD leave 1 to 7 segments a strip
@pytest.mark.parametrize("nx,ny,tunes", [
    (61, 57, (256, 29, 20, 14, 12, 9, 8, 7, 5, 4)),
    (130, 100, (50, 34, 25, 20, 17, 15, 13)),
    (9000, 21, (-1, -2, -3)),
    (40000, 21, (-1, -2, -4)),
])
@pytest.mark.parametrize("variant", ["approx", "S21-frame"])
def test_segments_as_asked(nx, ny, tunes, variant):
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    kw = {} if variant == "approx" else dict(wl.SCHEMES_2D["S21"], frame=1, shift_row=6)
    pr = wl.problem(2, (nx, ny), alpha0_deg=17.0, seed=4, seed_radius=5.0, **kw)
    strips = -(-nx // 60)
    ref = _run(pr, pfiso.PF_F32, -64)
    for tune in tunes:
        waves, psi, U = _run(pr, pfiso.PF_F32, tune)
        segs = -(-ny // tune) if tune > 0 else max(1, min(ny, -tune * 4 * cus // strips))
        assert waves == strips * segs, tune
        assert np.array_equal(psi, ref[1]) and np.array_equal(U, ref[2]), tune
