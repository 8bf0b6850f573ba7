"""pf_create's checks of the initial fields on lattices that are split over host
threads: one bad value anywhere is found, also at the ends of a thread's piece
and in the last cell (CPU: the checks run before a device is touched)."""
import numpy as np
import pytest

from paper_2110_12448_amd import pfiso
from paper_2110_12448_amd import workloads as wl
from test_abi import _create

NX, NY = 1100, 1000                     # 4 pieces of at least 2^18 cells
N = NX * NY


@pytest.fixture(scope="module")
def problem():
    return wl.problem(2, (NX, NY), noise=0.0)


def _cells():
    at = {0, N - 1}
    for k in (2, 3, 4):                 # pieces, by the hardware threads there are
        for i in range(1, k):
            at |= {N * i // k - 1, N * i // k}
    return sorted(at)


@pytest.mark.parametrize("precision", [pfiso.PF_F32, pfiso.PF_F64])
@pytest.mark.parametrize("field", ["psi0", "U0"])
@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
def test_nonfinite_cell_is_found(problem, precision, field, value):
    f = problem[field].copy()
    pr = dict(problem, **{field: f})
    for c in _cells():
        keep, f.flat[c] = f.flat[c], value
        rc, _, _ = _create(pr, precision)
        f.flat[c] = keep
        assert rc == pfiso.PF_ERR_NONFINITE, c


@pytest.mark.parametrize("value", [2, -1, 127, -128])
def test_grain_index_out_of_range_is_found(problem, value):
    g = np.zeros((NY, NX), dtype=np.int8)
    pr = dict(problem, grain=g, rot=np.stack([wl.rotation_2d(a) for a in (0.0, 20.0)]))
    for c in _cells():
        g.flat[c] = value
        rc, msg, _ = _create(pr)
        g.flat[c] = 0
        assert rc == pfiso.PF_ERR_ARG and "grain" in msg, c
