"""The FP64 kernels' tanh, through the reduction on caller-held fields: phi of
uniform fields from the solid fraction, and its relative accuracy near 0 from
the height of a phi = 0 crossing.  Reference: 80-bit long doubles."""
import ctypes as C

import numpy as np
import pytest

from paper_2110_12448_amd import pfiso

pytestmark = pytest.mark.gpu


def _tip(psi, U):
    import torch
    t = pfiso.pf_tip()
    a, b = (torch.as_tensor(f, device="cuda:0") for f in (psi, U))
    st = torch.cuda.current_stream().cuda_stream
    rc = pfiso.load().pf_tip_fields(C.c_void_p(a.data_ptr()), C.c_void_p(b.data_ptr()),
                                    pfiso.PF_F64, psi.shape[1], psi.shape[0], 1, 1.0, 0,
                                    C.c_void_p(st), C.byref(t))
    return rc, t


# edges of the argument reduction (2x = (n + 1/2) ln 2), of the rounding to 1 and of the clamp
_ARGS = [0.0, 1e-300, 1e-9, 0.1, 0.173286795139986, 0.17328679513998635, 0.52, 0.9, 3.0, 18.36,
         18.541728866794482, 18.956948792718986, 19.0, 19.1, 25.0, 39.999, 40.1, 1e6, 1e300]


@pytest.mark.parametrize("x", _ARGS + [-v for v in _ARGS])
def test_phi_of_a_uniform_field(x):
    psi = np.full((4, 64), x * np.sqrt(2.0))
    rc, t = _tip(psi, np.zeros_like(psi))
    assert rc == pfiso.PF_OK
    # the kernel's argument is psi times the rounded 1/sqrt 2
    arg = np.longdouble(psi[0, 0] * 0.70710678118654752)
    want = (1 + np.tanh(arg)) / 2
    # phi to 1 ulp of 1, the sum 1 + phi and the mean to half an ulp each
    assert abs(np.longdouble(t.solid_fraction) - want) <= 3e-16


@pytest.mark.parametrize("a,b", [(1e-12, 3e-12), (0.02, 0.3), (0.24, 0.26), (2e-200, 1e-200)])
def test_crossing_height(a, b):
    psi = np.empty((4, 64))
    psi[:2], psi[2:] = a, -b
    rc, t = _tip(psi, np.zeros_like(psi))
    assert rc == pfiso.PF_OK and t.found == 1
    f0, f1 = (np.tanh(np.longdouble(v * 0.70710678118654752)) for v in (a, -b))
    assert abs(np.longdouble(t.y_frame) - (1 + f0 / (f0 - f1))) <= 1e-15


@pytest.mark.parametrize("v", [np.nan, np.inf, -np.inf])
def test_non_finite_values_are_reported(v):
    psi = np.zeros((8, 64))
    psi[3, 7] = v
    rc, t = _tip(psi, np.zeros_like(psi))
    assert rc == pfiso.PF_ERR_NONFINITE and t.nonfinite == 1
