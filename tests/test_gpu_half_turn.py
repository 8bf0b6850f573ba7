"""2D grains whose proper rotation turns the crystal over (a half turn about an
in-plane axis: R_zz = -1).  The cubic form does not change under a half turn
about a crystal axis, so such a grain is the one of the same angle about z: in
FP64 every variant matches the oracle, which applies the full rotation, and in
FP32 the two ways to write the grain give the same bits."""
import numpy as np
import pytest

import oracle
from paper_2110_12448_amd import pfiso
from paper_2110_12448_amd import workloads as wl

pytestmark = pytest.mark.gpu

_VARIANTS = {
    "approx-shells": dict(),
    "full-shells": dict(wl.SCHEMES_2D["S21"]),
    "full-two-point": dict(wl.SCHEMES_2D["S10"]),
    "approx-two-point": dict(scheme="std", two_point=1),
}


def _turned(deg):
    return wl.rotation_2d(deg) @ np.diag([1.0, -1.0, -1.0])


def _problem(variant, rots):
    nx, ny = 70, 48
    grain = (np.arange(nx)[None, :] * len(rots) // nx).astype(np.int8)
    return wl.problem(2, (nx, ny), eps4=0.05, rot=np.stack(rots),
                      grain=np.ascontiguousarray(np.broadcast_to(grain, (ny, nx))),
                      seed=3, seed_radius=12.0, **_VARIANTS[variant])


def _run(pr, precision, steps):
    s = pfiso.Solver(pr, precision=precision)
    s.step(steps)
    _, U, psi, _ = s.read_fields()
    s.close()
    return psi, U


@pytest.mark.parametrize("grains", [1, 2])
@pytest.mark.parametrize("variant", sorted(_VARIANTS))
def test_turned_over_grain(variant, grains):
    degs = (17.0, 31.0)[:grains]
    pr = _problem(variant, [_turned(a) for a in degs])
    psi, U = _run(pr, pfiso.PF_F64, 40)
    opsi, oU, _ = oracle.step(oracle.Params.from_problem(pr), pr["psi0"], pr["U0"], pr["grain"], 40)
    # the bound of the FP64 parity tests: only the order of summation differs
    assert np.max(np.abs(np.tanh(psi / np.sqrt(2.0)) - np.tanh(opsi / np.sqrt(2.0)))) < 1e-10
    assert np.max(np.abs(U - oU)) < 1e-10
    z = _problem(variant, [wl.rotation_2d(a) for a in degs])
    for a, b in zip(_run(pr, pfiso.PF_F32, 40), _run(z, pfiso.PF_F32, 40)):
        assert np.array_equal(a, b)
