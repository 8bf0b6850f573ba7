"""2D step: segments that share their junction rows inside a workgroup give
bit for bit the fields of independent segments (one row each), for every
variant, at the smallest shared segments and at uneven splits."""
import numpy as np
import pytest

from paper_2110_12448_amd import pfiso
from paper_2110_12448_amd import workloads as wl

pytestmark = pytest.mark.gpu

_NF = wl.NOFLUX
_VARIANTS = {
    "iso": dict(),
    "iso-noflux": dict(bc=(_NF, _NF, _NF)),
    "iso-periodic-y": dict(bc=(wl.PERIODIC, wl.PERIODIC, wl.PERIODIC), thermal="isothermal",
                           seed_shape="disc"),
    "frame": dict(frame=1),
    "S21": dict(wl.SCHEMES_2D["S21"], bc=(_NF, _NF, _NF)),
    "S21-frame": dict(wl.SCHEMES_2D["S21"], frame=1),
    "S10": dict(wl.SCHEMES_2D["S10"]),
    "approx-two-point": dict(scheme="std", two_point=1),
    "dynamic-grains": dict(dynamic_grains=1, frame=1),
}


def _problem(nx, ny, name):
    kw = dict(_VARIANTS[name])
    if name == "dynamic-grains":
        kw.update(rot=np.stack([wl.rotation_2d(a) for a in (0.0, 20.0, 40.0)]),
                  grain=(np.arange(nx)[None, :] * 3 // nx).astype(np.int8))
    if name == "iso-periodic-y":
        kw["y_front"] = (ny // 2) * 0.8      # the disc away from the seam
    if kw.get("frame"):
        kw["shift_row"] = max(1, min(ny - 2, 6))
    return wl.problem(2, (nx, ny), alpha0_deg=17.0, seed=4, seed_radius=5.0, **kw) \
        if "rot" not in kw else wl.problem(2, (nx, ny), seed=4, seed_radius=5.0, **kw)


def _run(pr, precision, rows, steps=8):
    s = pfiso.Solver(pr, precision=precision)
    s.tune(rows)
    s.step(steps)
    _, U, psi, grain = s.read_fields()
    s.close()
    return psi, U, grain


@pytest.mark.parametrize("precision", [pfiso.PF_F32, pfiso.PF_F64])
@pytest.mark.parametrize("name", sorted(_VARIANTS))
@pytest.mark.parametrize("nx,ny", [(31, 12), (61, 13), (130, 57), (64, 100)])
def test_bitwise_equal_to_independent_segments(precision, name, nx, ny):
    pr = _problem(nx, ny, name)
    ref = _run(pr, precision, -64)         # as many segments as rows: independent
    assert all(np.isfinite(f).all() for f in ref[:2])
    for rows in (4, 5, 9, 30, 256):        # rounded to a multiple of four segments
        for a, b in zip(ref, _run(pr, precision, rows)):
            assert np.array_equal(a, b), rows


@pytest.mark.parametrize("frame", [0, 1])
def test_batched_members_bitwise(frame):
    prs = [wl.problem(2, shape, alpha0_deg=11.0, seed=2, seed_radius=5.0, frame=frame, shift_row=6)
           for shape in ((31, 32), (70, 35), (61, 67), (130, 129))]
    solo = [_run(pr, pfiso.PF_F32, -64, 13) for pr in prs]
    ss = [pfiso.Solver(pr, precision=pfiso.PF_F32) for pr in prs]
    for s in ss:
        s.tune(8)
    b = pfiso.Batch(ss, graph_steps=6)
    b.step(13)
    for s, ref in zip(ss, solo):
        _, U, psi, _ = s.read_fields()
        assert np.array_equal(psi, ref[0]) and np.array_equal(U, ref[1])
    b.close()
    for s in ss:
        s.close()


@pytest.mark.parametrize("members,rows", [(4, 1500), (8, 4100), (20, 4200)])
def test_default_batch_rows_bitwise(members, rows):
    """Members nobody tuned, at 12, 64 and 164 strip rows per SIMD of 256 CUs:
    each side of the lines where a batch takes longer segments."""
    prs = [wl.problem(2, (61 + i % 3, rows + 13 * i), alpha0_deg=11.0, seed=i, seed_radius=5.0)
           for i in range(members)]
    prs += [wl.problem(2, (70, 33), alpha0_deg=11.0, seed=3, seed_radius=5.0)]
    ss = [pfiso.Solver(pr, precision=pfiso.PF_F32) for pr in prs]
    b = pfiso.Batch(ss, graph_steps=4)
    b.step(9)
    for i in (0, 1, members // 2, members - 1, members):
        psi, U, _ = _run(prs[i], pfiso.PF_F32, -64, 9)
        _, bU, bpsi, _ = ss[i].read_fields()
        assert np.array_equal(psi, bpsi) and np.array_equal(U, bU), i
    b.close()
    for s in ss:
        s.close()
