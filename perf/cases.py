"""Workloads of the phase-field library, timed and checked one pass at a time.

Each case is one call of a user's solve loop through the Python binding: a
few time steps of a resident solve (``Solver.step``), the tip query of a
monitoring loop, a batched step, a snapshot to the host, or a served trace.
``exact`` restates the scheme in plain torch FP64 for the same inputs.

Fields start from developed states as well as from seeds: fingers (capsules
along y) with tips at random heights, a rough slab, or one disc, so that both
interface and bulk cells are met.
"""
import math

import numpy as np
import torch

from paper_2110_12448_amd import pfiso, serve

SQ2 = math.sqrt(2.0)


# ------------------------------------------------------------------ the cases

def listed():
    return [
        # the monitoring loop of a small solve: a few steps, then where the tip is
        dict(name="small2d_128_tip", kind="tip", dim=2, nx=128, ny=128, nz=1, f64=False, steps=20,
             scheme="iso", state="disc", grains=1, frame=False, thermal="frozen", walls="xper"),
        # free growth between no-flux walls with the full anti-trapping current (the scheme
        # comparison's lattice)
        dict(name="iso2d_781_S21", kind="step", dim=2, nx=781, ny=781, nz=1, f64=False, steps=20,
             scheme="S21", state="centre", grains=1, frame=False, thermal="isothermal",
             walls="noflux"),
        # directional growth in a moving frame, the ordinary 2D production run
        dict(name="dir2d_1024x2048", kind="step", dim=2, nx=1024, ny=2048, nz=1, f64=False,
             steps=20, scheme="iso", state="fingers", grains=1, frame=True, thermal="frozen",
             walls="xper"),
        # the same in double precision (reference runs)
        dict(name="dir2d_1024x2048_f64", kind="step", dim=2, nx=1024, ny=2048, nz=1, f64=True,
             steps=10, scheme="iso", state="fingers", grains=1, frame=True, thermal="frozen",
             walls="xper"),
        # a large bicrystal array on sides that no tile divides
        dict(name="dir2d_4000x4099_multi", kind="step", dim=2, nx=4000, ny=4099, nz=1, f64=False,
             steps=4, scheme="iso", state="fingers", grains=4, frame=True, thermal="frozen",
             walls="xper"),
        # a parameter sweep: uneven 2D solves in one launch per step, replayed from a graph
        dict(name="batch2d_16", kind="batch", dim=2, nx=256, ny=1024, nz=1, f64=False, steps=10,
             scheme="iso", state="disc", grains=1, frame=False, thermal="frozen", walls="xper",
             members=16),
        # the 3D production run: polycrystal with 8 random grains
        dict(name="poly3d_256", kind="step", dim=3, nx=256, ny=256, nz=256, f64=False, steps=4,
             scheme="iso", state="slab", grains=8, frame=False, thermal="frozen", walls="xper"),
        # a developed polycrystal on the 27-point stencils
        dict(name="poly3d_160_441", kind="step", dim=3, nx=160, ny=160, nz=160, f64=False, steps=4,
             scheme="441", state="fingers", grains=8, frame=False, thermal="frozen", walls="xper"),
        # one 3D grain of the served sizes
        dict(name="seed3d_128", kind="step", dim=3, nx=128, ny=128, nz=128, f64=False, steps=10,
             scheme="iso", state="fingers", grains=1, frame=False, thermal="frozen", walls="xper"),
        # a ragged 3D box in double precision, moving frame, no-flux walls
        dict(name="poly3d_97x131x90_f64", kind="step", dim=3, nx=97, ny=131, nz=90, f64=True,
             steps=5, scheme="iso", state="fingers", grains=3, frame=True, thermal="frozen",
             walls="noflux"),
        # a snapshot of the ordinary 2D run to the host
        dict(name="snapshot_1024x2048", kind="snapshot", dim=2, nx=1024, ny=2048, nz=1, f64=False,
             steps=0, scheme="iso", state="fingers", grains=1, frame=False, thermal="frozen",
             walls="xper"),
        # a handful of queued requests served to completion (creation, steps, read-back)
        dict(name="serve_8", kind="serve", dim=2, nx=192, ny=448, nz=1, f64=False, steps=200,
             scheme="iso", state="disc", grains=1, frame=False, thermal="frozen", walls="xper",
             members=8),
    ]


def draw(rng):
    """Another case of the same ranges."""
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["step", "step", "step", "step", "step", "tip", "batch", "snapshot"])
    if kind == "batch":
        lo = log(64, 400)
        return dict(kind="batch", dim=2, nx=lo, ny=min(1024, lo * rng.randint(2, 4)), nz=1,
                    f64=rng.random() < 0.25, steps=rng.choice([4, 10, 12]), scheme="iso",
                    state=rng.choice(["disc", "fingers"]), grains=1, frame=False,
                    thermal=rng.choice(["frozen", "isothermal"]), walls=rng.choice(["xper", "noflux"]),
                    members=rng.randint(2, 16))
    f64 = rng.random() < 0.35
    frame = kind == "step" and rng.random() < 0.5
    common = dict(f64=f64, grains=rng.choice([1, 1, 2, 5, 8]), frame=frame,
                  thermal="frozen" if frame else rng.choice(["frozen", "frozen", "isothermal"]),
                  walls=rng.choice(["xper", "noflux"]))
    if rng.random() < 0.5:
        nx, ny = log(64, 3000), log(100, 4000)
        most = (16 if f64 else 60) * 1000000
        return dict(kind=kind, dim=2, nx=nx, ny=ny, nz=1,
                    steps=0 if kind == "snapshot" else max(1, min(20, most // (nx * ny))),
                    scheme=rng.choice(["iso", "iso", "iso", "S21", "S10"]),
                    state=rng.choice(["disc", "fingers", "slab"]), **common)
    nx, ny, nz = log(24, 240), log(32, 240), log(24, 240)
    most = (8 if f64 else 40) * 1000000
    return dict(kind=kind, dim=3, nx=nx, ny=ny, nz=nz,
                steps=0 if kind == "snapshot" else max(1, min(10, most // (nx * ny * nz))),
                scheme=rng.choice(["iso", "iso", "441"]),
                state=rng.choice(["disc", "fingers", "slab"]), **common)


def _sides(case):
    """Sides of the members of a batch or a served trace, between nx and ny."""
    lo, hi, n = case["nx"], case["ny"], case["members"]
    return [lo + (hi - lo) * ((5 * i) % n) // max(1, n - 1) for i in range(n)]


def _members(case):
    """The single solves that a case steps."""
    if case["kind"] == "batch":
        return [dict(case, nx=s, ny=s) for s in _sides(case)]
    if case["kind"] == "serve":
        # one request in four is three-dimensional
        return [dict(case, dim=3, nx=64 + 16 * i, ny=64, nz=72, state="slab") if i % 4 == 3
                else dict(case, nx=s, ny=s) for i, s in enumerate(_sides(case))]
    return [case]


def work(case):
    """Bytes and operations one pass cannot do without: each step reads psi, U
    (and the grain map) and writes psi, U."""
    size = 8 if case["f64"] else 4
    nbytes = flops = 0.0
    for m in _members(case):
        n = m["nx"] * m["ny"] * (m["nz"] if m["dim"] == 3 else 1)
        per = {"iso": 209, "S21": 295, "S10": 199} if m["dim"] == 2 else {"iso": 530, "441": 599}
        nbytes += n * m["steps"] * (4 * size + (1 if m["grains"] > 1 else 0))
        flops += n * m["steps"] * per[m["scheme"]]
        if case["kind"] == "tip":
            nbytes += n * 2 * size
        if case["kind"] in ("snapshot", "serve"):
            nbytes += n * (2 * size + 24)       # fields read, FP64 psi, U, phi written
    return {"bytes": nbytes, "flops": flops}


# ----------------------------------------------------------------- the inputs

def _device():
    return torch.device("cuda:0" if torch.cuda.is_available() else "cpu")


def _rotations(dim, n, gen):
    """Proper crystal -> lab rotations: about z in 2D, uniform in 3D."""
    out = []
    for _ in range(n):
        if dim == 2:
            a = math.radians(45.0 * float(torch.rand((), generator=gen)))
            out.append([[math.cos(a), -math.sin(a), 0.0], [math.sin(a), math.cos(a), 0.0],
                        [0.0, 0.0, 1.0]])
        else:
            w, x, y, z = (torch.randn(4, generator=gen, dtype=torch.float64)).tolist()
            s = 2.0 / (w * w + x * x + y * y + z * z)
            out.append([[1 - s * (y * y + z * z), s * (x * y - w * z), s * (x * z + w * y)],
                        [s * (x * y + w * z), 1 - s * (x * x + z * z), s * (y * z - w * x)],
                        [s * (x * z - w * y), s * (y * z + w * x), 1 - s * (x * x + y * y)]])
    return np.array(out)


def _problem(case, seed):
    """One solve: scalar parameters and FP64 fields, as the binding takes them."""
    dim, nx, ny, nz = case["dim"], case["nx"], case["ny"], case["nz"] if case["dim"] == 3 else 1
    gen = torch.Generator().manual_seed(int(seed) % (1 << 62))
    dev = _device()
    dgen = torch.Generator(device=dev).manual_seed(int(seed) % (1 << 62) + 1)
    if case["thermal"] == "isothermal":
        h, k, eps4 = 1.2, 0.1, 0.014
        lam = 5.0 * SQ2 / 8.0 * 16.0
        D = 47.0 / 75.0 * lam
    else:
        h, k, eps4, D = 0.8, 0.15, 0.02, 2.0
        lam = D / (47.0 / 75.0)
    H = ny * h
    lT = 40.0 * H if case["thermal"] == "frozen" else 0.0
    # a moving frame follows tips that are pulled about as fast as they grow
    pull = 0.0 if not lT else (1.0 if case["frame"] else 0.05)

    def rand(*shape):
        return torch.rand(shape, generator=gen, dtype=torch.float64)

    X = torch.arange(nx, device=dev, dtype=torch.float64).view(1, 1, nx) * h
    Y = torch.arange(ny, device=dev, dtype=torch.float64).view(1, ny, 1) * h
    Z = torch.arange(nz, device=dev, dtype=torch.float64).view(nz, 1, 1) * h
    per = 1 if case["walls"] == "xper" else 0

    def apart(a, at, side):
        """Distance along x or z to `at`, the short way around where periodic."""
        d = (a - at).abs()
        return torch.minimum(d, side * h - d) if per else d

    grain = np.zeros((nz, ny, nx), dtype=np.int8)
    if case["grains"] > 1:
        # columns along y: nearest of one random site per grain
        sites = rand(case["grains"], 2)
        d = [apart(X, float(a) * nx * h, nx) ** 2 + apart(Z, float(b) * nz * h, nz) ** 2
             for a, b in sites]
        gid = torch.stack(d).argmin(0).expand(nz, ny, nx)
        grain = gid.to(torch.int8).cpu().numpy()
    if case["state"] == "fingers":
        # primary spacing of about 60 cells, trunks of 6 to 12 W, tips around mid-height
        across = max(1, round(nx / 60)) if dim == 2 else max(1, round(nx / 60) * round(nz / 60) or 1)
        across = min(across, 80)
        psi = 4.0 * h - Y
        for i in range(across):
            u = rand(4).tolist()
            r = 6.0 + 6.0 * u[0]
            xc = (i + 0.25 + 0.5 * u[1]) / across * nx * h if dim == 2 else u[1] * nx * h
            zc = 0.0 if dim == 2 else u[2] * nz * h
            top = max(0.0, (0.35 + 0.1 * u[3]) * H - r)
            dy = (Y - top).clamp(min=0.0)
            psi = torch.maximum(psi, r - torch.sqrt(apart(X, xc, nx) ** 2 +
                                                        apart(Z, zc, nz) ** 2 + dy ** 2))
    elif case["state"] == "slab":
        psi = (5.0 * h + 0.6 * h * rand(1).item()) - Y
        psi = psi + 0.8 * torch.sin(X * (2 * math.pi / (nx * h)) * 3 + rand(1).item() * 6.28)
    else:
        yc = 0.5 * H if case["state"] == "centre" else 0.0
        r = (10.0 + rand(1).item()) * h
        psi = r - torch.sqrt(apart(X, (nx // 2) * h, nx) ** 2 + (Y - yc) ** 2 +
                             apart(Z, (nz // 2) * h, nz) ** 2)
    psi = psi.expand(nz, ny, nx).contiguous()
    noise = torch.rand(psi.shape, generator=dgen, device=dev, dtype=torch.float64) * 0.04 - 0.02
    psi = torch.where(psi.abs() < 3.0, psi + noise, psi)
    phi = torch.tanh(psi / SQ2)
    if case["thermal"] == "frozen":
        U = (k / ((1.0 - phi) / 2.0 + k * (1.0 + phi) / 2.0) - 1.0) / (1.0 - k)
    else:
        U = torch.full_like(psi, -0.43)
    U = U + 0.002 * torch.sin(X * (2 * math.pi * round(nx / 72 + 1) / (nx * h))) * torch.cos(Y / 7.0)
    shape = (nz, ny, nx) if dim == 3 else (ny, nx)
    w = {"iso": (2 / 3, 1 / 3, 0.0) if dim == 2 else (1 / 3, 2 / 3, 0.0),
         "441": (4 / 9, 4 / 9, 1 / 9), "S21": (2 / 3, 1 / 3, 0.0), "S10": (1.0, 0.0, 0.0)}
    return dict(dim=dim, nx=nx, ny=ny, nz=nz, w=w[case["scheme"]], k=k, eps4=eps4, D=D, lam=lam,
                h=h, dt=0.8 * h * h / (2 * dim * D), Vp=pull, lT=lT, y0=-0.5 * lT,
                bc=(per, 0, per if dim == 3 else 0), frame=int(case["frame"]),
                shift_row=ny // 2, rot=_rotations(dim, case["grains"], gen),
                psi0=psi.cpu().numpy().reshape(shape), U0=U.cpu().numpy().reshape(shape),
                grain=grain.reshape(shape), antitrapping=int(case["scheme"] in ("S21", "S10")),
                two_point=int(case["scheme"] == "S10"), dynamic_grains=0)


def prepare(case, seed):
    problems = [_problem(m, seed * 64 + i) for i, m in enumerate(_members(case))]
    precision = pfiso.PF_F64 if case["f64"] else pfiso.PF_F32
    state = dict(case=case)
    if case["kind"] == "serve":
        state["requests"] = [serve.Request(i, 0.0, p, case["steps"], precision)
                             for i, p in enumerate(problems)]
        return state
    state["solvers"] = [pfiso.Solver(p, precision=precision) for p in problems]
    if case["kind"] == "batch":
        state["batch"] = pfiso.Batch(state["solvers"],
                                     graph_steps=10 if case["steps"] % 10 == 0 else 0)
    return state


def _device_fields(s):
    """The solver's current psi and U as tensors over its own workspace."""
    dtype = torch.float64 if s.precision == pfiso.PF_F64 else torch.float32
    nbytes = math.prod(s.shape) * dtype.itemsize
    base = s.workspace.data_ptr()
    return [s.workspace[p - base:p - base + nbytes].view(dtype).view(s.shape)
            for p in s.device_fields()]


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "serve":
        srv = serve.Server(2 << 30, keep_fields=True, streams=4, max_waves=8192)
        done = srv.run(state["requests"], realtime=False)
        # results are kept in the precision of the solves
        return [[f.astype(np.float32) for f in r.fields] for r in sorted(done, key=lambda r: r.rid)]
    if kind == "batch":
        state["batch"].step(case["steps"])
        return [_device_fields(s) for s in state["solvers"]]
    s = state["solvers"][0]
    if kind == "snapshot":
        phi, U, psi, grain = s.read_fields()
        return dict(phi=phi, U=U, psi=psi, grain=grain)
    s.step(case["steps"])
    psi, U = _device_fields(s)
    out = dict(psi=psi, U=U)
    if kind == "tip":
        t = s.tip_state()
        out["y"] = np.float32(t["y_lab"])
        out["solid"] = np.float32(t["solid_fraction"])
        out["shift"] = t["frame_shift"]
    return out


# ------------------------------------------------------- the same in 64 bits

def _pad(f, bc, w):
    """Ghost cells, w deep on each side of every axis longer than one cell:
    wrapped where periodic, mirrored about the boundary face otherwise."""
    for axis, b in ((2, bc[0]), (1, bc[1]), (0, bc[2])):
        n = f.shape[axis]
        if n == 1:
            continue
        if b:
            lo, hi = f.narrow(axis, n - w, w), f.narrow(axis, 0, w)
        else:
            lo, hi = f.narrow(axis, 0, w).flip(axis), f.narrow(axis, n - w, w).flip(axis)
        f = torch.cat([lo, f, hi], axis)
    return f


class _Stencil:
    """A padded field read at cell offsets; `ring` more cells on each side."""

    def __init__(self, f, bc, w):
        self.flat = f.shape[0] == 1
        self.n, self.w, self.f = f.shape, w, _pad(f, bc, w)

    def __call__(self, dx, dy, dz=0, ring=0):
        f = self.f
        for axis, d in ((2, dx), (1, dy), (0, dz)):
            if axis == 0 and self.flat:
                continue
            f = f.narrow(axis, self.w - ring + d, self.n[axis] + 2 * ring)
        return f


def _inner(f, flat):
    """The interior of a field with one ring of ghost cells."""
    f = f[:, 1:-1, 1:-1]
    return f if flat else f[1:-1]


def _aniso(g, R, eps4, which):
    """a_s, or component `which` of a^2 g + |g|^2 a da/dg."""
    g2 = sum(v * v for v in g)
    on = g2 > 1e-12
    r2 = 1.0 / torch.where(on, g2, torch.ones_like(g2))
    c = [sum(R[3 * i + j] * g[i] for i in range(len(g))) for j in range(3)]
    s4 = sum((v * v * r2) ** 2 for v in c)
    a = 1.0 - 3.0 * eps4 + 4.0 * eps4 * s4
    if which is None:
        return torch.where(on, a, torch.ones_like(a))
    j = [v * (a * a - 16.0 * eps4 * a * s4 + 16.0 * eps4 * a * v * v * r2) for v in c]
    return torch.where(on, sum(R[3 * which + i] * j[i] for i in range(3)), g[which])


def _offsets(shell, flat):
    zs = (0,) if flat else (-1, 0, 1)
    return [(dx, dy, dz) for dz in zs for dy in (-1, 0, 1) for dx in (-1, 0, 1)
            if abs(dx) + abs(dy) + abs(dz) == shell]


def _app_b(p, mid):
    """h |grad psi|, fourth order, at a flux point: the east face, the north
    face or the north-east corner of each cell (and one ring around)."""
    def v(x, y):
        return p(x, y, ring=1)
    if mid == "E":
        a = [v(1, 1) - v(0, -1), v(2, 1) - v(-1, -1), v(1, 2) - v(0, -2)]
        b = [v(1, -1) - v(0, 1), v(2, -1) - v(-1, 1), v(1, -2) - v(0, 2)]
    elif mid == "N":
        a = [v(-1, 1) - v(1, 0), v(-1, 2) - v(1, -1), v(-2, 1) - v(2, 0)]
        b = [v(1, 1) - v(-1, 0), v(1, 2) - v(-1, -1), v(2, 1) - v(-2, 0)]
    else:
        a = [v(1, 1) - v(0, 0), v(2, 1) - v(-1, 0), v(1, 2) - v(0, -1)]
        b = [v(1, 0) - v(0, 1), v(2, 0) - v(-1, 1), v(1, -1) - v(0, 2)]
    c1, c2 = ((5 / 8, 1 / 48, 1 / 16), (5 / 8, 1 / 16, 1 / 48)) if mid == "NE" else \
             ((35 / 48, 1 / 48, 1 / 6), (35 / 96, 1 / 32, 1 / 24))
    gx = c1[0] * (a[0] + b[0]) - c1[1] * (a[1] + b[1]) - c1[2] * (a[2] + b[2])
    gy = c2[0] * (a[0] - b[0]) - c2[1] * (a[1] - b[1]) - c2[2] * (a[2] - b[2])
    return gx * gx + gy * gy


def _inv(g2, h):
    """h / |h g|, nothing where the gradient vanishes (|g|^2 <= 1e-12)."""
    on = g2 > 1e-12 * h * h
    return torch.where(on, h / torch.sqrt(torch.where(on, g2, torch.ones_like(g2))),
                       torch.zeros_like(g2))


def _divergence2d(q, al, be, psi, full):
    """div[al grad be] on the 2D shells or two-point faces; `full` divides
    each flux by |grad psi| at its flux point."""
    h, w = q["h"], q["w"]
    def A(x, y):
        return al(x, y, ring=1)
    def B(x, y):
        return be(x, y, ring=1) - be(0, 0, ring=1)
    if q["two_point"]:
        fE, fN = 0.5 * (A(0, 0) + A(1, 0)) * B(1, 0), 0.5 * (A(0, 0) + A(0, 1)) * B(0, 1)
        if full:
            def P(x, y):
                return psi(x, y, ring=1)
            tE = 0.25 * (P(0, 1) + P(1, 1) - P(0, -1) - P(1, -1))
            tN = 0.25 * (P(1, 0) + P(1, 1) - P(-1, 0) - P(-1, 1))
            fE = fE * _inv((P(1, 0) - P(0, 0)) ** 2 + tE ** 2, h)
            fN = fN * _inv((P(0, 1) - P(0, 0)) ** 2 + tN ** 2, h)
        d = fE[:, 1:-1, 1:-1] - fE[:, 1:-1, :-2] + fN[:, 1:-1, 1:-1] - fN[:, :-2, 1:-1]
        return d / (h * h)
    def plaq(x, y):   # mean of the plaquette whose lower left cell is (x, y)
        return 0.25 * (A(x, y) + A(x + 1, y) + A(x, y + 1) + A(x + 1, y + 1))
    fE = 0.25 * (A(0, 0) + A(1, 0) + plaq(0, 0) + plaq(0, -1)) * B(1, 0)
    fN = 0.25 * (A(0, 0) + A(0, 1) + plaq(0, 0) + plaq(-1, 0)) * B(0, 1)
    fNE, fNW = plaq(0, 0) * B(1, 1), plaq(-1, 0) * B(-1, 1)
    if full:
        iE, iN, iNE = (_inv(_app_b(psi, m), h) for m in ("E", "N", "NE"))
        fE, fN, fNE = fE * iE, fN * iN, fNE * iNE
        # the north-west corner is the north-east one of the cell to the left
        fNW = fNW[:, :, 1:] * iNE[:, :, :-1]
        fNW = torch.cat([torch.zeros_like(fNW[:, :, :1]), fNW], 2)
    d10 = fE[:, 1:-1, 1:-1] - fE[:, 1:-1, :-2] + fN[:, 1:-1, 1:-1] - fN[:, :-2, 1:-1]
    d11 = fNE[:, 1:-1, 1:-1] - fNE[:, :-2, :-2] + fNW[:, 1:-1, 1:-1] - fNW[:, :-2, 2:]
    return (w[0] * d10 + w[1] * 0.5 * d11) / (h * h)


def _divergence3d(q, al, be):
    """div[al grad be] on the 3D shells, link by link."""
    h, w = q["h"], q["w"]
    b0 = be(0, 0, 0)
    out = torch.zeros_like(b0)
    for shell in (1, 2, 3):
        if w[shell - 1] == 0.0:
            continue
        acc = torch.zeros_like(b0)
        for d in _offsets(shell, False):
            if shell == 1:
                cross = [(a, b, c) for a, b, c in _offsets(1, False)
                         if a * d[0] + b * d[1] + c * d[2] == 0]
                abar = (al(0, 0, 0) + al(*d)) / 4.0
                for o in cross:
                    abar = abar + (al(*o) + al(d[0] + o[0], d[1] + o[1], d[2] + o[2])) / 16.0
            else:
                # corners of the plaquette or cube spanned by the link
                xs, ys, zs = ((0, v) if v else (0,) for v in d)
                box = [(a, b, c) for a in xs for b in ys for c in zs]
                if shell == 3:
                    abar = sum(al(*o) for o in box) / 8.0
                else:
                    axis = d.index(0)
                    abar = sum(al(*o) for o in box) * (3.0 / 16.0)
                    for s in (-1, 1):
                        for o in box:
                            o = tuple(s if i == axis else v for i, v in enumerate(o))
                            abar = abar + al(*o) / 32.0
            acc = acc + abar * (be(*d) - b0)
        out = out + w[shell - 1] * acc * (1.0 if shell == 1 else 0.25) / (h * h)
    return out


def _step(q, psi, U, grain, n, shift):
    """One explicit step of psi and U (frame coordinates)."""
    dim, h, bc, eps4 = q["dim"], q["h"], q["bc"], q["eps4"]
    flat = dim == 2
    w = q["w"]
    p = _Stencil(psi, bc, 3)
    rot = torch.as_tensor(q["rot"], device=psi.device).reshape(-1, 9)
    gp = _Stencil(grain, bc, 1)(0, 0, 0, ring=1)
    Rr = [rot[:, i][gp] for i in range(9)] if rot.shape[0] > 1 else [rot[0, i] for i in range(9)]
    Ri = [_inner(r, flat) if r.dim() else r for r in Rr]
    axes = 2 if flat else 3
    unit = [tuple(int(i == a) for i in range(3)) for a in range(3)]

    def central(a, at, ring):
        lo = tuple(at[i] - unit[a][i] for i in range(3))
        hi = tuple(at[i] + unit[a][i] for i in range(3))
        return (p(*hi, ring=ring) - p(*lo, ring=ring)) / (2.0 * h)

    p0 = p(0, 0, 0)
    sums, grads = [], []
    for shell in (1, 2, 3)[:axes]:
        offs = _offsets(shell, flat)
        sums.append(sum(p(*o) - p0 for o in offs))
        half = [o for o in offs if next(v for v in o if v) > 0]
        grads.append(sum((p(*o) - p(*[-v for v in o])) ** 2 for o in half))
    if flat:
        L = (w[0] * sums[0] + w[1] * sums[1] / 2.0) / h ** 2
        G = (w[0] * grads[0] / 4.0 + w[1] * grads[1] / 8.0) / h ** 2
    else:
        L = (w[0] * sums[0] + w[1] * sums[1] / 4.0 + w[2] * sums[2] / 4.0) / h ** 2
        G = (w[0] * grads[0] / 4.0 + w[1] * grads[1] / 16.0 + w[2] * grads[2] / 16.0) / h ** 2
    ac = _aniso([central(a, (0, 0, 0), 0) for a in range(axes)], Ri, eps4, None)
    rest = -ac ** 2 * sums[0] / h ** 2
    for a in range(axes):
        g = [(p(*unit[a], ring=1) - p(0, 0, 0, ring=1)) / h if b == a else
             0.5 * (central(b, (0, 0, 0), 1) + central(b, unit[a], 1)) for b in range(axes)]
        J = _aniso(g, Rr, eps4, a)      # the grain of the lower cell
        here = _inner(J, flat)
        cut = [slice(None) if (flat and i == 0) else slice(1, -1) for i in range(3)]
        cut[2 - a] = slice(0, -2)
        rest = rest + (here - J[tuple(cut)]) / h
    F1, F2 = 1.0, U
    if q["lT"] > 0.0:
        y = torch.arange(psi.shape[1], device=psi.device, dtype=torch.float64).view(1, -1, 1)
        zeta = (y + shift) * h - q["y0"] - q["Vp"] * n * q["dt"]
        F1, F2 = 1.0 - (1.0 - q["k"]) * zeta / q["lT"], U + zeta / q["lT"]
    phi = torch.tanh(psi / SQ2)
    omp = 1.0 - phi * phi
    rate = (ac ** 2 * (L - SQ2 * phi * G) + rest + SQ2 * (phi - q["lam"] * omp * F2)) / (F1 * ac ** 2)
    aA = (1.0 + (1.0 - q["k"]) * U) * omp * rate / 2.0
    sA, sD, sU = _Stencil(aA, bc, 2), _Stencil(q["D"] * (1.0 - phi), bc, 2), _Stencil(U, bc, 2)
    if flat:
        div = _divergence2d(q, sD, sU, p, False) + _divergence2d(q, sA, p, p, q["antitrapping"])
    else:
        div = _divergence3d(q, sD, sU) + _divergence3d(q, sA, p)
    dU = (div + SQ2 * aA) / (1.0 + q["k"] - (1.0 - q["k"]) * phi)
    return psi + q["dt"] * rate, U + q["dt"] * dU, phi


def _crossings(phi, h):
    """Heights of the phi = 0 crossings between rows j and j + 1 (-inf elsewhere)."""
    lo, hi = phi[:, :-1], phi[:, 1:]
    j = torch.arange(lo.shape[1], device=phi.device, dtype=torch.float64).view(1, -1, 1)
    on = (lo >= 0) & (hi < 0)
    d = torch.where(on, lo - hi, torch.ones_like(lo))
    return torch.where(on, (j + lo / d) * h, torch.full_like(lo, -math.inf))


def _shifted(f):
    return torch.cat([f[:, 1:], f[:, -1:]], 1)


def _solve(q, steps):
    """psi and U after `steps`, stored as the solver stores them (a frame shift
    that the last step decided is still owed), the shift and whether it is."""
    dev = _device()
    shape = (q["nz"], q["ny"], q["nx"])
    psi, U = (torch.as_tensor(q[f], device=dev).reshape(shape) for f in ("psi0", "U0"))
    grain = torch.as_tensor(q["grain"], device=dev).reshape(shape).long()
    base, owed = 0, False
    for n in range(steps):
        if owed:
            psi, U, base = _shifted(psi), _shifted(U), base + 1
        psi, U, phi = _step(q, psi, U, grain, n, base)
        owed = bool(q["frame"]) and \
            float(_crossings(phi, q["h"]).max()) >= q["shift_row"] * q["h"]
    return psi, U, base, owed


def exact(case, seed):
    problems = [_problem(m, seed * 64 + i) for i, m in enumerate(_members(case))]
    kind, steps = case["kind"], case["steps"]
    got = []
    for q in problems:
        if kind in ("snapshot", "serve") and not case["f64"]:
            # what the solver holds: the fields in its own precision
            q = dict(q, psi0=q["psi0"].astype(np.float32).astype(np.float64),
                     U0=q["U0"].astype(np.float32).astype(np.float64))
        shape = q["psi0"].shape
        psi, U, base, owed = _solve(q, steps)
        if kind in ("snapshot", "serve"):
            phi = torch.tanh(psi / SQ2)
            got.append([f.cpu().numpy().reshape(shape) for f in (phi, U, psi)])
        else:
            out = dict(psi=psi.reshape(shape), U=U.reshape(shape))
            if kind == "tip":
                if owed:
                    psi = _shifted(psi)
                phi = torch.tanh(psi / SQ2)
                out["y"] = np.float64(float(_crossings(phi, q["h"]).max()) +
                                      (base + owed) * q["h"])
                out["solid"] = np.float64(float((1.0 + phi).mean()) / 2.0)
                out["shift"] = None
            got.append(out)
    if kind == "serve":
        return got
    if kind == "snapshot":
        return dict(phi=got[0][0], U=got[0][1], psi=got[0][2], grain=None)
    if kind == "batch":
        return [[o["psi"], o["U"]] for o in got]
    return got[0]
