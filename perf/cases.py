"""The work that a program built on this library has it do, as timed cases.

A case is one pass through the public entry points on one shell (mt, nr):

  apply    one operator apply y = K(eta) [u; p]: the step of a program's own Krylov
           solver, in FP32 and FP64, with the options of the operator (no slip, free
           slip, hourglass control, two-point rule, compressible mass rows, A alone);
  vcycle   one multigrid V-cycle of the velocity block, the preconditioner of a
           program's own iteration (FP32 as in a mixed solve, FP64);
  solve    about ten FGMRES iterations of the Stokes solve for a new viscosity (set-up
           included), the solve of one time step of the paper;
  step     one coupled Stokes-energy time step (SUPG or MMOC) with ten FGMRES iterations;
  energy   one SUPG energy apply: the step of a program's own energy solver;
  fields   a new temperature: viscosity on every level, its diagonals and pressure mass,
           and the buoyancy (what a program's own solver sets up per time step);
  advect   one MMOC advection of the temperature along a flow;
  serve    a burst of requests through the server, ten FGMRES iterations each.

The shells are those of the repository's tests and benchmark, (8,8) to (256,256), and
ragged ones whose radial count is no power of two.
"""
import math

import numpy as np
import torch

import paper_2609_21633_amd as tng

R_IN, R_OUT = 0.55, 1.0
RA = 1e5
E, F = math.log(1e3), math.log(10.0)    # viscosity exp(-E T + F (1 - r))
TYPES = {"f32": torch.float32, "f64": torch.float64}
# operator options of an apply: flags and hourglass scale
FLAGS = {
    "K": (tng.OP_A | tng.OP_BT | tng.OP_B | tng.OP_DIRICHLET, 0.0),
    "A": (tng.OP_A | tng.OP_DIRICHLET, 0.0),
    "K+freeslip": (tng.OP_A | tng.OP_BT | tng.OP_B | tng.OP_DIRICHLET | tng.OP_FREESLIP_OUTER, 0.0),
    "K+hourglass": (tng.OP_A | tng.OP_BT | tng.OP_B | tng.OP_DIRICHLET, 0.1),
    "K+twopoint": (tng.OP_A | tng.OP_BT | tng.OP_B | tng.OP_DIRICHLET | tng.OP_TWOPOINT, 0.0),
    "K+tala": (tng.OP_A | tng.OP_BT | tng.OP_B | tng.OP_DIRICHLET | tng.OP_TALA, 0.0),
}


def listed():
    return [
        # the headline apply of the benchmark: one Krylov step of a mixed solve
        {"name": "apply f32 128x128", "kind": "apply", "mt": 128, "nr": 128, "dtype": "f32", "op": "K"},
        # the same in FP64, a medium shell: the outer residual of the refinement
        {"name": "apply f64 64x64", "kind": "apply", "mt": 64, "nr": 64, "dtype": "f64", "op": "K"},
        # the smallest call: a coarse level of a program's own multigrid, launches count
        {"name": "apply f32 8x8", "kind": "apply", "mt": 8, "nr": 8, "dtype": "f32", "op": "K"},
        # free slip on the outer sphere (the verification setup), a ragged radial count
        {"name": "apply f64 freeslip 32x90", "kind": "apply", "mt": 32, "nr": 90, "dtype": "f64", "op": "K+freeslip"},
        # the preconditioner of a mixed solve at the headline size
        {"name": "vcycle f32 128x128", "kind": "vcycle", "mt": 128, "nr": 128, "dtype": "f32", "smooth": 2},
        # the same of a small FP64 solve, where launches count
        {"name": "vcycle f64 32x32", "kind": "vcycle", "mt": 32, "nr": 32, "dtype": "f64", "smooth": 2},
        # a small solve from a new viscosity: set-up and ten iterations
        {"name": "solve f64 32x32", "kind": "solve", "mt": 32, "nr": 32, "its": 10},
        # a time step on a medium shell
        {"name": "step supg 64x64", "kind": "step", "mt": 64, "nr": 64, "scheme": "supg", "courant": 1.0},
        # the energy operator on the large shell of the coupled runs
        {"name": "energy f32 256x256", "kind": "energy", "mt": 256, "nr": 256, "dtype": "f32"},
        # a new temperature at the headline size
        {"name": "fields f64 128x128", "kind": "fields", "mt": 128, "nr": 128, "dtype": "f64"},
        # advection of the temperature, twice the CFL step
        {"name": "advect 64x64", "kind": "advect", "mt": 64, "nr": 64, "courant": 2.0},
        # a burst of small requests
        {"name": "serve 16x16", "kind": "serve", "mt": 16, "nr": 16, "requests": 8},
    ]


def _log_choice(rng, values, top):
    return rng.choice([v for v in values if v <= top])


def draw(rng):
    kind = rng.choice(["apply", "apply", "apply", "vcycle", "vcycle", "solve", "step", "energy", "energy", "fields",
                       "advect", "serve"])
    dtype = rng.choice(["f32", "f64"])
    if kind == "apply":
        mt = _log_choice(rng, (4, 8, 16, 32, 64, 128), 128 if dtype == "f32" else 64)
        nr = 2 * int(round(math.exp(rng.uniform(math.log(4), math.log(64)))))
        op = rng.choice(["K", "K", "K", "A", "A", "K+freeslip", "K+hourglass", "K+twopoint", "K+tala"])
        return {"kind": kind, "mt": mt, "nr": nr, "dtype": dtype, "op": op}
    if kind in ("vcycle", "solve", "step", "serve"):
        # the coarsest level is (2, 2) or (2, 3): a whole number of radial cells on every level
        mt = _log_choice(rng, (8, 16, 32, 64, 128), {"vcycle": 128 if dtype == "f32" else 64, "solve": 32, "step": 64,
                                                     "serve": 16}[kind])
        c = {"kind": kind, "mt": mt, "nr": mt // 2 * rng.choice([2, 3])}
        if kind == "vcycle":
            c.update(dtype=dtype, smooth=rng.choice([1, 2, 3]))
        elif kind == "solve":
            c["its"] = rng.randint(5, 12)
        elif kind == "step":
            c.update(scheme=rng.choice(["supg", "mmoc"]), courant=round(rng.uniform(0.5, 2.0), 2))
        else:
            c["requests"] = rng.randint(1, 8)
        return c
    nr = int(round(math.exp(rng.uniform(math.log(8), math.log(128)))))
    if kind == "energy":
        return {"kind": kind, "mt": _log_choice(rng, (8, 16, 32, 64, 128, 256), 256 if dtype == "f32" else 128),
                "nr": nr, "dtype": dtype}
    if kind == "fields":
        return {"kind": kind, "mt": _log_choice(rng, (8, 16, 32, 64, 128), 128), "nr": max(8, nr // 4 * 4),
                "dtype": dtype}
    return {"kind": kind, "mt": _log_choice(rng, (8, 16, 32, 64), 64), "nr": min(nr, 64),
            "courant": round(rng.uniform(0.5, 4.0), 2)}


# ---- shell geometry in the library's layout (include/tng.h) ---------------------------

def _corners():
    n, s = np.array([0.0, 0.0, 1.0]), np.array([0.0, 0.0, -1.0])
    z, c = 1 / math.sqrt(5.0), 2 / math.sqrt(5.0)

    def ring(k, up):
        a = 2 * math.pi * (k % 5) / 5 + (0.0 if up else math.pi / 5)
        return np.array([c * math.cos(a), c * math.sin(a), z if up else -z])
    north = [(n, ring(d, True), ring(d + 1, True), ring(d, False)) for d in range(5)]
    south = [(ring(d - 4, True), ring(d - 5, False), ring(d - 4, False), s) for d in range(5, 10)]
    return north + south


class _Shell:
    """Unit vectors [10][m+1][m+1][3], node radii, and the shared lateral nodes."""

    def __init__(self, mt, nr, device):
        g = np.array([[[a, b], [c, d]] for a, c, b, d in _corners()])   # [10][i][j][3]
        while g.shape[1] < mt + 1:
            k = g.shape[1]
            f = np.empty((10, 2 * k - 1, 2 * k - 1, 3))
            f[:, ::2, ::2] = g
            f[:, 1::2, ::2] = g[:, :-1] + g[:, 1:]
            f[:, ::2, 1::2] = g[:, :, :-1] + g[:, :, 1:]
            f[:, 1::2, 1::2] = g[:, 1:, :-1] + g[:, :-1, 1:]
            f[:, 1::2] /= np.linalg.norm(f[:, 1::2], axis=-1, keepdims=True)
            f[:, ::2, 1::2] /= np.linalg.norm(f[:, ::2, 1::2], axis=-1, keepdims=True)
            g = f
        self.m, self.n = mt, nr
        # the first slot of every lateral node: only diamond edges are shared
        flat, edge = g.reshape(-1, 3), np.zeros((10, mt + 1, mt + 1), bool)
        edge[:, [0, -1]] = edge[:, :, [0, -1]] = True
        at = np.flatnonzero(edge.ravel())
        _, first, inv = np.unique(np.round(flat[at] * 1e9).astype(np.int64), axis=0, return_index=True,
                                  return_inverse=True)
        owner = np.arange(len(flat))
        owner[at] = at[first[inv.ravel()]]
        self.owner = torch.tensor(owner, device=device)
        self.s = torch.tensor(g, device=device)
        self.r = torch.linspace(R_IN, R_OUT, nr + 1, dtype=torch.float64, device=device)
        self.shape = (10, mt + 1, mt + 1, nr + 1)

    def same(self, f):
        """The first copy's value in every copy."""
        v = f.reshape(-1, len(self.owner), f.shape[-1])
        return v[:, self.owner].reshape(f.shape)

    def total(self, f):
        """The sum over the copies in every copy."""
        v = f.reshape(-1, len(self.owner), f.shape[-1])
        return torch.zeros_like(v).index_add_(1, self.owner, v)[:, self.owner].reshape(f.shape)


def _pattern(sh, gen, dev):
    """A smooth lateral pattern of largest size one: waves of degree 1 to 8."""
    a = torch.zeros(sh.s.shape[:3], dtype=torch.float64, device=dev)
    for l in range(1, 9):
        w = torch.randn(5, generator=gen, dtype=torch.float64)
        k = l * w[:3] / w[:3].norm()
        a += w[3].item() * torch.cos(sh.s @ k.to(dev) + 3 * w[4].item())
    return a / a.abs().max()


def _bump(sh):
    return torch.sin(math.pi * (sh.r - R_IN) / (R_OUT - R_IN))


def _temperature(sh, gen, dev):
    prof = R_IN * (R_OUT - sh.r) / (sh.r * (R_OUT - R_IN))
    return sh.same(prof + 0.01 * _pattern(sh, gen, dev)[..., None] * _bump(sh))


def _flow(sh, gen, dev, size):
    """A smooth flow, tangential and radial, zero on both spheres, |u| up to `size`."""
    u = torch.zeros((3,) + sh.shape, dtype=torch.float64, device=dev)
    for _ in range(3):
        a = torch.randn(3, generator=gen, dtype=torch.float64).to(dev)
        t = torch.cross(a.expand_as(sh.s), sh.s, dim=-1) * _pattern(sh, gen, dev)[..., None]
        u += torch.movedim(t, -1, 0)[..., None] * _bump(sh)
    u += torch.movedim(sh.s * _pattern(sh, gen, dev)[..., None], -1, 0)[..., None] * _bump(sh)
    return sh.same(u * (size / u.norm(dim=0).max()))


def _rho(sh):
    return 2.0 - sh.r     # denser below


def _inputs(case, seed):
    """The case's inputs in FP64, from the seed alone."""
    dev = torch.device("cuda", 0)
    gen = torch.Generator().manual_seed(seed)
    cgen = torch.Generator(device=dev).manual_seed(seed)
    sh = _Shell(case["mt"], case["nr"], dev)
    d = {"shell": sh, "dev": dev}
    kind = case["kind"]

    def uniform(shape):
        return 2 * torch.rand(shape, generator=cgen, dtype=torch.float64, device=dev) - 1
    if kind == "serve":
        d["T"] = [_temperature(sh, gen, dev) for _ in range(case["requests"])]
        d["contrast"] = (2 + 4 * torch.rand(case["requests"], generator=gen, dtype=torch.float64)).tolist()
        return d
    if kind == "energy":
        d["T"], d["u"] = _temperature(sh, gen, dev), _flow(sh, gen, dev, 300.0)
        return d
    d["T"] = _temperature(sh, gen, dev)
    if kind in ("apply", "vcycle", "solve"):
        d["eta"] = torch.stack([_eta(d["T"], sh.r, w, case["mt"], case["nr"]) for w in range(2)], -1)
    if kind == "apply":
        # a Krylov vector of a solve with zero boundary velocities
        d["u"] = sh.same(uniform((3,) + sh.shape))
        d["u"][..., 0] = 0.0
        if case["op"] != "K+freeslip":
            d["u"][..., -1] = 0.0
        d["psh"] = _Shell(case["mt"] // 2, case["nr"] // 2, dev)
        d["p"] = d["psh"].same(uniform(d["psh"].shape))
    elif kind == "vcycle":
        b = sh.same(uniform((3,) + sh.shape))
        b[..., 0] = b[..., -1] = 0.0
        d["b"] = b
    elif kind == "step":
        d["H"] = sh.same(5 + 5 * uniform(sh.shape))
    elif kind == "advect":
        u = _flow(sh, gen, dev, 300.0)
        # the step of `courant` cells laterally and radially at the largest speed
        d["u"], d["dt"] = u, case["courant"] * min(1.2 / case["mt"] * R_IN, (R_OUT - R_IN) / case["nr"]) / 300.0
    return d


def _levels(mt):
    return int(math.log2(mt))


def prepare(case, seed):
    d = _inputs(case, seed)
    kind, dev = case["kind"], d["dev"]
    dt = TYPES[case.get("dtype", "f64")]
    ctx = tng.Context(0)
    st = {"kind": kind, "ctx": ctx, "case": case}
    if kind == "serve":
        st["server"] = tng.Server(ctx, [(case["mt"], case["nr"])], 16 << 30, max_slots=16, mixed=0, max_iters=10)
        st["T"], st["contrast"] = d["T"], d["contrast"]
        mesh = tng.Mesh(None, case["mt"], case["nr"], levels=2)
        st["u"] = [torch.zeros((3,) + mesh.shape(0), dtype=torch.float64, device=dev) for _ in d["T"]]
        st["p"] = [torch.zeros(mesh.shape(1), dtype=torch.float64, device=dev) for _ in d["T"]]
        torch.cuda.synchronize()
        return st
    nlev = {"apply": 2, "energy": 1, "fields": 3, "advect": 1}.get(kind) or _levels(case["mt"])
    mesh = tng.Mesh(ctx, case["mt"], case["nr"], R_IN, R_OUT, levels=nlev)
    st["mesh"] = mesh
    if kind in ("apply", "vcycle", "solve"):
        st["eta"] = d["eta"].to(dt)
    if kind == "apply":
        if case["op"] == "K+tala":
            mesh.set_density(_rho(d["shell"]).cpu().numpy())
        st["u"], st["p"] = d["u"].to(dt), d["p"].to(dt)
        st["yu"], st["yp"] = torch.zeros_like(st["u"]), torch.zeros_like(st["p"])
    elif kind == "energy":
        st["T"], st["u"] = d["T"].to(dt), d["u"].to(dt)
        st["y"] = torch.zeros_like(st["T"])
    elif kind == "vcycle":
        mixed = 1 if case["dtype"] == "f32" else 0
        st["solver"] = tng.StokesSolver(ctx, mesh, mixed=mixed, restart=2, pre=case["smooth"],
                                          post=case["smooth"])
        st["solver"].setup(st["eta"].double())
        st["b"] = d["b"].to(dt)
        st["x"] = torch.zeros_like(st["b"])
    elif kind in ("solve", "step"):
        st["solver"] = tng.StokesSolver(ctx, mesh, mixed=0, max_iters=case.get("its", 10))
        st["u"] = torch.zeros((3,) + mesh.shape(0), dtype=torch.float64, device=dev)
        st["p"] = torch.zeros(mesh.shape(1), dtype=torch.float64, device=dev)
        st["f"] = torch.empty_like(st["u"])
        tng.rhs_buoyancy(ctx, mesh, 0, d["T"], RA, st["f"])
        st["T"], st["H"] = d["T"], d.get("H")
    elif kind == "fields":
        st["T"] = d["T"].to(dt)
        st["eta"] = [torch.zeros(mesh.wedge_shape(l), dtype=dt, device=dev) for l in range(nlev)]
        st["diag"] = [torch.zeros((3,) + mesh.shape(l), dtype=dt, device=dev) for l in range(nlev)]
        st["mass"] = torch.zeros(mesh.shape(1), dtype=dt, device=dev)
        st["f"] = torch.zeros((3,) + mesh.shape(0), dtype=dt, device=dev)
    elif kind == "advect":
        st["T"], st["u"], st["dt"] = d["T"], d["u"], d["dt"]
        st["That"] = torch.zeros_like(d["T"])
    torch.cuda.synchronize()
    return st


def run(st):
    kind, ctx, case = st["kind"], st["ctx"], st["case"]
    mesh = st.get("mesh")
    if kind == "apply":
        flags, hg = FLAGS[case["op"]]
        if case["op"] == "A":
            tng.stokes_apply(ctx, mesh, 0, flags, st["eta"], st["u"], None, st["yu"], None, hg_alpha=hg)
            return st["yu"]
        tng.stokes_apply(ctx, mesh, 0, flags, st["eta"], st["u"], st["p"], st["yu"], st["yp"], hg_alpha=hg)
        return st["yu"], st["yp"]
    if kind == "vcycle":
        st["solver"].vcycle(st["b"], st["x"])
        return st["x"]
    if kind == "solve":
        st["solver"].solve(st["f"], None, st["u"], st["p"], eta=st["eta"], raise_on_fail=False)
        return st["u"], st["p"]
    if kind == "step":
        T = st["T"].clone()      # the program keeps T^n
        st["solver"].energy_step(T, st["u"], st["p"], H=st["H"], Ra=RA, E=E, F=F, courant=case["courant"],
                                 scheme=case["scheme"], raise_on_fail=False)
        return T, st["u"], st["p"]
    if kind == "energy":
        tng.energy_apply(ctx, mesh, 0, st["u"], 1e-4, st["T"], st["y"])
        return st["y"]
    if kind == "fields":
        eta, n = st["eta"], len(st["eta"])
        tng.eta_from_temperature(ctx, mesh, 0, st["T"], E, F, eta[0])
        for l in range(n - 1):
            tng.eta_coarsen(ctx, mesh, l, eta[l], eta[l + 1])
        for l in range(n):
            tng.diag_A(ctx, mesh, l, eta[l], st["diag"][l])
        tng.pressure_mass(ctx, mesh, 0, eta[0], st["mass"])
        tng.rhs_buoyancy(ctx, mesh, 0, st["T"], RA, st["f"])
        return eta, st["diag"], st["mass"], st["f"]
    if kind == "advect":
        tng.mmoc_advect(ctx, mesh, 0, st["u"], st["dt"], st["T"], st["That"])
        return st["That"]
    srv = st["server"]
    tickets = [srv.submit(0, T, lc, RA, u, p) for T, lc, u, p in zip(st["T"], st["contrast"], st["u"], st["p"])]
    srv.wait()
    for t in tickets:
        srv.poll(t)
    return st["u"], st["p"]


def _slots(m, n):
    return 10 * (m + 1) ** 2 * (n + 1)


def work(case):
    """Every input read once and every output written once; about 300 floating-point
    operations a wedge of the Stokes operator, 200 of the energy operator."""
    kind, m, n = case["kind"], case["mt"], case["nr"]
    es = 4 if case.get("dtype") == "f32" else 8
    ns, wd, ps = _slots(m, n), 20 * m * m * n, _slots(m // 2, n // 2)
    if kind == "apply":
        a = case["op"] == "A"
        return {"bytes": es * (6 * ns + wd + (0 if a else 2 * ps)), "flops": (250 if a else 300) * wd}
    # V-cycle: right-hand side and result, viscosity and inverse diagonal of each level
    # (8/7 of the finest); four operator applies a smoothing step before and after it, less
    # the one that starts from zero, and one for the residual
    cyc = {"bytes": es * (6 * ns + 8 / 7 * (wd + 3 * ns)), "flops": 8 / 7 * 4 * case.get("smooth", 2) * 250 * wd}
    if kind == "vcycle":
        return cyc
    # set-up (viscosity, power iterations) and the iterations: a V-cycle and an apply each
    its = case.get("its", 10)
    sol = {"bytes": its * (cyc["bytes"] + es * (6 * ns + wd + 2 * ps)) + es * (6 * ns + ps + wd),
           "flops": its * (cyc["flops"] + 300 * wd) + 10 * 8 / 7 * 250 * wd}
    if kind == "solve":
        return sol
    if kind == "serve":
        return {k: v * case["requests"] for k, v in sol.items()}
    if kind == "step":
        return {"bytes": sol["bytes"] + es * 10 * 5 * ns, "flops": sol["flops"] + 10 * 200 * wd}
    if kind == "energy":
        return {"bytes": es * 5 * ns, "flops": 200 * wd}
    if kind == "fields":
        return {"bytes": es * (ns + 8 / 7 * (2 * wd + 3 * ns) + ps + wd + 3 * ns), "flops": 300 * wd}
    return {"bytes": es * 5 * ns, "flops": 600 * ns}


# ---- the same in 64 bits, in plain torch, per wedge ------------------------------------

_LAT = (((0, 0), (1, 0), (0, 1)), ((1, 1), (0, 1), (1, 0)))   # lateral nodes of the two wedges


def _at(f, w, j, m, n):
    """Node j (0-2 below, 3-5 above) of wedge w of every cell, f = [..., m+1, m+1, n+1]."""
    (a, b), c = _LAT[w][j % 3], j // 3
    return f[..., a:a + m, b:b + m, c:c + n]


def _basis(s, r, w, zeta=0.0):
    """V and the basis gradients of wedge w at (1/3, 1/3, zeta) in one diamond, s = [m+1, m+1, 3]."""
    m, n = s.shape[0] - 1, len(r) - 1
    x = s.movedim(-1, 0)[..., None] * r                       # [3, m+1, m+1, n+1]
    third = 1.0 / 3.0
    dlat = ((-1.0, -1.0), (1.0, 0.0), (0.0, 1.0))
    rad = (0.5 * (1 - zeta), 0.5 * (1 + zeta))
    dn = [(dlat[j % 3][0] * rad[j // 3], dlat[j % 3][1] * rad[j // 3], third * (0.5 if j > 2 else -0.5))
          for j in range(6)]
    J = [sum(dn[j][k] * _at(x, w, j, m, n) for j in range(6) if dn[j][k]) for k in range(3)]
    c = [torch.linalg.cross(J[1], J[2], dim=0), torch.linalg.cross(J[2], J[0], dim=0),
         torch.linalg.cross(J[0], J[1], dim=0)]
    det = (J[0] * c[0]).sum(0)
    g = [(dn[j][0] * c[0] + dn[j][1] * c[1] + dn[j][2] * c[2]) / det for j in range(6)]
    return det.abs(), g


def _add(y, w, j, m, n, v):
    (a, b), c = _LAT[w][j % 3], j // 3
    y[..., a:a + m, b:b + m, c:c + n] += v


def _to_fine(c):
    """W1 interpolation of one node field [10, ...] to the next finer level."""
    _, a, b, k = c.shape
    f = c.new_empty((10, 2 * a - 1, 2 * b - 1, k))
    f[:, ::2, ::2] = c
    f[:, 1::2, ::2] = 0.5 * (c[:, 1:] + c[:, :-1])
    f[:, ::2, 1::2] = 0.5 * (c[:, :, 1:] + c[:, :, :-1])
    f[:, 1::2, 1::2] = 0.5 * (c[:, 1:, :-1] + c[:, :-1, 1:])
    o = f.new_empty(f.shape[:3] + (2 * k - 1,))
    o[..., ::2] = f
    o[..., 1::2] = 0.5 * (f[..., 1:] + f[..., :-1])
    return o


def _to_coarse(f):
    """The transpose of _to_fine."""
    c = f[..., ::2].clone()
    c[..., 1:] += 0.5 * f[..., 1::2]
    c[..., :-1] += 0.5 * f[..., 1::2]
    o = c[:, ::2, ::2].clone()
    h = 0.5 * c[:, 1::2, ::2]
    o[:, 1:] += h
    o[:, :-1] += h
    h = 0.5 * c[:, ::2, 1::2]
    o[:, :, 1:] += h
    o[:, :, :-1] += h
    h = 0.5 * c[:, 1::2, 1::2]
    o[:, 1:, :-1] += h
    o[:, :-1, 1:] += h
    return o


def _eta(T, r, w, m, n):
    rm = 0.5 * (r[1:] + r[:-1])
    return torch.exp(-E * sum(_at(T, w, j, m, n) for j in range(6)) / 6 + F * (1 - rm))


def _exact_apply(case, d):
    sh, m, n = d["shell"], case["mt"], case["nr"]
    op, (_, alpha) = case["op"], FLAGS[case["op"]]
    dt = TYPES[case["dtype"]]
    u0, p = d["u"].to(dt).double(), d["p"].to(dt).double()      # what the call is given
    u = u0.clone()
    u[..., 0] = 0.0
    rhat = sh.s.movedim(-1, 0)
    if op == "K+freeslip":
        u[..., -1] -= rhat * (rhat * u[..., -1]).sum(0)
    else:
        u[..., -1] = 0.0
    full = op != "A"
    pf = _to_fine(p)
    y, yd = torch.zeros_like(u), torch.zeros_like(u[0])
    h = [[((1.0 if j % 3 == a else 0.0) - 1 / 3) * (1.0 if j > 2 else -1.0) for j in range(6)] for a in range(3)]
    for q in range(10):
        for w in range(2):
            eta = d["eta"][q, ..., w].to(dt).double()
            un = [_at(u[:, q], w, j, m, n) for j in range(6)]
            V, g = _basis(sh.s[q], sh.r, w)
            pts = [(V, g, 1.0)] if op != "K+twopoint" else [
                _basis(sh.s[q], sh.r, w, z) + (0.5,) for z in (-1 / math.sqrt(3.0), 1 / math.sqrt(3.0))]
            for Vq, gq, wt in pts:
                L = sum(un[j][:, None] * gq[j][None] for j in range(6))
                S = L + L.transpose(0, 1)
                tr = L[0, 0] + L[1, 1] + L[2, 2]
                for k in range(3):
                    S[k, k] -= 2.0 / 3.0 * tr
                S *= wt * Vq * eta
                for j in range(6):
                    _add(y[:, q], w, j, m, n, (S * gq[j][None]).sum(1))
            if alpha:
                eps = alpha / 18.0 * (10.0 / 3.0) * V * eta * sum((g[j] ** 2).sum(0) for j in range(6))
                for a in range(3):
                    v = eps * sum(h[a][j] * un[j] for j in range(6))
                    for j in range(6):
                        _add(y[:, q], w, j, m, n, h[a][j] * v)
            if full:
                pb = sum(_at(pf[q], w, j, m, n) for j in range(6)) / 6
                rho = _rho(sh) if op == "K+tala" else torch.ones_like(sh.r)
                dv = -V * sum((un[j] * g[j]).sum(0) * rho[j // 3:j // 3 + n] for j in range(6)) / 6
                for j in range(6):
                    _add(y[:, q], w, j, m, n, -V * pb * g[j])
                    _add(yd[q], w, j, m, n, dv)
    y = sh.total(y)
    y[..., 0] = u0[..., 0]
    if op == "K+freeslip":
        y[..., -1] += rhat * (rhat * (u0[..., -1] - y[..., -1])).sum(0)
    else:
        y[..., -1] = u0[..., -1]
    return (y, d["psh"].total(_to_coarse(yd))) if full else y


def _exact_energy(case, d):
    sh, m, n = d["shell"], case["mt"], case["nr"]
    dt = TYPES[case["dtype"]]
    T, u = d["T"].to(dt).double(), d["u"].to(dt).double()
    y = torch.zeros_like(T)
    for q in range(10):
        for w in range(2):
            V, g = _basis(sh.s[q], sh.r, w)
            Tn = [_at(T[q], w, j, m, n) for j in range(6)]
            gT = sum(Tn[j] * g[j] for j in range(6))
            ub = sum(_at(u[:, q], w, j, m, n) for j in range(6)) / 6
            size, hh = ub.norm(dim=0), V ** (1 / 3)
            pe = 0.5 * size * hh
            pl = pe.clamp_min(0.05)
            z = pe * pe
            series = (1 - z / 15 * (1 - 2 * z / 21 * (1 - z / 10))) / 3
            tau = 0.25 * hh * hh * torch.where(pe < 0.05, series, (1 / torch.tanh(pl) - 1 / pl) / pl)
            a = (ub * gT).sum(0)
            for j in range(6):
                _add(y[q], w, j, m, n, V * (Tn[j] / 6 / 1e-4 + (g[j] * gT).sum(0) + a / 6 +
                                            tau * (ub * g[j]).sum(0) * a))
    y = sh.total(y)
    y[..., 0], y[..., -1] = T[..., 0], T[..., -1]
    return y


def _exact_fields(case, d):
    m, n, dev = case["mt"], case["nr"], d["dev"]
    dt = TYPES[case["dtype"]]
    T = d["T"].to(dt).double()
    sh = d["shell"]
    eta = [torch.stack([_eta(T, sh.r, w, m, n) for w in range(2)], -1)]
    for _ in range(2):
        e = eta[-1].reshape((10, eta[-1].shape[1] // 2, 2, eta[-1].shape[2] // 2, 2, eta[-1].shape[3] // 2, 2, 2)).sum(6)
        # four lateral children: three corner triangles and the centre one
        c0 = e[:, :, 0, :, 0, :, 0] + e[:, :, 1, :, 0, :, 0] + e[:, :, 0, :, 1, :, 0] + e[:, :, 0, :, 0, :, 1]
        c1 = e[:, :, 1, :, 1, :, 1] + e[:, :, 0, :, 1, :, 1] + e[:, :, 1, :, 0, :, 1] + e[:, :, 1, :, 1, :, 0]
        eta.append(torch.stack([c0, c1], -1) / 8)
    diag, mass, f = [], None, None
    for l in range(3):
        ml, nl = m >> l, n >> l
        s = sh if l == 0 else _Shell(ml, nl, dev)
        dg = torch.zeros((3,) + s.shape, dtype=torch.float64, device=dev)
        pm = torch.zeros(s.shape, dtype=torch.float64, device=dev)
        b = torch.zeros_like(dg) if l == 0 else None
        for q in range(10):
            for w in range(2):
                V, g = _basis(s.s[q], s.r, w)
                e = eta[l][q, ..., w]
                if l == 0:
                    Tq = sum(_at(T[q], w, j, ml, nl) for j in range(6)) / 6
                    dirn = sum(s.s[q][a:a + ml, c:c + ml] for a, c in _LAT[w])
                    dirn = (dirn / dirn.norm(dim=-1, keepdim=True)).movedim(-1, 0)[..., None]
                for j in range(6):
                    _add(dg[:, q], w, j, ml, nl, V * e * ((g[j] ** 2).sum(0) + g[j] ** 2 / 3))
                    if l == 0:
                        _add(pm[q], w, j, ml, nl, V / e / 6)
                        _add(b[:, q], w, j, ml, nl, V / 6 * RA * Tq * dirn)
        dg = s.total(dg)
        dg[..., 0] = dg[..., -1] = 1.0
        diag.append(dg)
        if l == 0:
            mass = _Shell(m // 2, n // 2, dev).total(_to_coarse(pm))
            f = s.total(b)
            f[..., 0] = f[..., -1] = 0.0
    return eta, diag, mass, f


def _locate(sh, x):
    """(flat first lateral slot index triple, weights) of the triangle whose cone holds each point x [N, 3]:
    the twenty faces, then one refinement at a time."""
    m, s = sh.m, sh.s
    def coef(d, i, j, S, w):
        w1 = w == 1
        z = torch.zeros_like(i)
        a = s[d, torch.where(w1, i + S, i), torch.where(w1, j + S, j)]
        b = s[d, torch.where(w1, i, i + S), torch.where(w1, j + S, j)]
        c = s[d, torch.where(w1, i + S, i), torch.where(w1, j, j + S)]
        k = torch.stack([(x * torch.linalg.cross(b, c)).sum(-1), (x * torch.linalg.cross(c, a)).sum(-1),
                         (x * torch.linalg.cross(a, b)).sum(-1)], -1) / (a * torch.linalg.cross(b, c)).sum(-1)[:, None]
        lam = k.sum(-1)
        return torch.where(lam > 0, k.min(-1).values / lam, torch.full_like(lam, -1e300)), k, z
    N, dev = len(x), x.device
    zero = torch.zeros(N, dtype=torch.long, device=dev)
    best = torch.full((N,), -1e301, dtype=torch.float64, device=dev)
    d, w = zero.clone(), zero.clone()
    for q in range(10):
        for t in range(2):
            sc = coef(zero + q, zero, zero, m, zero + t)[0]
            up = sc > best
            best, d, w = torch.where(up, sc, best), torch.where(up, zero + q, d), torch.where(up, zero + t, w)
    i, j, S = zero.clone(), zero.clone(), m
    while S > 1:
        h, w1 = S // 2, w == 1
        kids = [(i + h * w1, j + h * w1, w), (i + h * ~w1, j + h * w1, w), (i + h * w1, j + h * ~w1, w),
                (i + h * w1, j + h * w1, 1 - w)]
        sc = torch.stack([coef(d, a, b, h, t)[0] for a, b, t in kids])
        at = sc.argmax(0)
        i, j, w = (torch.stack([k[c] for k in kids]).gather(0, at[None])[0] for c in range(3))
        S = h
    return d, i, j, w, coef(d, i, j, 1, w)[1]


def _interp(sh, where, f):
    d, i, j, w, k = where
    m1, n = sh.m + 1, sh.n
    lam = k.sum(-1)
    lat = k / lam[:, None]
    lam = lam.clamp(R_IN, R_OUT)
    h = (R_OUT - R_IN) / n
    kk = ((lam - R_IN) / h).floor().long().clamp(0, n - 1)
    t = (lam - R_IN) / h - kk
    v = torch.zeros_like(lam)
    off = torch.tensor(_LAT, device=lam.device)
    flat = f.reshape(-1)
    for a in range(3):
        at = ((d * m1 + i + off[w, a, 0]) * m1 + j + off[w, a, 1]) * (n + 1) + kk
        v += lat[:, a] * ((1 - t) * flat[at] + t * flat[at + 1])
    return v


def _exact_advect(case, d):
    sh, u, dt = d["shell"], d["u"], d["dt"]
    x = (sh.s[..., None, :] * sh.r[:, None]).reshape(-1, 3)
    uu = u.reshape(3, -1).T
    out = []
    for a in range(0, len(x), 1 << 19):
        xs = x[a:a + (1 << 19)]
        mid = _locate(sh, xs - 0.5 * dt * uu[a:a + (1 << 19)])
        um = torch.stack([_interp(sh, mid, u[c]) for c in range(3)], -1)
        out.append(_interp(sh, _locate(sh, xs - dt * um), d["T"]))
    return sh.same(torch.cat(out).reshape(sh.shape))


def exact(case, seed):
    kind = case["kind"]
    # a preconditioner cycle, a solve stopped after ten iterations, a step and a request
    # have no value of their own in 64 bits beside the iteration that makes them
    if kind in ("vcycle", "solve", "step", "serve"):
        return None
    d = _inputs(case, seed)
    return {"apply": _exact_apply, "energy": _exact_energy, "fields": _exact_fields, "advect": _exact_advect}[kind](case, d)
