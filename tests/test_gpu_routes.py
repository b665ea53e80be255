"""Which kernels a call takes, and parity of the ones that the default choice leaves to larger
shells than the oracle's: small levels gather per node unless a band count is forced."""
import time

import numpy as np
import pytest
import scipy.sparse as sp
import scipy.sparse.linalg as spla

import synthetic
from oracle.mesh import ShellMesh
from oracle.solver_ref import chebyshev, velocity_prolongation
from oracle.stokes import (StokesOracle, boundary_projections, element_matrices, element_matrices_2pt,
                           element_matrices_hg)
from tests._support import LayoutMap

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tng():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_21633_amd as t
    return t


@pytest.fixture(scope="module")
def ctx(tng):
    return tng.Context(0)


@pytest.fixture
def profiled(ctx):
    """The context with event timers on; band count and timers are reset afterwards."""
    ctx.profile(True)
    yield ctx
    ctx.profile(False)
    ctx.set_apply_bands(0)


_cache = {}


def shell(tng, ctx, mt, nr, levels=2):
    """(mesh, oracle mesh, layout maps, viscosity, oracle) of one (mt, nr) shell."""
    key = (mt, nr, levels)
    if key not in _cache:
        mesh = tng.Mesh(ctx, mt, nr, levels=levels)
        om = ShellMesh(mt, nr)
        omp = ShellMesh(mt // 2, nr // 2, hierarchy=om.h)
        lm, lmp = LayoutMap(*mesh.coords(0), om), LayoutMap(*mesh.coords(1), omp)
        eta, _, _ = synthetic.uniform_operator_inputs(om.n_wedges, om.n_nodes, omp.n_nodes, 3)
        _cache[key] = (mesh, om, omp, lm, lmp, eta, StokesOracle(mt, nr, eta, hierarchy=om.h))
    return _cache[key]


def smoother_case(tng, ctx, mt, nr, dt):
    """(mesh, om, layout map, A_D, viscosity, diagonal, [b, x] of the oracle, [b, x] of the library)."""
    import torch
    mesh = tng.Mesh(ctx, mt, nr, levels=1)
    om = ShellMesh(mt, nr)
    lm = LayoutMap(*mesh.coords(0), om)
    rng = np.random.default_rng(5)
    eta = 10.0 ** rng.uniform(-1.0, 1.0, om.n_wedges)
    wn = om.wedge_nodes()
    dof = (wn[:, :, None] * 3 + np.arange(3)).reshape(len(wn), 18)
    A = sp.csr_matrix((element_matrices(om.node_xyz()[wn], eta).ravel(),
                       (np.repeat(dof, 18, axis=1).ravel(), np.tile(dof, (1, 18)).ravel())))
    keep = sp.diags(np.repeat(~om.boundary_nodes(), 3).astype(np.float64))
    A = (keep @ A @ keep + sp.identity(A.shape[0]) - keep).tocsr()
    bx = rng.standard_normal((2, om.n_nodes, 3))
    eta_t = torch.tensor(eta[lm.wedge_index()], device="cuda").to(dt)
    d = torch.empty((3,) + mesh.shape(0), dtype=dt, device="cuda")
    tng.diag_A(ctx, mesh, 0, eta_t, d)
    lib = [torch.tensor(lm.to_lib(v), device="cuda").to(dt).contiguous() for v in bx]
    return mesh, om, lm, A, eta_t, d, bx, lib


def applies(ctx):
    """{"<variant>/<m>x<n>/<form>": launches} of the timed operator kernels, over both precisions."""
    out = {}
    for name, (_, n) in ctx.kernel_stats_all().items():
        if name.startswith("stokes_apply/"):
            key = name.split("/", 2)[2]
            out[key] = out.get(key, 0) + n
    return out


# the streaming apply and its fused Chebyshev update on shells that gather by default: one
# radial stretch and two, one band and several, an odd band count
@pytest.mark.parametrize("dtype,tol", [("float64", 1e-12), ("float32", 1e-5)])
@pytest.mark.parametrize("mt,nr,degree,bands", [(4, 61, 2, 1), (8, 62, 3, 3), (4, 130, 1, 2), (16, 12, 2, 5)])
def test_forced_bands_stream_the_smoother(tng, profiled, dtype, tol, mt, nr, degree, bands):
    """Two steps against the textbook iteration on the assembled operator (bounds of the gathered
    form's test: a few hundred roundings), every operator apply in the forced decomposition."""
    import torch
    mesh, om, lm, A, eta_t, d, (b, x), lib = smoother_case(tng, profiled, mt, nr, getattr(torch, dtype))
    profiled.set_apply_bands(bands)
    tng.smooth(profiled, mesh, 0, eta_t, d, lib[0], lib[1], degree, 2, 0.3, 3.3)
    torch.cuda.synchronize()
    want = chebyshev(A, A.diagonal(), b.ravel(), x.ravel(), degree, 2, 0.3, 3.3).reshape(-1, 3)
    got = lm.from_lib(lib[1].double().cpu().numpy(), check_dups=tol)
    assert np.linalg.norm(got - want) <= tol * np.linalg.norm(want)
    assert applies(profiled) == {f"A/{mt}x{nr}/b{bands}": 2 * degree}


@pytest.mark.parametrize("mixed", [0, 1])
def test_forced_bands_stream_the_solve(tng, profiled, mixed):
    """Residuals and power iterations too: a whole solve without a gathered apply, against the
    sparse direct solve (relative residual 1e-10: 1e-7 on the solution, as by default)."""
    import torch
    mesh, om, omp, lm, lmp, eta, orc = shell(tng, profiled, 8, 8, levels=3)
    f = np.random.default_rng(9).standard_normal((om.n_nodes, 3))
    f[om.boundary_nodes()] = 0.0
    profiled.set_apply_bands(2)
    s = tng.StokesSolver(profiled, mesh, mixed=mixed, rtol=1e-10, max_iters=400)
    u = torch.empty((3,) + mesh.shape(0), dtype=torch.float64, device="cuda")
    p = torch.empty(mesh.shape(1), dtype=torch.float64, device="cuda")
    s.solve(torch.tensor(lm.to_lib(f), device="cuda").contiguous(), None, u, p,
            eta=torch.tensor(eta[lm.wedge_index()], device="cuda"))
    uo, po = orc.solve(f)
    gu, gp = lm.from_lib(u.cpu().numpy(), check_dups=1e-12), lmp.from_lib(p.cpu().numpy(), check_dups=1e-12)
    assert np.linalg.norm(gu - uo) <= 1e-7 * np.linalg.norm(uo)
    assert np.linalg.norm(gp - po) <= 1e-7 * np.linalg.norm(po)
    seen = applies(profiled)
    assert all("/ring" not in k for k in seen) and {"A/8x8/b2", "A/4x4/b2", "K/8x8/b2"} <= set(seen), seen
    s.close()


# levels that gather: the smoother, its residual and the power iteration are timed like the
# applies of the streaming form
@pytest.mark.parametrize("dtype", ["float64", "float32"])
def test_gathered_smoother_is_timed(tng, profiled, dtype):
    import torch
    mesh, om, lm, A, eta_t, d, bx, lib = smoother_case(tng, profiled, 4, 6, getattr(torch, dtype))
    tng.smooth(profiled, mesh, 0, eta_t, d, lib[0], lib[1], 2, 3, 0.3, 3.3)
    assert applies(profiled) == {"A/4x6/ring": 6}
    ms, n = profiled.kernel_stats("stokes_apply")
    assert n == 6 and ms > 0.0


def test_gathered_solver_applies_are_timed(tng, profiled):
    """Set-up: power_its applies on each smoothed level; a V-cycle from zero: per level one apply
    less than degree times steps before the coarse correction, the residual, and degree times
    steps after it."""
    import torch
    mesh = shell(tng, profiled, 8, 8, levels=3)[0]
    s = tng.StokesSolver(profiled, mesh, mixed=0, pre=1, post=2, cheb_degree=2, power_its=5)
    s.setup(torch.ones(mesh.wedge_shape(0), dtype=torch.float64, device="cuda"))
    assert applies(profiled) == {"A/8x8/ring": 5, "A/4x4/ring": 5}
    profiled.profile(True)
    b = torch.ones((3,) + mesh.shape(0), dtype=torch.float64, device="cuda")
    s.vcycle(b, torch.empty_like(b))
    assert applies(profiled) == {"A/8x8/ring": 6, "A/4x4/ring": 6}
    s.close()


# the viscous block alone in FP64: columns of one stretch stream above 14,000 slots a cell row
@pytest.mark.parametrize("mt,nr,form", [(32, 38, "ring"), (32, 44, "stream"), (64, 8, "ring"), (16, 64, "ring"),
                                        (16, 160, "ring")])
def test_form_of_the_viscous_block(tng, profiled, mt, nr, form):
    import torch
    mesh = tng.Mesh(profiled, mt, nr, levels=1)
    g = torch.Generator(device="cuda").manual_seed(1)
    eta = 0.5 + torch.rand(mesh.wedge_shape(0), generator=g, dtype=torch.float64, device="cuda")
    u = torch.ones((3,) + mesh.shape(0), dtype=torch.float64, device="cuda") * torch.rand(
        nr + 1, generator=g, dtype=torch.float64, device="cuda")      # the same in all copies
    y = [torch.full_like(u, float("nan")) for _ in range(2)]
    tng.stokes_apply(profiled, mesh, 0, tng.OP_A | tng.OP_DIRICHLET, eta, u, None, y[0], None)
    assert [k.rstrip("0123456789") for k in applies(profiled)] == [f"A/{mt}x{nr}/" + ("ring" if form == "ring" else "b")]
    profiled.set_apply_bands(3)
    tng.stokes_apply(profiled, mesh, 0, tng.OP_A | tng.OP_DIRICHLET, eta, u, None, y[1], None)
    assert float((y[0] - y[1]).abs().max()) <= 1e-13 * float(y[1].abs().max())


def viscous_block(om, eta, u, dirichlet):
    """A u (A_D u) in extended precision, wedge by wedge: on thin layers the assembled FP64 matrix is
    itself off by the roundoff over the layer's thickness (2e-13 on 320 layers)."""
    ld = np.longdouble
    m, wn = om.nr, om.wedge_nodes()
    r = ld(0.55) + (ld(1.0) - ld(0.55)) * np.arange(m + 1) / ld(m)
    x = (om.s.astype(ld)[:, None] * r[None, :, None]).reshape(-1, 3)[wn]          # [wedge, node, 3]
    third, half = ld(1) / 3, ld(1) / 2
    dn = np.array([[-half, -half, -third / 2], [half, 0, -third / 2], [0, half, -third / 2],
                   [-half, -half, third / 2], [half, 0, third / 2], [0, half, third / 2]], dtype=ld)
    J = [(x * dn[None, :, k, None]).sum(1) for k in range(3)]                     # dx/dxi_k
    c = [np.cross(J[1], J[2]), np.cross(J[2], J[0]), np.cross(J[0], J[1])]
    det = (J[0] * c[0]).sum(1)
    g = sum(dn[None, :, k, None] * c[k][:, None] for k in range(3)) / det[:, None, None]
    bnd = om.boundary_nodes()
    v = u.astype(ld)
    if dirichlet:
        v = np.where(bnd[:, None], ld(0), v)
    L = sum(v[wn[:, j]][:, :, None] * g[:, j][:, None] for j in range(6))         # [wedge, c, d]
    S = L + L.transpose(0, 2, 1) - 2 * third * np.trace(L, axis1=1, axis2=2)[:, None, None] * np.eye(3, dtype=ld)
    S *= (np.abs(det) * eta)[:, None, None]
    y = np.zeros((om.n_nodes, 3), dtype=ld)
    for j in range(6):
        np.add.at(y, wn[:, j], (S * g[:, j][:, None]).sum(2))
    return np.where(bnd[:, None], u, y) if dirichlet else y


# the streaming viscous block alone, as the smoother of a large level runs it: columns of one to
# several radial stretches and ranges, unequal bands
@pytest.mark.parametrize("dtype,tol", [("float64", 1e-13), ("float32", 3e-6)])
@pytest.mark.parametrize("mt,nr,bands", [(4, 96, 1), (4, 160, 2), (4, 320, 1), (8, 62, 3), (16, 12, 5)])
def test_streaming_viscous_block(tng, profiled, dtype, tol, mt, nr, bands):
    """Element-wise on the row's term magnitudes, with Dirichlet rows and without them (the bounds
    of the gathered form: sums of at most 72 wedge terms of some 50 roundings each)."""
    import torch
    dt = getattr(torch, dtype)
    mesh, om, omp, lm, lmp, eta, orc = shell(tng, profiled, mt, nr)
    u = np.random.default_rng(9).uniform(-1, 1, (om.n_nodes, 3))
    eta_t = torch.tensor(eta[lm.wedge_index()], device="cuda").to(dt)
    ut = torch.tensor(lm.to_lib(u), device="cuda").to(dt).contiguous()
    profiled.set_apply_bands(bands)
    for flags, M in ((tng.OP_A | tng.OP_DIRICHLET, orc.A_D), (tng.OP_A, orc.A)):
        y = torch.full_like(ut, float("nan"))
        tng.stokes_apply(profiled, mesh, 0, flags, eta_t, ut, None, y, None)
        torch.cuda.synchronize()
        got = lm.from_lib(y.double().cpu().numpy(), check_dups=1e-15).ravel()
        want = viscous_block(om, eta, u, bool(flags & tng.OP_DIRICHLET)).ravel()
        scale = abs(M) @ np.abs(u.ravel())
        assert (np.abs(got - want) <= tol * scale).all(), (flags, (np.abs(got - want) / scale).max())
    assert applies(profiled) == {f"A/{mt}x{nr}/b{bands}": 2}


@pytest.mark.parametrize("bands", [0, 2])
@pytest.mark.parametrize("mixed,smooth", [(0, 2), (1, 2), (0, 0)])
def test_vcycle_of_fields_laid_out_otherwise(tng, ctx, mixed, smooth, bands):
    """Separate tensors, components in another order, a base off the 16-byte grid, in place and
    overlapping: copied into the solver's layout first, so the bits are those of one [3, ...] field."""
    import torch
    dt = torch.float32 if mixed else torch.float64
    mesh, om, omp, lm, lmp, eta, orc = shell(tng, ctx, 8, 8, levels=3)
    b = np.random.default_rng(5).standard_normal((om.n_nodes, 3))
    b[om.boundary_nodes()] = 0.0
    b = torch.tensor(lm.to_lib(b), device="cuda").to(dt).contiguous()
    n = b[0].numel()
    ctx.set_apply_bands(bands)
    try:
        s = tng.StokesSolver(ctx, mesh, mixed=mixed, pre=smooth, post=smooth)
        s.setup(torch.tensor(eta[lm.wedge_index()], device="cuda"))
        want = torch.full_like(b, float("nan"))
        s.vcycle(b, want)
        room = torch.empty(8 * n + 8, dtype=dt, device="cuda")

        def field(*starts):
            return [room[q:q + n].view(b[0].shape) for q in starts]
        layouts = {
            "separate": (field(0, n + 4, 2 * n + 8), field(4 * n, 5 * n + 4, 6 * n + 8)),
            "reversed": (field(2 * n, n, 0), field(6 * n, 5 * n, 4 * n)),
            "unaligned": (field(1, n + 1, 2 * n + 1), field(4 * n + 1, 5 * n + 1, 6 * n + 1)),
            "in place": (field(0, n, 2 * n), field(0, n, 2 * n)),
            "overlapping": (field(0, n, 2 * n), field(n, 2 * n, 3 * n)),
        }
        for what, (bb, xx) in layouts.items():
            room.fill_(float("nan"))
            for c in range(3):
                bb[c].copy_(b[c])
            s.vcycle(bb, xx)
            assert all(torch.equal(xx[c], want[c]) for c in range(3)), what
        s.close()
    finally:
        ctx.set_apply_bands(0)


# the other forms of the ring kernels at the edges of their decompositions (five-rings next to
# every node, layers around the workgroup's nodes)
@pytest.mark.parametrize("dtype,tol", [("float64", 1e-12), ("float32", 1e-6)])
@pytest.mark.parametrize("form", ["hourglass", "two points"])
@pytest.mark.parametrize("mt,nr", [(2, 2), (4, 30), (4, 34), (2, 258), (8, 62)])
def test_diagonal_of_the_other_forms(tng, ctx, dtype, tol, form, mt, nr):
    """Sums of at most 24 positive terms formed in FP64 (bounds as for the plain diagonal)."""
    import torch
    dt = getattr(torch, dtype)
    mesh, om, omp, lm, lmp, eta, _ = shell(tng, ctx, mt, nr)
    kw, okw = ({"hg_alpha": 0.3}, {"hg_alpha": 0.3}) if form == "hourglass" else ({"twopoint": True}, {"quad": "two"})
    d = torch.full((3,) + mesh.shape(0), float("nan"), dtype=dt, device="cuda")
    tng.diag_A(ctx, mesh, 0, torch.tensor(eta[lm.wedge_index()], device="cuda").to(dt), d, **kw)
    torch.cuda.synchronize()
    want = StokesOracle(mt, nr, eta, hierarchy=om.h, **okw).diag_A()
    got = lm.from_lib(d.double().cpu().numpy(), check_dups=1e-15)
    assert (np.abs(got - want) <= tol * np.abs(want)).all()


# unknowns of the coarsest level from 126 to 1008, as for the plain operator; free slip adds those
# of a sphere
@pytest.mark.parametrize("form", ["hourglass", "two points", "free slip outside", "free slip inside"])
@pytest.mark.parametrize("mt,nr", [(4, 4), (4, 6), (8, 4), (4, 16)])
def test_coarse_correction_of_the_other_forms(tng, ctx, form, mt, nr):
    """A V-cycle without smoothing is P A_c^-1 P^T, with free slip followed by the normal rows
    x <- P_s x + N_s b: assembly and inverse against a sparse solve of the same matrix, to 1e-10
    (condition numbers below 1e4 and 50 roundings)."""
    import torch
    mesh, om, omp, lm, lmp, eta, orc = shell(tng, ctx, mt, nr)
    bc = {"free slip outside": ("noslip", "freeslip"), "free slip inside": ("freeslip", "noslip")}.get(
        form, ("noslip", "noslip"))
    opts = {"hourglass": {"hg_alpha": 0.3}, "two points": {"op_flags": tng.OP_TWOPOINT},
            "free slip outside": {"op_flags": tng.OP_FREESLIP_OUTER},
            "free slip inside": {"op_flags": tng.OP_FREESLIP_INNER}}[form]
    eta_t = torch.tensor(eta[lm.wedge_index()], device="cuda")
    eta_c = torch.empty(mesh.wedge_shape(1), dtype=torch.float64, device="cuda")
    tng.eta_coarsen(ctx, mesh, 0, eta_t, eta_c)
    ec = np.empty(omp.n_wedges)
    ec[lmp.wedge_index().ravel()] = eta_c.cpu().numpy().ravel()
    s = tng.StokesSolver(ctx, mesh, mixed=0, levels=2, pre=0, post=0, **opts)
    s.setup(eta_t)
    b = np.random.default_rng(6).standard_normal((om.n_nodes, 3))
    layer = np.tile(np.arange(nr + 1), om.n_lat)
    for k, kind in ((0, bc[0]), (nr, bc[1])):
        if kind == "noslip":
            b[layer == k] = 0.0
    x = torch.full((3,) + mesh.shape(0), float("nan"), dtype=torch.float64, device="cuda")
    s.vcycle(torch.tensor(lm.to_lib(b), device="cuda").contiguous(), x)
    torch.cuda.synchronize()
    s.close()
    wn = omp.wedge_nodes()
    dof = (wn[:, :, None] * 3 + np.arange(3)).reshape(len(wn), 18)
    xw = omp.node_xyz()[wn]
    Ae = (element_matrices_hg(xw, ec, 0.3) if form == "hourglass" else
          element_matrices_2pt(xw, ec) if form == "two points" else element_matrices(xw, ec))
    A = sp.csr_matrix((Ae.ravel(), (np.repeat(dof, 18, axis=1).ravel(), np.tile(dof, (1, 18)).ravel())))
    Pc, Nc = boundary_projections(omp, bc)
    Pf, Nf = boundary_projections(om, bc)
    R = velocity_prolongation(orc)
    rhs = Pc @ (R.T @ b.ravel())
    want = R @ spla.spsolve((Pc @ A @ Pc + Nc).tocsc(), rhs)
    if "free slip" in form:
        want = Pf @ want + Nf @ b.ravel()
    want = want.reshape(-1, 3)
    got = lm.from_lib(x.cpu().numpy(), check_dups=1e-13)
    assert np.linalg.norm(got - want) <= 1e-10 * np.linalg.norm(want)


# batched launches of the streaming applies (the small shells of the server's other tests gather):
# the full operator on (32,32), also the viscous block and its fused passes on (64,64)
@pytest.mark.parametrize("mixed,tol", [(0, 1e-9), (1, 1e-4)])
@pytest.mark.parametrize("mt", [32, 64])
def test_batched_streaming_matches_single(tng, ctx, mt, mixed, tol):
    """Three requests in lockstep, each ten iterations: the result of the request alone, whose
    launches are not batched, up to their roundings (1e-16, in the FP32 inner solve 6e-8, grown at
    most a thousandfold over ten steps); in FP64 that of the single solver too, which scales its
    starting vector to the same bits."""
    import torch
    opts = dict(mixed=mixed, max_iters=10, max_outer=1, inner_max_iters=10, inner_rtol=1e-12, rtol=1e-13)
    srv = tng.Server(ctx, [(mt, mt)], budget_bytes=24 << 30, max_slots=3, **opts)
    mesh = tng.Mesh(ctx, mt, mt, levels=int(np.log2(mt)))
    xyz, r = mesh.coords(0)
    single = None if mixed else tng.StokesSolver(ctx, mesh, **opts)

    def rel(a, b):
        return float(np.max([float((x - y).norm() / y.norm()) for x, y in zip(a, b)]))   # NaN stays NaN

    def out():
        return (torch.empty((3,) + mesh.shape(0), dtype=torch.float64, device="cuda"),
                torch.empty(mesh.shape(1), dtype=torch.float64, device="cuda"))
    reqs = []
    for i in range(3):
        T = synthetic.temperature(xyz.reshape(-1, 3), r, seed=700 + i, lmin=1, lmax=8)
        Tt, alone = torch.tensor(T.reshape(mesh.shape(0)), device="cuda"), out()
        torch.cuda.synchronize()
        t = srv.submit(0, Tt, 1.0 + i, 1e5, *alone)
        srv.wait(t)
        assert srv.poll(t)["inner_its"] == 10
        if single:
            eta = torch.empty(mesh.wedge_shape(0), dtype=torch.float64, device="cuda")
            tng.eta_from_temperature(ctx, mesh, 0, Tt, (1.0 + i) * np.log(10.0), 0.0, eta)
            f, own = torch.empty_like(alone[0]), out()
            tng.rhs_buoyancy(ctx, mesh, 0, Tt, 1e5, f)
            assert single.solve(f, None, *own, eta=eta, raise_on_fail=False)["inner_its"] == 10
            assert rel(alone, own) <= tol
        reqs.append((Tt, 1.0 + i, alone, out()))
    torch.cuda.synchronize()
    # a pause of this thread between two submissions (a garbage collection) can outlast a solve, the
    # third then takes an idle slot: the group is sent again until all three ran at one time
    for attempt in range(20):
        for _, _, _, got in reqs:
            for x in got:
                x.fill_(float("nan"))
        torch.cuda.synchronize()
        sent = [(time.perf_counter(), srv.submit(0, Tt, lc, 1e5, *got)) for Tt, lc, _, got in reqs]
        srv.wait(0)
        infos = [srv.poll(t) for _, t in sent]
        for info, (_, lc, alone, got) in zip(infos, reqs):
            assert info["inner_its"] == 10
            d = rel(got, alone)
            print(f"({mt},{mt}) mixed={mixed} contrast 1e{lc:.0f}: in the batch against alone {d:.1e}", flush=True)
            assert d <= tol
        starts = [t0 + info["queue"] for (t0, _), info in zip(sent, infos)]
        ends = [t0 + info["latency"] for (t0, _), info in zip(sent, infos)]
        if srv.stats()["slots"] == 3 and max(starts) < min(ends):
            break
    else:
        raise AssertionError(f"never three at one time: {srv.stats()}, {infos}")
    if single:
        single.close()
    srv.close()
