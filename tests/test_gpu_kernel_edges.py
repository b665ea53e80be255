"""GPU parity of the kernels that gather over a node's ring of triangles and of the small
fused kernels of the solver, at the edges of their decompositions: the smallest shells
(every node next to a five-ring vertex), radial counts around the tiles and the workgroup
sizes, and the largest radial counts of the streamed kernels."""
import numpy as np
import pytest
import scipy.sparse as sp
import scipy.sparse.linalg as spla

import synthetic
from oracle.mesh import ShellMesh
from oracle.solver_ref import chebyshev, lumped_pressure_mass, velocity_prolongation
from oracle.stokes import StokesOracle, buoyancy_rhs, element_matrices, element_matrices_hg
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


_cache = {}


def shell(tng, ctx, mt, nr, levels=2):
    """(mesh, oracle meshes, layout maps, viscosity, oracle) of one (mt, nr) shell."""
    if (mt, nr) not in _cache:
        mesh = tng.Mesh(ctx, mt, nr, levels=levels)
        om = ShellMesh(mt, nr)
        omp = ShellMesh(mt // 2, nr // 2, hierarchy=om.h)
        lm, lmp = LayoutMap(*mesh.coords(0), om), LayoutMap(*mesh.coords(1), omp)
        eta, _, _ = synthetic.uniform_operator_inputs(om.n_wedges, om.n_nodes, omp.n_nodes, 3)
        _cache[(mt, nr)] = (mesh, om, omp, lm, lmp, eta, StokesOracle(mt, nr, eta, hierarchy=om.h))
    return _cache[(mt, nr)]


# one radial cell pair; layers around the pressure-mass tile (16 coarse layers) and the
# 256 threads of a workgroup; several workgroups per level
RING_SHELLS = [(2, 2), (4, 30), (4, 34), (2, 258), (8, 62)]


@pytest.mark.parametrize("dtype,tol", [("float64", 1e-12), ("float32", 1e-6)])
@pytest.mark.parametrize("mt,nr", RING_SHELLS)
def test_diagonal_pressure_mass_buoyancy(tng, ctx, dtype, tol, mt, nr):
    """Sums of at most twelve (diagonal) or 128 (mass) positive terms formed in FP64: element-
    wise within 1e-12, in FP32 the rounding of the inputs and of the stored value (below
    1e-6).  The buoyancy cancels between wedges: held to the largest entry."""
    import torch
    dt = getattr(torch, dtype)
    mesh, om, omp, lm, lmp, eta, orc = shell(tng, ctx, mt, nr)
    eta_t = torch.tensor(eta[lm.wedge_index()], device="cuda").to(dt)
    d = torch.full((3,) + mesh.shape(0), float("nan"), dtype=dt, device="cuda")
    tng.diag_A(ctx, mesh, 0, eta_t, d)
    pm = torch.full(mesh.shape(1), float("nan"), dtype=dt, device="cuda")
    tng.pressure_mass(ctx, mesh, 0, eta_t, pm)
    T = synthetic.temperature(om.s, om.r, seed=3).ravel()
    f = torch.full((3,) + mesh.shape(0), float("nan"), dtype=dt, device="cuda")
    tng.rhs_buoyancy(ctx, mesh, 0, torch.tensor(lm.to_lib(T), device="cuda").to(dt), 1e5, f)
    torch.cuda.synchronize()
    want_d, want_m = orc.diag_A(), lumped_pressure_mass(orc, eta)
    want_f = buoyancy_rhs(om, T, 1e5)
    want_f[om.boundary_nodes()] = 0.0
    got_d = lm.from_lib(d.double().cpu().numpy(), check_dups=1e-15)
    got_m = lmp.from_lib(pm.double().cpu().numpy(), check_dups=1e-15)
    got_f = lm.from_lib(f.double().cpu().numpy(), check_dups=1e-15)
    assert (np.abs(got_d - want_d) <= tol * np.abs(want_d)).all()
    assert (np.abs(got_m - want_m) <= tol * np.abs(want_m)).all()
    assert np.abs(got_f - want_f).max() <= 10 * tol * np.abs(want_f).max()


# unknowns of the coarsest level: 126 (a part of a pivot block left over), 252 and 486, and
# 1008 (the largest that the refinement leaves below the limit of 1024)
@pytest.mark.parametrize("mt,nr", [(4, 4), (4, 6), (8, 4), (4, 18)])
def test_coarse_correction(tng, ctx, mt, nr):
    """A V-cycle without smoothing is P A_c^-1 P^T: assembly, blocked inverse and solve of the
    coarsest level against the oracle's sparse solve, to 1e-10 (the matrix's condition number,
    below 1e4 on these shells, times 50 roundings)."""
    import torch
    mesh, om, omp, lm, lmp, eta, orc = shell(tng, ctx, mt, nr)
    eta_t = torch.tensor(eta[lm.wedge_index()], device="cuda")
    eta_c = torch.empty(mesh.wedge_shape(1), dtype=torch.float64, device="cuda")
    tng.eta_coarsen(ctx, mesh, 0, eta_t, eta_c)
    ec = np.empty(omp.n_wedges)
    ec[lmp.wedge_index().ravel()] = eta_c.cpu().numpy().ravel()
    s = tng.StokesSolver(ctx, mesh, mixed=0, levels=2, pre=0, post=0)
    s.setup(eta_t)
    b = np.random.default_rng(6).standard_normal((om.n_nodes, 3))
    b[om.boundary_nodes()] = 0.0
    bt = torch.tensor(lm.to_lib(b), device="cuda").contiguous()
    x = torch.full_like(bt, float("nan"))
    s.vcycle(bt, x)
    torch.cuda.synchronize()
    P = velocity_prolongation(orc)
    wn = omp.wedge_nodes()
    dof = (wn[:, :, None] * 3 + np.arange(3)).reshape(len(wn), 18)
    A = sp.csr_matrix((element_matrices(omp.node_xyz()[wn], ec).ravel(),
                       (np.repeat(dof, 18, axis=1).ravel(), np.tile(dof, (1, 18)).ravel())))
    inner = np.setdiff1d(np.arange(3 * omp.n_nodes),
                         (3 * np.flatnonzero(omp.boundary_nodes())[:, None] + np.arange(3)).ravel())
    c = np.zeros(3 * omp.n_nodes)
    c[inner] = spla.spsolve(A[inner][:, inner].tocsc(), (P.T @ b.ravel())[inner])
    want = (P @ c).reshape(-1, 3)
    got = lm.from_lib(x.cpu().numpy(), check_dups=1e-13)
    assert np.linalg.norm(got - want) <= 1e-10 * np.linalg.norm(want)


# gathered smoother: the smallest shell, 62-node blocks around the columns (62, 63 and 64
# layers) and several blocks; with hourglass control (hg) the streaming apply and its update
@pytest.mark.parametrize("dtype,tol", [("float64", 1e-12), ("float32", 1e-5)])
@pytest.mark.parametrize("mt,nr,degree,hg", [(2, 2, 2, 0.0), (4, 61, 2, 0.0), (4, 62, 3, 0.0), (8, 63, 1, 0.0),
                                             (16, 12, 2, 0.0), (16, 12, 2, 0.1), (8, 62, 3, 0.1)])
def test_smoother(tng, ctx, dtype, tol, mt, nr, degree, hg):
    """Two Chebyshev steps against the textbook iteration on the assembled operator, also with
    non-zero boundary velocities (their columns are dropped, their rows are identity)."""
    import torch
    dt = getattr(torch, dtype)
    mesh = tng.Mesh(ctx, mt, nr, levels=1)
    om = ShellMesh(mt, nr)
    lm = LayoutMap(*mesh.coords(0), om)
    eta = 10.0 ** np.random.default_rng(5).uniform(-1.0, 1.0, om.n_wedges)
    wn = om.wedge_nodes()
    dof = (wn[:, :, None] * 3 + np.arange(3)).reshape(len(wn), 18)
    A = sp.csr_matrix((element_matrices_hg(om.node_xyz()[wn], eta, hg).ravel(),
                       (np.repeat(dof, 18, axis=1).ravel(), np.tile(dof, (1, 18)).ravel())))
    keep = sp.diags(np.repeat(~om.boundary_nodes(), 3).astype(np.float64))
    A = (keep @ A @ keep + sp.identity(A.shape[0]) - keep).tocsr()
    rng = np.random.default_rng(4)
    b, x = rng.standard_normal((2, om.n_nodes, 3))
    eta_t = torch.tensor(eta[lm.wedge_index()], device="cuda").to(dt)
    d = torch.empty((3,) + mesh.shape(0), dtype=dt, device="cuda")
    tng.diag_A(ctx, mesh, 0, eta_t, d, hg_alpha=hg)
    lib = [torch.tensor(lm.to_lib(v), device="cuda").to(dt).contiguous() for v in (b, x)]
    tng.smooth(ctx, mesh, 0, eta_t, d, lib[0], lib[1], degree, 2, 0.3, 3.3, hg_alpha=hg)
    torch.cuda.synchronize()
    want = chebyshev(A, A.diagonal(), b.ravel(), x.ravel(), degree, 2, 0.3, 3.3).reshape(-1, 3)
    got = lm.from_lib(lib[1].double().cpu().numpy(), check_dups=tol)
    assert np.linalg.norm(got - want) <= tol * np.linalg.norm(want)


@pytest.mark.parametrize("dtype,tol", [("float64", 1e-13), ("float32", 1e-6)])
@pytest.mark.parametrize("mt,nr", [(2, 2), (4, 6), (2, 130), (8, 62)])
def test_transfers(tng, ctx, dtype, tol, mt, nr):
    """Restriction over the fine ring and prolongation against the oracle's P: weighted sums of
    at most 21 values, in FP32 a few roundings of 6e-8."""
    import torch
    dt = getattr(torch, dtype)
    mesh, om, omp, lm, lmp, eta, orc = shell(tng, ctx, mt, nr)
    rng = np.random.default_rng(3)
    f, c = rng.standard_normal((om.n_nodes, 3)), rng.standard_normal((omp.n_nodes, 3))
    ct = torch.full((3,) + mesh.shape(1), float("nan"), dtype=dt, device="cuda")
    ft = torch.full((3,) + mesh.shape(0), float("nan"), dtype=dt, device="cuda")
    tng.restrict(ctx, mesh, 0, torch.tensor(lm.to_lib(f), device="cuda").to(dt).contiguous(), ct)
    tng.prolong(ctx, mesh, 0, torch.tensor(lmp.to_lib(c), device="cuda").to(dt).contiguous(), ft)
    torch.cuda.synchronize()
    P = velocity_prolongation(orc)
    want_c = (P.T @ f.ravel()).reshape(-1, 3)
    want_c[omp.boundary_nodes()] = 0.0
    want_f = (P @ c.ravel()).reshape(-1, 3)
    got_c = lmp.from_lib(ct.double().cpu().numpy(), check_dups=1e-15)
    got_f = lm.from_lib(ft.double().cpu().numpy(), check_dups=1e-15)
    assert np.linalg.norm(got_c - want_c) <= tol * np.linalg.norm(want_c)
    assert np.linalg.norm(got_f - want_f) <= tol * np.linalg.norm(want_f)


# one refinement step and more, points beyond both spheres and several cells away (the flow
# crosses diamond edges and five-ring vertices)
@pytest.mark.parametrize("mt,nr,dt", [(2, 3, 2e-3), (8, 5, 5e-3), (16, 7, 2e-3)])
def test_advection(tng, ctx, mt, nr, dt):
    """Departure points by descent against the oracle's brute-force location: the interpolant is
    continuous across wedges, so rounding at an edge stays rounding (1e-12 of max |T| = 1)."""
    import torch
    from oracle.mmoc import departure_points, interpolate
    mesh = tng.Mesh(ctx, mt, nr, levels=1)
    om = ShellMesh(mt, nr)
    lm = LayoutMap(*mesh.coords(0), om)
    rng = np.random.default_rng(8)
    u = 30.0 * rng.standard_normal((om.n_nodes, 3))
    T = rng.uniform(0.0, 1.0, om.n_nodes)
    out = torch.full(mesh.shape(0), float("nan"), dtype=torch.float64, device="cuda")
    tng.mmoc_advect(ctx, mesh, 0, torch.tensor(lm.to_lib(u), device="cuda").contiguous(), dt,
                    torch.tensor(lm.to_lib(T), device="cuda"), out)
    torch.cuda.synchronize()
    want = interpolate(om, T, departure_points(om, u, dt))
    assert np.abs(lm.from_lib(out.cpu().numpy(), check_dups=1e-15) - want).max() <= 1e-12


# full operator and viscous block gathered per node: the smallest shell (five-rings, one
# coarse cell), 62-node blocks around the columns, remainders of the four coarse nodes a
# workgroup takes
@pytest.mark.parametrize("dtype,tol", [("float64", 1e-13), ("float32", 3e-6)])
@pytest.mark.parametrize("mt,nr", [(2, 2), (4, 30), (4, 34), (2, 258), (8, 62)])
def test_small_apply(tng, ctx, dtype, tol, mt, nr):
    """Gathered in one launch against the assembled operator, with Dirichlet rows and without
    them, element-wise on the row's term magnitudes: sums of at most 72 wedge terms of some
    50 roundings each (1e-13 in FP64, 3e-6 in FP32)."""
    import torch
    dt = getattr(torch, dtype)
    mesh, om, omp, lm, lmp, eta, orc = shell(tng, ctx, mt, nr)
    rng = np.random.default_rng(9)
    u, p = rng.uniform(-1, 1, (om.n_nodes, 3)), rng.uniform(-1, 1, omp.n_nodes)
    eta_t = torch.tensor(eta[lm.wedge_index()], device="cuda").to(dt)
    ut = torch.tensor(lm.to_lib(u), device="cuda").to(dt).contiguous()
    pt = torch.tensor(lmp.to_lib(p), device="cuda").to(dt).contiguous()
    K = tng.OP_A | tng.OP_BT | tng.OP_B
    nu = 3 * om.n_nodes
    for flags, A, BT, B in ((K | tng.OP_DIRICHLET, orc.A_D, orc.BT_D, orc.B_D), (K, orc.A, orc.B.T, orc.B),
                            (tng.OP_A | tng.OP_DIRICHLET, orc.A_D, None, None), (tng.OP_A, orc.A, None, None)):
        yu, yp = torch.full_like(ut, float("nan")), torch.full_like(pt, float("nan"))
        full = BT is not None
        tng.stokes_apply(ctx, mesh, 0, flags, eta_t, ut, pt if full else None, yu, yp if full else None)
        torch.cuda.synchronize()
        M = sp.bmat([[A, BT], [B, None]], format="csr") if full else A
        x = np.concatenate([u.ravel(), p]) if full else u.ravel()
        want, scale = M @ x, abs(M) @ np.abs(x)
        got = lm.from_lib(yu.double().cpu().numpy(), check_dups=1e-15).ravel()
        if full:
            got = np.concatenate([got, lmp.from_lib(yp.double().cpu().numpy(), check_dups=tol)])
        assert len(got) == (nu + omp.n_nodes if full else nu)
        assert (np.abs(got - want) <= tol * scale).all(), (flags, (np.abs(got - want) / scale).max())


# the streaming apply on the shells that the gathered form takes by default: columns of one
# to several radial stretches and ranges, unequal bands
@pytest.mark.parametrize("dtype,tol", [("float64", 1e-12), ("float32", 1e-5)])
@pytest.mark.parametrize("mt,nr,bands", [(4, 96, 1), (4, 160, 2), (4, 320, 1), (8, 62, 3)])
def test_streaming_apply(tng, ctx, dtype, tol, mt, nr, bands):
    import torch
    dt = getattr(torch, dtype)
    mesh, om, omp, lm, lmp, eta, orc = shell(tng, ctx, mt, nr)
    rng = np.random.default_rng(10)
    u, p = rng.uniform(-1, 1, (om.n_nodes, 3)), rng.uniform(-1, 1, omp.n_nodes)
    ut = torch.tensor(lm.to_lib(u), device="cuda").to(dt).contiguous()
    pt = torch.tensor(lmp.to_lib(p), device="cuda").to(dt).contiguous()
    yu, yp = torch.full_like(ut, float("nan")), torch.full_like(pt, float("nan"))
    ctx.set_apply_bands(bands)
    try:
        tng.stokes_apply(ctx, mesh, 0, tng.OP_A | tng.OP_BT | tng.OP_B | tng.OP_DIRICHLET,
                         torch.tensor(eta[lm.wedge_index()], device="cuda").to(dt), ut, pt, yu, yp)
        torch.cuda.synchronize()
    finally:
        ctx.set_apply_bands(0)
    ru, rp = orc.apply(u, p)
    gu, gp = lm.from_lib(yu.double().cpu().numpy()), lmp.from_lib(yp.double().cpu().numpy())
    assert np.linalg.norm(gu - ru) <= tol * np.linalg.norm(ru) and np.linalg.norm(gp - rp) <= tol * np.linalg.norm(rp)
