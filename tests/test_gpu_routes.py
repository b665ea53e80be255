"""Which kernels a call takes, and parity of the ones that the default choice leaves to larger
shells than the oracle's: small levels gather per node unless a band count is forced."""
import numpy as np
import pytest
import scipy.sparse as sp

import synthetic
from oracle.mesh import ShellMesh
from oracle.solver_ref import chebyshev
from oracle.stokes import StokesOracle, element_matrices
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
