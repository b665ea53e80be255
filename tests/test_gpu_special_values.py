"""Infinities and the largest finite values in the field kernels: they reach the nodes whose
sums hold them, as the sums of the definitions do, and no others."""
import numpy as np
import pytest

from oracle.mesh import ShellMesh
from tests._support import LayoutMap

pytestmark = pytest.mark.gpu

SHELLS = [(4, 6), (8, 62)]


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


def shell(tng, ctx, mt, nr):
    """(mesh, oracle mesh, layout map, unique lateral ids of both levels)."""
    if (mt, nr) not in _cache:
        mesh = tng.Mesh(ctx, mt, nr, levels=2)
        om = ShellMesh(mt, nr)
        _cache[(mt, nr)] = (mesh, om, LayoutMap(*mesh.coords(0), om),
                            [np.asarray(mesh.unique_ids(l)).ravel() for l in range(2)])
    return _cache[(mt, nr)]


def to_fine(c):
    """W1 interpolation of node fields [..., 10, m+1, m+1, n+1] to the next finer level, in FP64."""
    for ax in (-3, -2, -1):
        s = list(c.shape)
        s[ax] = 2 * s[ax] - 1
        f = np.empty(s)
        ix = lambda sl: tuple([Ellipsis] + [sl if a == ax else slice(None) for a in (-3, -2, -1)])
        lo, hi = c[ix(slice(None, -1))], c[ix(slice(1, None))]
        f[ix(slice(None, None, 2))] = c
        f[ix(slice(1, None, 2))] = 0.5 * lo + 0.5 * hi
        if ax == -2:
            # the centre of a coarse quad is the midpoint of its split diagonal
            odd = f[..., 1::2, 1::2, :]
            odd[:] = 0.5 * c0[..., 1:, :-1, :] + 0.5 * c0[..., :-1, 1:, :]
        if ax == -3:
            c0 = c
        c = f
    return c


@pytest.mark.parametrize("dtype,tol", [("float64", 1e-14), ("float32", 1e-6)])
@pytest.mark.parametrize("mt,nr", SHELLS)
def test_prolongation_of_the_largest_values(tng, ctx, dtype, tol, mt, nr):
    """Masks of the type's lowest and largest value: coarse nodes are copied to the bit and the
    mean of such a value and an ordinary one is finite (a few roundings)."""
    import torch
    dt = getattr(torch, dtype)
    mesh, om, lm, uid = shell(tng, ctx, mt, nr)
    rng = np.random.default_rng(1)
    c = rng.uniform(-1.0, 1.0, (3, uid[1].max() + 1, nr // 2 + 1))
    big = float(torch.finfo(dt).max)
    for comp, node, k, v in ((0, 0, 1, -big), (1, uid[1][1], 2, big), (2, uid[1].max(), 0, -big), (0, 7, nr // 2, big)):
        c[comp, node, k] = v
    ct = torch.tensor(c[:, uid[1]].reshape((3,) + mesh.shape(1)), device="cuda").to(dt).contiguous()
    f = torch.full((3,) + mesh.shape(0), float("nan"), dtype=dt, device="cuda")
    tng.prolong(ctx, mesh, 0, ct, f)
    torch.cuda.synchronize()
    assert torch.equal(f[:, :, ::2, ::2, ::2], ct)
    want = to_fine(ct.double().cpu().numpy())
    assert (np.abs(f.double().cpu().numpy() - want) <= tol * np.maximum(1.0, np.abs(want))).all()


# a wedge at a five-ring vertex, one with an edge on a diamond's boundary, one inside
@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("form", ["one point", "hourglass", "two points"])
@pytest.mark.parametrize("cell", [(0, 0, 0, 1, 0), (3, 1, 0, 2, 1), (9, 1, 2, 3, 0)])
@pytest.mark.parametrize("mt,nr", SHELLS)
def test_diagonal_with_an_infinite_viscosity(tng, ctx, dtype, form, cell, mt, nr):
    """Infinite at the wedge's nodes (positive terms), the same bits elsewhere."""
    import torch
    dt = getattr(torch, dtype)
    mesh, om, lm, uid = shell(tng, ctx, mt, nr)
    eta = torch.tensor(np.random.default_rng(2).uniform(0.5, 1.5, mesh.wedge_shape(0)), device="cuda").to(dt)
    kw = {"hg_alpha": 0.1} if form == "hourglass" else {"twopoint": form == "two points"}
    out = []
    for v in (1.0, float("inf")):
        eta[cell] = v
        d = torch.full((3,) + mesh.shape(0), float("nan"), dtype=dt, device="cuda")
        tng.diag_A(ctx, mesh, 0, eta, d, **kw)
        torch.cuda.synchronize()
        out.append(d.cpu().numpy())
    q, i, j, k, w = cell
    m1 = mt + 1
    lat = [(q * m1 + i + a) * m1 + j + b for a, b in (((0, 0), (1, 0), (0, 1)), ((1, 1), (0, 1), (1, 0)))[w]]
    hit = np.isin(uid[0], uid[0][lat]).reshape(10, m1, m1)[..., None] & np.isin(np.arange(nr + 1), (k, k + 1))
    assert (out[1][:, hit] == np.inf).all()
    assert np.array_equal(out[1][:, ~hit], out[0][:, ~hit])


@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("at", ["vertex", "neighbour"])
@pytest.mark.parametrize("mt,nr", SHELLS)
def test_buoyancy_of_an_infinite_temperature(tng, ctx, dtype, at, mt, nr):
    """Around the five-ring vertex on the z axis every direction has a positive z component: the
    force there is infinite at the nodes of the wedges that hold the node, finite elsewhere."""
    import torch
    dt = getattr(torch, dtype)
    mesh, om, lm, uid = shell(tng, ctx, mt, nr)
    slot = 0 if at == "vertex" else 1          # (0, 0) of diamond 0 and the next node along j
    node, k = lm.slot2lat[slot], 2
    T = np.random.default_rng(3).uniform(0.0, 1.0, (om.n_lat, nr + 1))
    T[node, k] = np.inf
    f = torch.full((3,) + mesh.shape(0), float("nan"), dtype=dt, device="cuda")
    tng.rhs_buoyancy(ctx, mesh, 0, torch.tensor(lm.to_lib(T.ravel()), device="cuda").to(dt), 1e5, f)
    torch.cuda.synchronize()
    near = np.unique(om.tris[(om.tris == node).any(axis=1)])
    hit = np.zeros((om.n_lat, nr + 1), bool)
    hit[near, k - 1:k + 2] = True
    hit[:, [0, -1]] = False                    # no-slip rows are zero
    fz = lm.from_lib(f[2].double().cpu().numpy()).reshape(om.n_lat, nr + 1)
    assert (fz[hit] == np.inf).all()
    assert np.isfinite(lm.from_lib(f.double().cpu().numpy())[~hit.ravel()]).all()
