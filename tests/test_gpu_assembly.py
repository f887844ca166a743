"""GPU parity of assembly (the global residual, Section 2) and of the element
restriction, through the C ABI.

FP64 assembly adds the same values in the same order as the oracle
(increasing element order, from zero), so the two agree bit for bit; FP32
assembly is compared with the oracle's FP64 sum of the same FP32 values
relative to the sum of magnitudes at each vertex. The restriction is a copy
and must be exact.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_1607_04245_amd import api, meshgen as mg
from paper_1607_04245_amd import _native as N

from _parity import TOL, assert_close, dev, oracle_reference, rounded

pytestmark = pytest.mark.gpu

DTYPES = [torch.float32, torch.float64]


def grid_workload(dim, phys, n_elem, seed=31):
    grid = mg.smallest_grid(dim, max(n_elem, 1))
    return mg.make_workload(f"a{dim}{phys}", dim, phys, grid, n_elem, mg.BASE_SEED + seed)


def assemble_scale(dim, nc, nv, conn, R):
    """Per vertex and component: sum of |R| over its slots (bounds every
    partial sum of the assembly)."""
    return oracle.assemble(dim, nc, nv, conn, np.abs(R))


@pytest.mark.parametrize("dim,nc", [(2, 1), (2, 2), (3, 1), (3, 3)])
@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("n_elem", [1, 65, 3001])
def test_assemble_matches_oracle(dim, nc, dtype, n_elem):
    wl = grid_workload(dim, mg.LAPLACE, n_elem)
    rng = np.random.default_rng(n_elem + 7 * nc)
    R = rounded(rng.normal(size=((dim + 1) * nc, wl.n_elem)), dtype)
    conn = dev(wl.conn, torch.int32)
    plan = api.AssemblyPlan(conn, wl.n_vert)
    F = plan.assemble(dev(R, dtype), nc).cpu().numpy()
    ref = oracle.assemble(dim, nc, wl.n_vert, wl.conn, R)
    if dtype == torch.float64:
        assert np.array_equal(F, ref), "FP64 assembly must equal the oracle's element-order sum bit for bit"
    else:
        scale = assemble_scale(dim, nc, wl.n_vert, wl.conn, R)
        err = np.abs(F - ref) / np.maximum(scale, 1e-300)
        assert err.max() <= TOL[dtype], f"max scaled error {err.max():.2e}"
    # vertices no element touches (the truncated grid keeps them) are zero
    used = np.zeros(wl.n_vert, bool)
    used[wl.conn.ravel()] = True
    assert np.all(F[~used] == 0)
    plan.close()


@pytest.mark.parametrize("dtype", DTYPES)
def test_assemble_repeatable_and_plan_independent(dtype):
    wl = grid_workload(3, mg.ELASTICITY, 20000)
    conn = dev(wl.conn, torch.int32)
    R = dev(np.random.default_rng(3).normal(size=(12, wl.n_elem)), dtype)
    p1, p2 = api.AssemblyPlan(conn, wl.n_vert), api.AssemblyPlan(conn, wl.n_vert)
    F1 = p1.assemble(R, 3)
    for _ in range(3):
        assert torch.equal(p1.assemble(R, 3), F1)
    assert torch.equal(p2.assemble(R, 3), F1)


@pytest.mark.parametrize("dim,nc", [(2, 1), (2, 2), (3, 1), (3, 3)])
@pytest.mark.parametrize("dtype", DTYPES)
def test_restrict_is_the_closure(dim, nc, dtype):
    wl = grid_workload(dim, mg.LAPLACE, 5003)
    W = np.random.default_rng(5).normal(size=(wl.n_vert, nc))
    got = api.fem_restrict(dev(wl.conn, torch.int32), dev(W, dtype)).cpu().numpy()
    assert np.array_equal(got, rounded(mg.closure(wl.conn, W), dtype))


def test_restrict_bad_index_gives_nan():
    wl = grid_workload(2, mg.LAPLACE, 100)
    conn = wl.conn.copy()
    conn[7, 2] = wl.n_vert
    conn[9, 0] = -5
    got = api.fem_restrict(dev(conn, torch.int32), dev(wl.u_vertex, torch.float32)).cpu().numpy()
    assert np.isnan(got[2, 7]) and np.isnan(got[0, 9])
    good = np.ones(got.shape, bool)
    good[2, 7] = good[0, 9] = False
    assert np.array_equal(got[good], rounded(mg.closure(wl.conn, wl.u_vertex), torch.float32)[good])


def test_plan_rejects_bad_connectivity():
    wl = grid_workload(3, mg.LAPLACE, 500)
    conn = wl.conn.copy()
    conn[17, 1] = wl.n_vert + 3
    with pytest.raises(N.FemError) as ei:
        api.AssemblyPlan(dev(conn, torch.int32), wl.n_vert)
    assert ei.value.status == N.FEM_ERR_INVALID_ARG
    empty = api.AssemblyPlan(torch.zeros((0, 4), dtype=torch.int32, device="cuda"), 10)
    F = empty.assemble(torch.zeros((4, 0), device="cuda"), 1)
    assert F.shape == (10, 1) and torch.all(F == 0)


@pytest.mark.parametrize("dim,phys", [(2, mg.LAPLACE), (3, mg.LAPLACE), (2, mg.ELASTICITY), (3, mg.ELASTICITY)])
@pytest.mark.parametrize("dtype", DTYPES)
def test_global_residual_pipeline(dim, phys, dtype):
    """Vertex field -> gather form -> assembly against the oracle's residual
    and assembly on the same (rounded) inputs."""
    wl = grid_workload(dim, phys, 6000)
    nc = wl.n_comp
    coords, conn = dev(wl.coords, torch.float64), dev(wl.conn, torch.int32)
    R = api.fem_integrate_residual_gather(dim, phys, wl.rule, coords, conn, dev(wl.u_vertex, dtype),
                                          dev(wl.coef, dtype))
    plan = api.AssemblyPlan(conn, wl.n_vert)
    F = plan.assemble(R, nc).cpu().numpy()
    ref_R, ref_abs, _, _ = oracle_reference(wl, dtype)
    ref_F = oracle.assemble(dim, nc, wl.n_vert, wl.conn, ref_R)
    scale = oracle.assemble(dim, nc, wl.n_vert, wl.conn, ref_abs)
    err = np.abs(F - ref_F) / np.maximum(scale, 1e-300)
    assert err.max() <= TOL[dtype], f"global residual scaled error {err.max():.2e}"


@pytest.mark.parametrize("dtype", DTYPES)
def test_patch_test_on_gpu(dtype):
    """Constant coefficient, linear u: interior rows of the assembled GPU
    residual vanish to rounding (scaled by the oracle's assembled
    magnitudes on the same rounded inputs)."""
    n = 12
    coords, conn = mg.tet_grid(n, None, np.random.default_rng(2))
    ne, nv = conn.shape[0], coords.shape[0]
    uv = coords @ np.array([[0.3, -0.7, 0.2]]).T + 0.5
    coef = np.full((1, 4, ne), 1.3)
    X, C = dev(coords, torch.float64), dev(conn, torch.int32)
    R = api.fem_integrate_residual_gather(3, mg.LAPLACE, mg.RULE_TET4, X, C, dev(uv, dtype), dev(coef, dtype))
    F = api.AssemblyPlan(C, nv).assemble(R, 1).cpu().numpy()[:, 0]
    ij, dj, _ = oracle.geometry(coords, conn)
    Ra = oracle.integrate_abs(3, mg.LAPLACE, mg.RULE_TET4, ij, dj, mg.closure(conn, rounded(uv, dtype)),
                              rounded(coef, dtype))
    scale = oracle.assemble(3, 1, nv, conn, Ra)[:, 0]
    idx = np.stack(np.unravel_index(np.arange(nv), (n + 1,) * 3), axis=1)
    interior = np.all((idx > 0) & (idx < n), axis=1)
    assert np.max(np.abs(F[interior]) / scale[interior]) <= TOL[dtype]
    assert np.abs(F[~interior]).max() > 1e-4


def test_autograd_through_restrict_integrate_assemble():
    """L = sum W . F(u_vertex, coef) with F = assemble(integrate(closure(u)))
    differentiated by torch through the three custom functions, against
    central differences (FP64)."""
    dt = torch.float64
    wl = grid_workload(3, mg.ELASTICITY, 300)
    conn = dev(wl.conn, torch.int32)
    plan = api.AssemblyPlan(conn, wl.n_vert)
    ij, dj = api.fem_geometry(dev(wl.coords, torch.float64), conn, dt)
    uv = dev(wl.u_vertex, dt).requires_grad_(True)
    cf = dev(wl.coef, dt).requires_grad_(True)
    W = dev(np.random.default_rng(9).normal(size=(wl.n_vert, 3)), dt)

    def L(u, c):
        R = api.integrate_residual(3, mg.ELASTICITY, wl.rule, ij, dj, api.restrict(plan, conn, u), c)
        return (api.assemble(plan, conn, R, 3) * W).sum()

    L(uv, cf).backward()
    gu, gc = uv.grad.cpu().numpy(), cf.grad.cpu().numpy()
    rng = np.random.default_rng(1)
    with torch.no_grad():
        for _ in range(5):
            v, c = int(rng.integers(wl.n_vert)), int(rng.integers(3))
            if not (wl.conn == v).any():
                continue
            h = 1e-3
            up, um = uv.detach().clone(), uv.detach().clone()
            up[v, c] += h
            um[v, c] -= h
            fd = (float(L(up, cf)) - float(L(um, cf))) / (2 * h)
            assert abs(fd - gu[v, c]) <= 1e-9 * max(1.0, np.abs(gu).max())
        for _ in range(5):
            m, q, e = int(rng.integers(2)), int(rng.integers(4)), int(rng.integers(wl.n_elem))
            h = 1e-3 * max(1.0, abs(wl.coef[m, q, e]))
            cp, cm = cf.detach().clone(), cf.detach().clone()
            cp[m, q, e] += h
            cm[m, q, e] -= h
            fd = (float(L(uv, cp)) - float(L(uv, cm))) / (2 * h)
            assert abs(fd - gc[m, q, e]) <= 1e-9 * max(1.0, np.abs(gc).max())


@pytest.mark.parametrize("cfg", [2, "3b"])
def test_full_size_assembly(cfg):
    """The benchmark meshes at full size: FP64 assembly bit for bit against
    the oracle, FP32 to the scaled bar."""
    wl = mg.config(cfg)
    nc = wl.n_comp
    conn = dev(wl.conn, torch.int32)
    plan = api.AssemblyPlan(conn, wl.n_vert)
    R = np.random.default_rng(4).normal(size=((wl.dim + 1) * nc, wl.n_elem))
    ref = oracle.assemble(wl.dim, nc, wl.n_vert, wl.conn, R)
    assert np.array_equal(plan.assemble(dev(R, torch.float64), nc).cpu().numpy(), ref)
    R32 = rounded(R, torch.float32)
    F32 = plan.assemble(dev(R32, torch.float32), nc).cpu().numpy()
    ref32 = oracle.assemble(wl.dim, nc, wl.n_vert, wl.conn, R32)
    scale = oracle.assemble(wl.dim, nc, wl.n_vert, wl.conn, np.abs(R32))
    assert (np.abs(F32 - ref32) / np.maximum(scale, 1e-300)).max() <= TOL[torch.float32]


# the longest row on both sides of the length that is sorted in LDS (256
# slots), no multiple of 64 vertices, and more vertex groups than one step of
# the offset scan takes (4096 of 64 vertices)
@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("n_elem,n_vert,star", [(1, 4, 1), (300, 129, 255), (300, 129, 256), (300, 129, 257), (5000, 70, 4000),
                                                (40000, 4096 * 64 + 65, 200)])
def test_assembly_rows_in_element_order(dim, n_elem, n_vert, star):
    rng = np.random.default_rng(n_elem + star)
    conn = rng.integers(1, n_vert, size=(n_elem, dim + 1)).astype(np.int32)
    conn[rng.permutation(n_elem)[:star], rng.integers(0, dim + 1)] = 0   # vertex 0 lies in `star` elements
    conn[-1, -1] = n_vert - 1
    R = rng.normal(size=((dim + 1) * 2, n_elem))
    plan = api.AssemblyPlan(dev(conn, torch.int32), n_vert)
    F = plan.assemble(dev(R, torch.float64), 2).cpu().numpy()
    assert np.array_equal(F, oracle.assemble(dim, 2, n_vert, conn, R))
    plan.close()


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("dim,nc", [(2, 2), (3, 2), (3, 3)])
# a wave per component below 2048 groups of 64 vertices, a wave per group from there on
@pytest.mark.parametrize("n_vert", [2047 * 64, 2047 * 64 + 1])
def test_assembly_component_split(dim, nc, dtype, n_vert):
    rng = np.random.default_rng(n_vert)
    n_elem = 60000
    conn = rng.integers(0, n_vert, size=(n_elem, dim + 1)).astype(np.int32)
    R = rng.integers(-8, 9, size=((dim + 1) * nc, n_elem)).astype(np.float64)   # exact sums in both types
    plan = api.AssemblyPlan(dev(conn, torch.int32), n_vert)
    F = plan.assemble(dev(R, dtype), nc).cpu().numpy()
    assert np.array_equal(F, oracle.assemble(dim, nc, n_vert, conn, R))
    plan.close()


# rows above 32 slots: a few among short ones, which the whole wave sorts one after
# the other (at the edges of 32, 64 and 256 entries), several in one group, and
# groups of wide rows only, where every lane sorts its own
@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("n_elem,n_vert,stars", [(300, 129, (32,)), (300, 129, (33,)), (300, 129, (64,)), (300, 129, (65, 200)),
                                                 (900, 400, (255, 128, 129, 40)), (3000, 70, (100,)), (2000, 129, (200, 33)),
                                                 (300, 64, (90, 90, 90))])
def test_assembly_wide_rows(dim, n_elem, n_vert, stars):
    rng = np.random.default_rng(n_elem + sum(stars))
    hubs = rng.permutation(min(n_vert, 64))[:len(stars)]    # all in the first group of 64 vertices
    conn = rng.choice(np.setdiff1d(np.arange(n_vert), hubs), size=(n_elem, dim + 1)).astype(np.int32)
    for hub, star in zip(hubs, stars):
        rows = rng.permutation(n_elem)[:star]
        conn[rows, rng.integers(0, dim + 1, star)] = hub
    R = rng.normal(size=((dim + 1) * 2, n_elem))
    plan = api.AssemblyPlan(dev(conn, torch.int32), n_vert)
    F = plan.assemble(dev(R, torch.float64), 2).cpu().numpy()
    assert np.array_equal(F, oracle.assemble(dim, 2, n_vert, conn, R))
    plan.close()
