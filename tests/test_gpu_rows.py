"""Rows at odd words: element counts and base addresses that put the SoA rows
off the 128-byte lines take other stores, another workgroup order and several
elements per lane, and must give the same bits. Every element is independent,
so the reference is the same call on a whole-line count (a multiple of 32),
cut to the count under test."""
import pytest
import torch

from paper_1607_04245_amd import _native as N
from paper_1607_04245_amd import api
from paper_1607_04245_amd import meshgen as mg

pytestmark = pytest.mark.gpu

DTYPES = [torch.float32, torch.float64]
SENTINEL = -7.0


def _rows(shape, n, dtype, gen, lo=-1.0, hi=1.0, pad=0):
    """Random rows [.., n]; the view starts pad words into its buffer and a
    guard row follows it. Returns (buffer, view)."""
    rows = 1
    for s in shape:
        rows *= s
    buf = torch.full((pad + (rows + 1) * n,), SENTINEL, dtype=dtype, device="cuda")
    view = buf[pad:pad + rows * n].view(*shape, n)
    if gen is not None:
        view.copy_(torch.rand((*shape, n), generator=gen, device="cuda", dtype=torch.float64) * (hi - lo) + lo)
    return buf, view


def _inputs(dim, physics, rule, order, n, dtype, seed=3):
    gen = torch.Generator("cuda").manual_seed(seed)
    nbt = api.n_basis(dim, order) * api.n_comp(dim, physics)
    nw = (api.n_coef(physics), api.n_qpts(dim, rule))
    ij = _rows((dim * dim,), n, dtype, gen)[1]
    dj = _rows((1,), n, dtype, gen, 0.5, 2.0)[1][0]
    u, w = _rows((nbt,), n, dtype, gen)[1], _rows((nbt,), n, dtype, gen)[1]
    coef = _rows(nw, n, dtype, gen, 0.5, 2.0)[1]
    return ij, dj, u, w, coef


def _cut(t, n, pad):
    """The first n columns of t as contiguous rows that start pad words into a buffer."""
    view = _rows(tuple(t.shape[:-1]), n, t.dtype, None, pad=pad)[1]
    view.copy_(t[..., :n])
    return view


def _call(kind, dim, physics, rule, order, ij, dj, u, w, coef, outs):
    if kind == "fwd":
        fn = (api.fem_integrate_residual, api.fem_integrate_residual_p2, api.fem_integrate_residual_p3)[order - 1]
        fn(dim, physics, rule, ij, dj, u, coef, out=outs[0])
    elif kind == "bwd":
        fn = (api.fem_integrate_residual_backward, api.fem_integrate_residual_p2_backward,
              api.fem_integrate_residual_p3_backward)[order - 1]
        fn(dim, physics, rule, ij, dj, u, coef, w, du=outs[0], dcoef=outs[1])
    else:
        api.fem_integrate_jacobian(dim, physics, rule, ij, dj, coef, out=outs[0], order=order)


def _compare(kind, dim, physics, rule, order, n, dtype, pad=0):
    big = (n + 31) // 32 * 32
    full = _inputs(dim, physics, rule, order, big, dtype)
    shapes = {"fwd": [full[2].shape[:-1]], "bwd": [full[2].shape[:-1], full[4].shape[:-1]],
              "mat": [(full[2].shape[0] ** 2,)]}[kind]
    ref = [_rows(tuple(s), big, dtype, None)[1] for s in shapes]
    _call(kind, dim, physics, rule, order, *full, ref)
    bufs, outs = zip(*[_rows(tuple(s), n, dtype, None, pad=pad) for s in shapes])
    _call(kind, dim, physics, rule, order, *[_cut(t, n, pad) for t in full], outs)
    torch.cuda.synchronize()
    for r, o, b in zip(ref, outs, bufs):
        assert torch.equal(r[..., :n], o)
        assert (b[:pad] == SENTINEL).all() and (b[pad + o.numel():] == SENTINEL).all()


RULES = {(2, 1): mg.RULE_TRI3, (3, 1): mg.RULE_TET4, (2, 2): mg.RULE_TRI6, (3, 2): mg.RULE_TET11,
         (2, 3): mg.RULE_TRI6, (3, 3): mg.RULE_TET11}


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("kind", ["fwd", "bwd"])
@pytest.mark.parametrize("dim,physics", [(2, mg.LAPLACE), (3, mg.LAPLACE), (3, mg.ELASTICITY), (2, mg.MASS)])
# one element, tile edges, and each side of the two counts from which a lane
# takes two and four elements (2 * 64 * 2048 and twice that)
@pytest.mark.parametrize("n,pad", [(1, 0), (3, 1), (63, 0), (64, 3), (129, 0), (4099, 0), (262143, 0), (262145, 0),
                                   (524287, 1), (524289, 0), (524290, 0), (524320, 1)])
def test_p1_rows(dim, physics, kind, dtype, n, pad):
    _compare(kind, dim, physics, RULES[dim, 1], 1, n, dtype, pad)


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("kind", ["fwd", "bwd", "mat"])
@pytest.mark.parametrize("dim,physics,order", [(2, mg.ELASTICITY, 2), (3, mg.LAPLACE, 2), (2, mg.LAPLACE, 3),
                                               (3, mg.LAPLACE, 3), (3, mg.ELASTICITY, 3), (3, mg.MASS, 3)])
@pytest.mark.parametrize("n,pad", [(1, 0), (257, 0), (8191, 0), (8192, 1)])
def test_high_order_rows(dim, physics, order, kind, dtype, n, pad):
    if kind == "mat" and order == 3 and physics == mg.ELASTICITY:
        n = min(n, 257)   # 3600 rows
    _compare(kind, dim, physics, RULES[dim, order], order, n, dtype, pad)


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("dim,physics", [(2, mg.ELASTICITY), (3, mg.ELASTICITY), (3, mg.MASS)])
@pytest.mark.parametrize("n,pad", [(1, 0), (65, 0), (8191, 0), (8192, 1)])
def test_p1_matrix_rows(dim, physics, dtype, n, pad):
    _compare("mat", dim, physics, RULES[dim, 1], 1, n, dtype, pad)


# launches of whole lines on both sides of the sizes at which the workgroup
# order and the stores change (192 and 512 MiB of rows)
@pytest.mark.parametrize("dtype,n", [(torch.float32, 1 << 20), (torch.float32, 1 << 21), (torch.float64, 1 << 20),
                                     (torch.float64, 1 << 21)])
@pytest.mark.parametrize("kind", ["fwd", "bwd"])
def test_large_whole_lines(kind, dtype, n):
    dim, physics, rule = 3, mg.ELASTICITY, mg.RULE_TET4
    full = _inputs(dim, physics, rule, 1, n, dtype)
    outs = [torch.empty_like(full[2])] + ([torch.empty_like(full[4])] if kind == "bwd" else [])
    _call(kind, dim, physics, rule, 1, *full, outs)
    for lo, hi in ((0, 4096), (n // 2 - 100, n // 2 + 924), (n - 4096, n)):
        part = [t[..., lo:hi].contiguous() for t in full]
        ref = [torch.empty_like(o[..., :hi - lo].contiguous()) for o in outs]
        _call(kind, dim, physics, rule, 1, *part, ref)
        for r, o in zip(ref, outs):
            assert torch.equal(r, o[..., lo:hi])


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("vec", [1, 2, 4])
@pytest.mark.parametrize("n", [1, 2, 5, 130, 1023])
def test_explicit_widths_any_count(vec, dtype, n):
    """A set width applies at every count; the words past the end stay untouched."""
    saved = [api.fem_get_tuning(3, mg.LAPLACE, mg.RULE_TET4, dtype, op=op) for op in (N.OP_RESIDUAL, N.OP_BACKWARD)]
    try:
        for op in (N.OP_RESIDUAL, N.OP_BACKWARD):
            api.fem_set_tuning(3, mg.LAPLACE, mg.RULE_TET4, dtype, vec=vec, waves_per_block=1, op=op)
        for kind in ("fwd", "bwd"):
            _compare(kind, 3, mg.LAPLACE, mg.RULE_TET4, 1, n, dtype, pad=1)
    finally:
        for op, t in zip((N.OP_RESIDUAL, N.OP_BACKWARD), saved):
            api.fem_set_tuning(3, mg.LAPLACE, mg.RULE_TET4, dtype, op=op, **t)


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("sizes", [(1, 3, 64, 1023), (300001, 2, 262144, 77, 200003)])
def test_batch_widths(dtype, sizes):
    """Batches below and above the size from which a lane takes several
    elements, meshes shorter than a lane's width among them."""
    meshes, refs = [], []
    for i, n in enumerate(sizes):
        dim, physics = [(2, mg.LAPLACE), (3, mg.ELASTICITY), (3, mg.MASS), (2, mg.ELASTICITY)][i % 4]
        ij, dj, u, _, coef = _inputs(dim, physics, RULES[dim, 1], 1, n, dtype, seed=i)
        refs.append(api.fem_integrate_residual(dim, physics, RULES[dim, 1], ij, dj, u, coef))
        buf, out = _rows(tuple(u.shape[:-1]), n, dtype, None, pad=i)
        meshes.append(dict(dim=dim, physics=physics, rule=RULES[dim, 1], inv_j=ij, det_j=dj, u=u, coef=coef, out=out,
                           buf=buf, pad=i))
    plan = api.BatchPlan(meshes)
    for run in (plan.run, lambda: api.batch_run_noalloc(meshes)):
        for m in meshes:
            m["buf"].fill_(SENTINEL)
        run()
        torch.cuda.synchronize()
        for m, r in zip(meshes, refs):
            assert torch.equal(m["out"], r)
            assert (m["buf"][:m["pad"]] == SENTINEL).all()
            assert (m["buf"][m["pad"] + r.numel():] == SENTINEL).all()
    plan.close()


# small meshes share a tile's matrices among workgroups: one per column or basis
# function (few tiles), some (8192 waves' worth of elements and below), none
@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("dim,physics,order", [(3, mg.LAPLACE, 1), (2, mg.MASS, 2), (3, mg.LAPLACE, 3), (2, mg.ELASTICITY, 3)])
@pytest.mark.parametrize("n", [1, 300, 20000, 70001, 262145])
def test_matrix_parts(dim, physics, order, dtype, n):
    ij, dj, _, _, coef = _inputs(dim, physics, RULES[dim, order], order, n, dtype)
    got = api.fem_integrate_jacobian(dim, physics, RULES[dim, order], ij, dj, coef, order=order)
    for lo, hi in ((0, min(n, 64)), (max(0, n - 100), n)):
        part = [t[..., lo:hi].contiguous() for t in (ij, dj, coef)]
        ref = api.fem_integrate_jacobian(dim, physics, RULES[dim, order], *part, order=order)
        assert torch.equal(got[..., lo:hi], ref)


# P1 matrices take 16 bytes per lane from 64 * 1024 (elasticity) or 64 * 2048
# (FP32 scalar forms at odd words) lanes on: both sides of either limit
@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("dim,physics", [(2, mg.ELASTICITY), (3, mg.ELASTICITY), (3, mg.LAPLACE), (2, mg.MASS)])
@pytest.mark.parametrize("n", [131071, 131073, 262143, 262144, 262147, 524287, 524290, 524291])
def test_matrix_vector_width(dim, physics, dtype, n):
    ij, dj, _, _, coef = _inputs(dim, physics, RULES[dim, 1], 1, n, dtype)
    got = api.fem_integrate_jacobian(dim, physics, RULES[dim, 1], ij, dj, coef)
    for lo, hi in ((0, 70), (n // 2, n // 2 + 300), (n - 70, n)):
        part = [t[..., lo:hi].contiguous() for t in (ij, dj, coef)]
        assert torch.equal(got[..., lo:hi], api.fem_integrate_jacobian(dim, physics, RULES[dim, 1], *part))
