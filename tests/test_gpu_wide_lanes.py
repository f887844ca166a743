"""Several elements per lane with coefficients in each space and either rule:
the counts at which a launch takes them, rows that start off the 128-byte
lines, the words around every output untouched. The reference is the same call
on a short part of the mesh, one element per lane, which other tests hold to
the oracle; elements are independent, so the bits must agree."""
import pytest
import torch

from paper_1607_04245_amd import api
from paper_1607_04245_amd import meshgen as mg

from test_gpu_rows import DTYPES, SENTINEL, _cut, _rows

pytestmark = pytest.mark.gpu

FULL = {2: mg.RULE_TRI3, 3: mg.RULE_TET4}
FORMS = [(mg.COEF_P1, True), (mg.COEF_P0, True), (mg.COEF_QUAD, False), (mg.COEF_P1, False), (mg.COEF_P0, False)]


def _mesh(dim, physics, full, space, n, dtype, pad, seed=17):
    """Inputs whose rows start pad words into their buffers."""
    rule = FULL[dim] if full else mg.RULE_CENTROID
    gen = torch.Generator("cuda").manual_seed(seed)
    nbt = api.n_basis(dim) * api.n_comp(dim, physics)
    ij = _rows((dim * dim,), n, dtype, gen, pad=pad)[1]
    dj = _rows((1,), n, dtype, gen, 0.5, 2.0, pad=pad)[1][0]
    u, w = _rows((nbt,), n, dtype, gen, pad=pad)[1], _rows((nbt,), n, dtype, gen, pad=pad)[1]
    coef = _rows((api.n_coef(physics), api.n_coef_words(dim, rule, space)), n, dtype, gen, 0.5, 2.0, pad=pad)[1]
    return rule, ij, dj, u, w, coef


def _parts(n):
    return (0, 70), (n // 2 - 1, n // 2 + 299), (n - 70, n)


def _check(outs, n, call, inputs):
    """outs: (buffer, view, words before the view); call(inputs, views or None) -> results"""
    for buf, view, _ in outs:
        view.fill_(float("nan"))
    call(inputs, [view for _, view, _ in outs])
    for lo, hi in _parts(n):
        ref = call([_cut(t[..., lo:hi], hi - lo, 0) for t in inputs], None)
        for (_, view, _), r in zip(outs, ref):
            assert torch.equal(view[..., lo:hi], r)
    for buf, view, pad in outs:
        assert (buf[:pad] == SENTINEL).all() and (buf[pad + view.numel():] == SENTINEL).all()
        assert not view.isnan().any()


# both sides of the counts from which a lane takes two and four elements, at odd words
COUNTS = [(262143, 0), (262145, 1), (524287, 0), (524289, 3), (524291, 0)]


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("space,full", FORMS)
@pytest.mark.parametrize("dim,physics", [(2, mg.ELASTICITY), (3, mg.LAPLACE), (3, mg.MASS)])
@pytest.mark.parametrize("n,pad", COUNTS)
def test_residual_and_adjoint(dim, physics, space, full, dtype, n, pad):
    rule, *inputs = _mesh(dim, physics, full, space, n, dtype, pad)
    u, coef = inputs[2], inputs[4]
    out = [_rows(tuple(t.shape[:-1]), n, dtype, None, pad=pad) + (pad,) for t in (u, u, coef)]

    def forward(t, views):
        return [api.fem_integrate_residual(dim, physics, rule, t[0], t[1], t[2], t[4], coef_space=space,
                                           out=views[0] if views else None)]

    def backward(t, views):
        return api.fem_integrate_residual_backward(dim, physics, rule, t[0], t[1], t[2], t[4], t[3], coef_space=space,
                                                   **dict(zip(("du", "dcoef"), views or [])))

    _check(out[:1], n, forward, inputs)
    _check(out[1:], n, backward, inputs)


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("space,full", [(mg.COEF_QUAD, True)] + FORMS)
@pytest.mark.parametrize("dim,physics", [(2, mg.ELASTICITY), (3, mg.ELASTICITY), (3, mg.LAPLACE), (2, mg.MASS)])
@pytest.mark.parametrize("n,pad", [(131073, 1), (262144, 0), (262147, 1), (524291, 3)])
def test_matrices(dim, physics, space, full, dtype, n, pad):
    rule, ij, dj, u, _, coef = _mesh(dim, physics, full, space, n, dtype, pad)
    out = _rows((u.shape[0] ** 2,), n, dtype, None, pad=pad) + (pad,)

    def matrices(t, views):
        return [api.fem_integrate_jacobian(dim, physics, rule, *t, coef_space=space, out=views[0] if views else None)]

    _check([out], n, matrices, [ij, dj, coef])


@pytest.mark.parametrize("dtype", DTYPES)
def test_batch(dtype):
    """One launch above the size from which a lane takes several elements, each
    space and rule in it."""
    sizes = [300001, 3, 262145, 77, 200003, 131073]
    meshes, outs, inputs = [], [], []
    for i, (n, (space, full)) in enumerate(zip(sizes, [(mg.COEF_QUAD, True)] + FORMS)):
        dim, physics = [(3, mg.LAPLACE), (2, mg.MASS), (2, mg.ELASTICITY)][i % 3]
        rule, ij, dj, u, _, coef = _mesh(dim, physics, full, space, n, dtype, pad=i, seed=i)
        buf, out = _rows(tuple(u.shape[:-1]), n, dtype, None, pad=i)
        out.fill_(float("nan"))
        meshes.append(dict(dim=dim, physics=physics, rule=rule, coef_space=space, inv_j=ij, det_j=dj, u=u, coef=coef,
                           out=out))
        outs.append((buf, out, i))
    plan = api.BatchPlan(meshes)
    plan.run()
    torch.cuda.synchronize()
    for m, (buf, out, pad) in zip(meshes, outs):
        n = out.shape[-1]
        for lo, hi in _parts(n) if n > 300 else ((0, n),):
            part = [_cut(m[k][..., lo:hi], hi - lo, 0) for k in ("inv_j", "det_j", "u", "coef")]
            ref = api.fem_integrate_residual(m["dim"], m["physics"], m["rule"], *part, coef_space=m["coef_space"])
            assert torch.equal(out[..., lo:hi], ref)
        assert not out.isnan().any()
        assert (buf[:pad] == SENTINEL).all() and (buf[pad + out.numel():] == SENTINEL).all()
    plan.close()
