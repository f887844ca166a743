"""Element matrices of every form (physics, order, rule, coefficient space, type)
against the FP64 oracle at counts that reach each kernel variant: a tile's
matrices shared among workgroups or not, rows on whole 128-byte lines (stores
that stream) or not, one or several elements per lane. Bars as in the residual
tests: 1e-5 in FP32 and 1e-12 in FP64 of the oracle's absolute-value sums."""
import numpy as np
import pytest
import torch

import oracle
from paper_1607_04245_amd import api
from paper_1607_04245_amd import meshgen as mg

from _parity import assert_close

pytestmark = pytest.mark.gpu

RULES = {(2, 1): (mg.RULE_TRI3, mg.RULE_CENTROID), (3, 1): (mg.RULE_TET4, mg.RULE_CENTROID),
         (2, 2): (mg.RULE_TRI3, mg.RULE_TRI6), (3, 2): (mg.RULE_TET4, mg.RULE_TET11)}
COUNTS = {1: (2999, 3008, 60003, 60000, 524291, 524288), 2: (2999, 3008, 60003, 60000)}


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("space", [mg.COEF_QUAD, mg.COEF_P1, mg.COEF_P0])
@pytest.mark.parametrize("which", [0, 1])
@pytest.mark.parametrize("dim,phys", [(2, mg.LAPLACE), (3, mg.LAPLACE), (2, mg.ELASTICITY), (3, mg.ELASTICITY),
                                      (2, mg.MASS), (3, mg.MASS)])
@pytest.mark.parametrize("order,n", [(o, n) for o, ns in COUNTS.items() for n in ns])
def test_matrix_forms(order, n, dim, phys, which, space, dtype):
    rule = RULES[dim, order][which]
    gen = torch.Generator("cuda").manual_seed(n + 10 * phys + space)
    rows = api.n_coef(phys), api.n_coef_words(dim, rule, space)
    ij = (torch.rand((dim * dim, n), generator=gen, device="cuda", dtype=torch.float64) * 2 - 1).to(dtype)
    dj = (torch.rand((n,), generator=gen, device="cuda", dtype=torch.float64) * 1.5 + 0.5).to(dtype)
    cf = (torch.rand((*rows, n), generator=gen, device="cuda", dtype=torch.float64) * 1.5 + 0.5).to(dtype)
    K = api.fem_integrate_jacobian(dim, phys, rule, ij, dj, cf, coef_space=space, order=order)
    cols = torch.tensor(sorted({0, 1, 63, 64, n // 2, n // 2 + 1, n - 66, n - 2, n - 1}), device="cuda")
    a = [np.ascontiguousarray(t[..., cols].double().cpu().numpy()) for t in (ij, dj, cf)]
    ref = oracle.jacobian(dim, phys, rule, *a, space=space, order=order)
    scale = oracle.jacobian_abs(dim, phys, rule, *a, space=space, order=order)
    assert_close(K[..., cols].cpu().numpy(), ref, scale, dtype, f"{dim}D phys {phys} P{order} rule {rule} space {space} n {n}")
