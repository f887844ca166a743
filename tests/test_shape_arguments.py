"""Shapes of the binding's arrays from whatever the C interface takes as an
integer: NumPy scalars and arrays and tensors of one element have __index__,
some of them cannot be hashed and some can change their value."""
import numpy as np
import pytest
import torch

from paper_1607_04245_amd import api, meshgen as mg
from paper_1607_04245_amd import _native as N

WANT = ((9, 7), (7,), (12, 7), (2, 4, 7))


@pytest.mark.parametrize("kind", [int, np.int64, np.array, torch.tensor, bool])
def test_index_like_arguments(kind):
    phys = mg.ELASTICITY if kind is not bool else True   # elasticity is 1
    assert api._shapes(kind(3) if kind is not bool else 3, kind(phys), mg.RULE_TET4, 7, N.COEF_QUAD, 1) == WANT


def test_argument_that_changes():
    dim = torch.tensor(2)
    first = api._shapes(dim, mg.ELASTICITY, mg.RULE_TET4, 7)
    dim.fill_(3)
    assert first == ((4, 7), (7,), (6, 7), (2, 3, 7))
    assert api._shapes(dim, mg.ELASTICITY, mg.RULE_TET4, 7) == WANT


@pytest.mark.parametrize("args", [(3.0, 1, 1), ("3", 1, 1), (3, 1, 1, 7)])
def test_refused_arguments(args):
    with pytest.raises((TypeError, ValueError)):
        api._shapes(*args[:3], 7, *args[3:])
