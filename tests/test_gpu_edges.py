"""Kernels at the sizes where their tiling can go wrong (block edges, remainders, list
capacities), against the float64 oracle."""
import numpy as np
import pytest
import torch

from tests.test_gpu_density import _check_densify

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2509_05216_amd as P
    return P


@pytest.fixture(scope="module")
def ctx(P):
    return P.Context(0)


# ---------------------------------------------------------------- densify
@pytest.mark.parametrize("n,deg,n_split", [
    (1024, 3, 8),      # one block, far more outputs than one run of it holds
    (2049, 0, 8),      # the fewest rows, a one-Gaussian last block
    (5000, 1, 5)])
def test_densify_many_children(P, ctx, n, deg, n_split):
    from paper_2509_05216_amd import density as D
    ri = _check_densify(P, D, ctx, n, deg, 31 + n, 20.0, n_split)
    assert ri["children"] > 0
