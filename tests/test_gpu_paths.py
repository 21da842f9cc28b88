"""Networks of different sizes and shapes side by side on one GPU: what one of
them sets up must not reach the others, and each takes the path meant for it."""
import numpy as np
import pytest

import gridgen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rh():
    import torch

    from paper_2201_00241_amd import rh

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return rh


def test_large_fronts_after_small_ones(rh):
    """The kernels' bound of dynamic LDS belongs to the kernels: the fronts of
    a network built in between must not lower it."""
    ctx = rh.Context(0)
    large, small = rh.Network(ctx, gridgen.config_grid("c2", 0)), rh.Network(ctx, gridgen.config_grid("c0", 0))
    large.solve_device()
    first = large.factors()
    small.solve_device()
    large.solve_device()
    for a, b in zip(first, large.factors()):
        assert np.array_equal(a, b)
