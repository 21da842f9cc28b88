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


@pytest.fixture(scope="module")
def mixed(rh):
    """Networks of 1,850, 18,599, 134,999 and 18,599 states: the one-workgroup
    path, and the tree path with three tiers and with five."""
    ctx = rh.Context(0)
    grids = [gridgen.config_grid("c1", 0), gridgen.config_grid("c2", 0), gridgen.config_grid("c3", 0),
             gridgen.perturb_loads(gridgen.config_grid("c2", 0), 9)]
    nets = [rh.Network(ctx, g) for g in grids]
    for n in nets:
        n.solve(1e-12, 30)
    return ctx, nets


@pytest.mark.parametrize("prec", ["fp64", "refined"])
@pytest.mark.parametrize("which", [(0, 1, 2, 3), (2, 1), (3, 2, 1)])
@pytest.mark.parametrize("recorded", [False, True])
def test_batch_over_networks_of_other_tiers(rh, mixed, which, prec, recorded):
    """One launch over networks of both paths, and of trees of other depths, in
    both precisions: every product has the bits that the network alone gives."""
    import torch

    ctx, nets = mixed
    p = rh.RH_FP64 if prec == "fp64" else rh.RH_FP32_REFINED
    nets, ks = [nets[i] for i in which], [(3, 17, 5, 33)[i] for i in which]
    W = [torch.from_numpy(np.ascontiguousarray(gridgen.directions(n.n_p, k, 40 + k).T)).cuda()
         for n, k in zip(nets, ks)]
    want, out = [torch.zeros_like(w) for w in W], [torch.zeros_like(w) for w in W]
    for n, w, o in zip(nets, W, want):
        n.hvp_device(w, o, prec=p)
    torch.cuda.synchronize()
    b = ctx.batch(nets, W, out, prec=p) if recorded else None
    for _ in range(3):
        for o in out:
            o.fill_(float("nan"))
        torch.cuda.synchronize()
        if recorded:
            b.launch()
        else:
            ctx.hvp_batch_device(nets, W, out, prec=p)
        torch.cuda.synchronize()
        for o, w in zip(out, want):
            assert torch.equal(o, w)


def test_refined_products_agree_with_fp64(rh, mixed):
    import torch

    ctx, nets = mixed
    for n in nets:
        W = torch.from_numpy(np.ascontiguousarray(gridgen.directions(n.n_p, 18, 7).T)).cuda()
        a, b = torch.zeros_like(W), torch.zeros_like(W)
        n.hvp_device(W, a)
        n.hvp_device(W, b, prec=rh.RH_FP32_REFINED)
        torch.cuda.synchronize()
        # corrections stop at a normwise backward error of 1e-13, three orders
        # below this at a condition number of 1e4 to 1e5
        assert float((a - b).abs().max()) <= 1e-7 * float(a.abs().max())
