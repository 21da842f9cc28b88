"""The tree path of the products (triangular solves as small dense products).

The plan is replayed on the CPU and compared with row-by-row sweeps; on the GPU
the products are compared with the oracle and with the one-workgroup path at
the sizes where a chunk of 16 directions, a round of chunks or a launch ends.
"""
import subprocess
from pathlib import Path

import numpy as np
import pytest

import gridgen
from test_native import GRIDS, _dump

ROOT = Path(__file__).resolve().parents[1]
CSRC = ROOT / "paper_2201_00241_amd" / "csrc"


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    out = tmp_path_factory.mktemp("native") / "check_tree"
    subprocess.run(["g++", "-O2", "-std=c++17", str(ROOT / "tests/native/check_tree.cpp"),
                    str(CSRC / "tree.cpp"), str(CSRC / "network.cpp"), str(CSRC / "sparse_lu.cpp"), "-o", str(out)],
                   check=True)
    return out


def _check(res):
    assert "violations 0" in res.stdout, res.stdout
    errs = {p[1]: float(p[2]) for p in (ln.split() for ln in res.stdout.splitlines()) if p[0] == "max_err"}
    assert set(errs) == {"L", "U", "Ut", "Lt"}
    # sums of at most a few hundred products of numbers of order one, nested
    # as deep as the tree: 1e-12 is three orders above their rounding
    assert all(e < 1e-12 for e in errs.values()), res.stdout


@pytest.mark.parametrize("name", ["geo60", "geo120", "c1", "c2"])
def test_plan_of_a_network(driver, tmp_path, name):
    _dump(GRIDS[name](), tmp_path / "grid.bin")
    _check(subprocess.run([str(driver), str(tmp_path / "grid.bin")], capture_output=True, text=True, check=True))


# one row; the edges of a tile, a leaf, an upper node and the top; and trees
# that are one path, one parent or no edges at all
@pytest.mark.parametrize("rows", [1, 16, 17, 64, 65, 448, 449, 1000, 3001])
@pytest.mark.parametrize("kind", ["chain", "star", "diagonal"])
def test_plan_of_a_made_up_tree(driver, kind, rows):
    res = subprocess.run([str(driver), kind, str(rows)], capture_output=True, text=True, check=True)
    if (kind, rows) == ("chain", 3001):
        assert "ok 0" in res.stdout  # a path this long has too many tiers: the other path takes it
    else:
        _check(res)


# ---- on the GPU -------------------------------------------------------------


@pytest.fixture(scope="module")
def solved():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from oracle import solve
    from paper_2201_00241_amd import rh

    g = gridgen.config_grid("c2", 0)  # 18,999 states: above the path's smallest network (16,000)
    ctx = rh.Context(0)
    net = rh.Network(ctx, g)
    net.solve()
    return rh, ctx, net, solve(g)


def _close(got, want, tol):
    assert np.max(np.abs(got - want)) <= tol * np.max(np.abs(want))


# a product's error: two solves with a 10,000-bus Jacobian (condition number
# about 1e4) in FP64 leave 1e-12 or so; corrections of FP32 solves stop at a
# normwise backward error of the solve's tolerance, three orders above that
TOL = {"fp64": 1e-10, "refined": 1e-8}


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["fp64", "refined"])
@pytest.mark.parametrize("k", [1, 15, 16, 17, 33])
def test_products_against_the_oracle(solved, k, prec):
    rh, _, net, s = solved
    W = gridgen.directions(net.n_p, k, 5)
    got = net.hvp(W, prec=rh.RH_FP64 if prec == "fp64" else rh.RH_FP32_REFINED)
    assert net.report()["dirs_per_group"] == 16  # the tree path's chunk
    _close(got, s.hvp(W), TOL[prec])


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["fp64", "refined"])
def test_other_path_agrees_and_bits_do_not_depend_on_the_launch(solved, prec, monkeypatch):
    rh, _, net, _ = solved
    p = rh.RH_FP64 if prec == "fp64" else rh.RH_FP32_REFINED
    W = gridgen.directions(net.n_p, 4112, 6)  # 257 chunks: two rounds, of 129 and 128
    got = net.hvp(W, prec=p)
    for at, k in ((0, 1), (15, 2), (31, 17), (1023, 17), (2060, 9), (4095, 17)):
        assert np.array_equal(net.hvp(np.ascontiguousarray(W[:, at:at + k]), prec=p), got[:, at:at + k])
    monkeypatch.setenv("RH_DIRS_PER_GROUP", "1")
    _close(net.hvp(np.ascontiguousarray(W[:, :40]), prec=p), got[:, :40], TOL[prec])


@pytest.mark.gpu
@pytest.mark.parametrize("recorded", [False, True])
def test_batch_with_networks_of_both_paths(solved, recorded):
    import torch

    rh, ctx, net, s = solved
    small = rh.Network(ctx, gridgen.config_grid("c1", 0))
    small.solve()
    nets, ks = [small, net, net], [3, 17, 1]
    W = [torch.from_numpy(np.ascontiguousarray(gridgen.directions(n.n_p, k, 7 + i).T)).cuda()
         for i, (n, k) in enumerate(zip(nets, ks))]
    want = [n.hvp(np.ascontiguousarray(w.cpu().numpy().T)) for n, w in zip(nets, W)]
    out = [torch.zeros_like(w) for w in W]
    torch.cuda.synchronize()
    if recorded:
        b = ctx.batch(nets, W, out)
        for _ in range(3):  # replays, with other work between them
            for o in out:
                o.zero_()
            torch.cuda.synchronize()
            b.launch()
            torch.cuda.synchronize()
            for o, w in zip(out, want):
                assert np.array_equal(o.cpu().numpy().T, w)
    else:
        ctx.hvp_batch_device(nets, W, out)
        torch.cuda.synchronize()
        for o, w in zip(out, want):
            assert np.array_equal(o.cpu().numpy().T, w)


@pytest.mark.gpu
@pytest.mark.parametrize("k_block", [100, 1024])
def test_full_hessian_into_a_padded_buffer(solved, k_block):
    import torch

    rh, _, net, s = solved
    n = net.n_p
    out = torch.full((n, n + 3), -7.0, dtype=torch.float64, device="cuda")
    net.reduced_hessian_device(out[:, :n], k_block=k_block)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    assert (got[:, n:] == -7.0).all()
    cols = [0, 15, 16, 99, 100, 1023, 1024, n - 1]
    E = np.zeros((n, len(cols)))
    E[cols, range(len(cols))] = 1.0
    want = net.hvp(E)
    assert np.array_equal(got[cols, :n].T, want)
    _close(want, s.hvp(E), TOL["fp64"])


# one node (up to 448 states), two tiers, three tiers; sizes that end within
# and at a tile
@pytest.mark.gpu
@pytest.mark.parametrize("n_bus", [9, 60, 75, 120, 200, 260, 1000, 2100, 2600])
def test_device_factors_by_fronts(n_bus):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2201_00241_amd import rh

    g = gridgen.config_grid("c0", 0) if n_bus == 9 else gridgen.geometric(
        n_bus, int(1.35 * n_bus), max(3, n_bus // 10), seed=500 + n_bus, alpha=0.2, kappa=0.017)
    ctx = rh.Context(0)
    host, dev = rh.Network(ctx, g), rh.Network(ctx, g)
    host.solve()
    for _ in range(2):  # the second solve finds the fronts of the first
        dev.solve_device()
    # the same elimination in another order of sums: a few hundred roundings
    # at most, on factors of a matrix whose pivots stay within 1e4 of another
    for d, h in zip(dev.factors(), host.factors()):
        assert np.max(np.abs(d - h)) <= 1e-11 * np.max(np.abs(h))
    assert np.max(np.abs(dev.state() - host.state())) <= 1e-11
