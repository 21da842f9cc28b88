"""Long grids (a radial feeder, a ladder): the paths of their elimination trees
are longer than the tree plan's tiers reach, so they keep the paths that other
networks of their size have left: the device Newton factors them row by row, and
the products stay on one workgroup whatever the number of states."""
import subprocess
from pathlib import Path

import numpy as np
import pytest

import gridgen
from test_native import _dump

ROOT = Path(__file__).resolve().parents[1]
CSRC = ROOT / "paper_2201_00241_amd" / "csrc"


def _grid(n, f, t, every):
    """Lines f - t of low impedance, a small load at each bus, and a generator
    at every `every`-th, which covers its neighbourhood."""
    rng = np.random.default_rng(n)
    m = len(f)
    gens = np.arange(0, n, every)
    Pd = rng.uniform(0.5, 1.5, n) * 2e-3
    Pg = np.full(gens.size, Pd.sum() / gens.size)
    return gridgen._finish(n, f, t, rng.uniform(1e-3, 2e-3, m), rng.uniform(5e-3, 1e-2, m), np.full(m, 1e-4), gens, Pd,
                           0.3 * Pd, Pg, rng.uniform(0.99, 1.01, gens.size), rng.uniform(0.5, 2.0, gens.size),
                           rng.uniform(1.0, 4.0, gens.size), np.zeros(gens.size), f"long{n}", {})


def feeder(n):
    return _grid(n, np.arange(n - 1), np.arange(1, n), 25)


def ladder(n):
    h = n // 2
    a = np.arange(h)
    return _grid(2 * h, np.concatenate([a[:-1], h + a[:-1], a]), np.concatenate([a[1:], h + a[1:], h + a]), 50)


GRIDS = {"feeder": lambda: feeder(1500), "ladder": lambda: ladder(1500)}


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    out = tmp_path_factory.mktemp("native") / "check_tree"
    subprocess.run(["g++", "-O2", "-std=c++17", str(ROOT / "tests/native/check_tree.cpp"),
                    str(CSRC / "tree.cpp"), str(CSRC / "network.cpp"), str(CSRC / "sparse_lu.cpp"), "-o", str(out)],
                   check=True)
    return out


@pytest.mark.parametrize("name", list(GRIDS))
def test_the_plan_refuses(driver, tmp_path, name):
    _dump(GRIDS[name](), tmp_path / "grid.bin")
    res = subprocess.run([str(driver), str(tmp_path / "grid.bin")], capture_output=True, text=True)
    assert "ok 0" in res.stdout, res.stdout


@pytest.mark.parametrize("name", list(GRIDS))
def test_host_solve_matches_the_oracle(name):
    from oracle import solve
    from paper_2201_00241_amd import rh

    g = GRIDS[name]()
    net = rh.Network(rh.Context(-1), g)
    net.solve(1e-12, 30)
    assert np.max(np.abs(net.state() - solve(g).x)) <= 1e-10


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(GRIDS))
def test_device_newton_row_by_row(name):
    import torch

    from oracle import solve
    from paper_2201_00241_amd import rh

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    g = GRIDS[name]()
    ctx = rh.Context(0)
    host, dev = rh.Network(ctx, g), rh.Network(ctx, g)
    host.solve(1e-12, 30)
    for _ in range(2):
        dev.solve_device(1e-12, 30)
    # the same elimination in another order of sums: a few hundred roundings
    for d, h in zip(dev.factors(), host.factors()):
        assert np.max(np.abs(d - h)) <= 1e-11 * np.max(np.abs(h))
    # a chain of a thousand lines: condition number of about 1e6
    assert np.max(np.abs(dev.state() - host.state())) <= 1e-9
    W = gridgen.directions(dev.n_p, 5, 3)
    want = solve(g).hvp(W)
    for net in (host, dev):
        assert np.max(np.abs(net.hvp(W) - want)) <= 1e-8 * np.max(np.abs(want))
