"""Dense Cholesky at the edges of its panels, strips and tiles: sizes around
multiples of 16 and 64, and right-hand sides that fill strips and tile rows of
their own."""
import numpy as np
import pytest
import torch

import scipy.linalg as sla
from paper_2201_00241_amd import rh

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return rh.Context(0)


def _spd(n, seed):
    Q, _ = np.linalg.qr(np.random.default_rng(seed).standard_normal((n, n)))
    return (Q * np.random.default_rng(seed + 1).uniform(0.1, 10.0, n)) @ Q.T


@pytest.mark.parametrize("n", [15, 16, 17, 63, 64, 65, 80, 127, 128, 129, 193, 321])
@pytest.mark.parametrize("nrhs", [0, 1, 64, 65, 200])
def test_factor_and_solution(ctx, n, nrhs):
    A = _spd(n, 7 * n)
    B = np.random.default_rng(n).standard_normal((n, max(nrhs, 1)))
    dev = torch.full((n, n + 5), 3.0, dtype=torch.float64, device="cuda")
    dev[:, :n] = torch.from_numpy(np.tril(A).T.copy())
    rhs = torch.from_numpy(B[:, :nrhs].T.copy()).cuda() if nrhs else torch.zeros((0, n), dtype=torch.float64,
                                                                                  device="cuda")
    assert ctx.cholesky_solve_device(dev[:, :n], rhs) == -1
    out = dev.cpu().numpy()
    assert (out[:, n:] == 3.0).all()
    L = out[:, :n].T
    assert (L[np.triu_indices(n, 1)] == 0.0).all()  # (the upper triangle is left alone)
    # backward errors of at most a few n units of rounding
    assert np.abs(L @ L.T - A).max() <= 4 * n * 2.3e-16 * np.abs(A).max()
    if nrhs:
        X = rhs.cpu().numpy().T
        want = sla.cho_solve((np.linalg.cholesky(A), True), B[:, :nrhs])
        # condition number 100
        assert np.abs(X - want).max() <= 100 * 4 * n * 2.3e-16 * np.abs(want).max()


# the first pivot that fails, in the first and last place of a tile, of a
# panel, and of the matrix
@pytest.mark.parametrize("n,bad", [(64, 0), (64, 15), (64, 16), (64, 63), (129, 64), (129, 79), (129, 128)])
def test_failing_column(ctx, n, bad):
    A = _spd(n, 3 * n + bad)
    A[bad, bad] -= np.linalg.cholesky(A)[bad, bad] ** 2 + 1.0
    dev, rhs = torch.from_numpy(A.T.copy()).cuda(), torch.ones((1, n), dtype=torch.float64, device="cuda")
    with pytest.raises(rh.RhError) as ei:
        ctx.cholesky_solve_device(dev, rhs)
    assert ei.value.status == rh.RH_ESINGULAR and ei.value.failed_col == bad
