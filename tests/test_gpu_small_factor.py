"""The blocked Cholesky with inverse at the edges of its 64-column blocks and 256-column panels, with
odd leading dimensions, against LAPACK in float64.

Tolerance: both sides factor the same matrix with backward errors of a few n u, so L and L^{-1} differ by
at most about n u cond(A) relative to their norms; with cond(A) <= 100 and n <= 577 that is 7e-12.
"""
import numpy as np
import pytest
import torch

from paper_1107_4192_amd import kfmeg
from paper_1107_4192_amd.synth import random_spd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 8, 9, 63, 64, 65, 127, 129, 255, 256, 257, 319, 321, 577])
@pytest.mark.parametrize("pad", [0, 3])
def test_blocks_and_panels(n, pad):
    A = random_spd(np.random.default_rng(n), n, cond=100.0)
    W = torch.full((n, n + pad), float("nan"), dtype=torch.float64, device="cuda")
    W[:, :n] = torch.tril(torch.as_tensor(A)).cuda() + torch.triu(torch.full((n, n), float("nan")), 1).cuda()
    Z = torch.full((n, n + pad), float("nan"), dtype=torch.float64, device="cuda")
    kfmeg.kfd_chol_inv(W, Z)
    L = np.linalg.cholesky(A)
    got_l = np.tril(W[:, :n].cpu().numpy())
    got_z = Z[:, :n].cpu().numpy()
    Li = np.linalg.inv(L)
    tol = 1e-16 * n * 100 + 1e-15
    assert np.abs(got_l - L).max() <= tol * np.abs(L).max()
    assert np.abs(got_z - Li).max() <= tol * np.abs(Li).max()
    assert not np.triu(got_z, 1).any()                 # explicit zeros
    assert torch.isnan(W[:, n:]).all() and torch.isnan(Z[:, n:]).all()


@pytest.mark.parametrize("n,row", [(64, 0), (64, 7), (65, 64), (300, 8), (300, 255), (300, 256), (300, 299)])
def test_bad_pivot_row(n, row):
    A = random_spd(np.random.default_rng(n + row), n, cond=10.0)
    A[row, row] = -1.0
    with pytest.raises(kfmeg.KFError) as ei:
        kfmeg.kfd_chol_inv(torch.as_tensor(A).cuda())
    assert f"row {row}" in str(ei.value)


@pytest.mark.parametrize("n", [1023, 1025, 1279, 1280, 1281])
def test_one_panel_up_to_1280(n):
    """The edges of the order up to which one matrix is a single panel; the same tolerance at cond 10."""
    A = random_spd(np.random.default_rng(n), n, cond=10.0)
    W = torch.tril(torch.as_tensor(A)).cuda()
    Z = torch.full((n, n), float("nan"), dtype=torch.float64, device="cuda")
    kfmeg.kfd_chol_inv(W, Z)
    L = np.linalg.cholesky(A)
    Li = np.linalg.inv(L)
    tol = 1e-16 * n * 10 + 1e-15
    assert np.abs(np.tril(W.cpu().numpy()) - L).max() <= tol * np.abs(L).max()
    assert np.abs(Z.cpu().numpy() - Li).max() <= tol * np.abs(Li).max()


@pytest.mark.parametrize("n", [15, 16, 17, 31, 33, 47, 48, 49])
def test_blocks_of_16(n):
    """The edges of a diagonal block's 16 columns: factor, inverse and the row of a bad pivot."""
    A = random_spd(np.random.default_rng(n), n, cond=100.0)
    W = torch.tril(torch.as_tensor(A)).cuda() + torch.triu(torch.full((n, n), float("nan"), dtype=torch.float64), 1).cuda()
    Z = torch.full((n, n), float("nan"), dtype=torch.float64, device="cuda")
    kfmeg.kfd_chol_inv(W, Z)
    L = np.linalg.cholesky(A)
    Li = np.linalg.inv(L)
    tol = 1e-16 * n * 100 + 1e-15
    assert np.abs(np.tril(W.cpu().numpy()) - L).max() <= tol * np.abs(L).max()
    assert np.abs(Z.cpu().numpy() - Li).max() <= tol * np.abs(Li).max()
    for row in (n - 1, 16 * ((n - 1) // 16)):
        for bad in (-1.0, 0.0, float("inf"), float("nan")):
            D = np.diag(np.full(n, 2.0))
            D[row, row] = bad
            with pytest.raises(kfmeg.KFError) as ei:
                kfmeg.kfd_chol_inv(torch.as_tensor(D).cuda())
            assert f"row {row}" in str(ei.value)
