"""The sensor-space filter and smoother with sensors that share a noise source (R = r (a a^T + floor I), a graded) and
see the sources through nearly the same weights, against the oracle's N x N recursions.

R S^{-1} is then far from normal (entries of 2 to 3 with eigenvalues below 1), so a recursion of B = X P that does not
keep X P X^T symmetric loses its digits exponentially. Tolerance: the float64 bar of every parity test, 1e-10
normwise per step; cond(S) <= 5e3, so T cond(S) u = 3e-11 bounds the rounding of either side.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_1107_4192_amd import kfmeg as F
from _helpers import dev, eps_d, eps_x

pytestmark = pytest.mark.gpu
TOL = 1e-10


def shared_noise(N, m, T, r, floor, delta, q, seed=0):
    rng = np.random.default_rng(seed)
    X = (np.ones((m, 1)) * rng.normal(size=N) + delta * rng.normal(size=(m, N))) / np.sqrt(N)
    a = np.linspace(1.0, 0.5, m)
    R = r * (np.outer(a, a) + floor * np.eye(m))
    x = np.cumsum(np.sqrt(q) * rng.normal(size=(T, N)), axis=0)
    Y = x @ X.T + rng.normal(size=(T, m)) @ np.linalg.cholesky(R).T
    return X, q * np.eye(N), R, np.zeros(N), np.eye(N), Y


@pytest.mark.parametrize("N,m,T,r,floor,delta,q", [(12, 2, 60, 1e-2, 1e-2, 0.1, 1e-2), (40, 8, 60, 1.0, 1e-2, 0.1, 1e-2),
                                                   (40, 8, 60, 1e-2, 1e-3, 0.1, 1e-4), (100, 20, 60, 1.0, 1e-2, 0.1, 1e-2),
                                                   (300, 33, 40, 1.0, 1e-2, 0.1, 1e-2)])
def test_shared_noise_against_oracle(N, m, T, r, floor, delta, q):
    p = shared_noise(N, m, T, r, floor, delta, q)
    xf, Pf, dPf = oracle.kf_filter(*p)
    xs, _, dPs = oracle.rts_smooth(xf, Pf, p[1])
    ks = F.KalmanSmoother(*(dev(v) for v in p[:5]), T_max=T)
    try:
        res = ks.run(dev(p[5]))
    finally:
        ks.close()
    assert eps_x(res.x_filt, xf) <= TOL and eps_d(res.Pdiag_filt, dPf) <= TOL
    assert eps_x(res.x_smooth, xs) <= TOL and eps_d(res.Pdiag_smooth, dPs) <= TOL


@pytest.mark.parametrize("gemm", [F.kfd_gemm, F.kfd_gemm_small])
@pytest.mark.parametrize("n,K,ksplit", [(1, 3, 2), (15, 40, 2), (16, 100, 7), (17, 129, 8), (33, 33, 9), (130, 300, 32)])
def test_symmetric_part(gemm, n, K, ksplit):
    """C = alpha (A B^T + B A^T) / 2 + beta Cin, both halves from Cin's lower one."""
    g = torch.Generator().manual_seed(n * 1000 + K + ksplit)
    A, B, Cin = (torch.randn(s, generator=g, dtype=torch.float64) for s in ((n, K), (n, K), (n, n)))
    flags = F.G_TB | F.G_SYMAVG
    kw = dict(alpha=-0.5, beta=2.0, Cin=Cin.cuda(), ksplit=ksplit)
    C = (gemm(A.cuda(), B.cuda(), n, n, K, flags, **kw)).cpu()
    low = torch.tril(Cin)
    want = -0.25 * (A @ B.T + B @ A.T) + 2.0 * (low + torch.tril(Cin, -1).T)
    # K products and ksplit sums on either side, and four more roundings
    bound = (2 * (K + ksplit) + 8) * 2.0 ** -53 * (A.abs() @ B.abs().T + B.abs() @ A.abs().T + 2 * want.abs())
    assert torch.equal(C, C.T)
    assert bool(((C - want).abs() <= bound).all())


@pytest.mark.parametrize("M,N,flags,ksplit", [(8, 8, 0, 1), (8, 9, 0, 2), (8, 8, F.G_LOWER, 2), (8, 8, F.G_MIRROR, 2)])
def test_symmetric_part_refused(M, N, flags, ksplit):
    A, B = torch.ones(M, 4, dtype=torch.float64, device="cuda"), torch.ones(N, 4, dtype=torch.float64, device="cuda")
    with pytest.raises(F.KFError):
        F.kfd_gemm(A, B, M, N, 4, F.G_TB | F.G_SYMAVG | flags, ksplit=ksplit)
