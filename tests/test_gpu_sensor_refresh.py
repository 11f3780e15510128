"""Long horizons of the sensor-space filter: B_t = X P_{t|t-1} is formed from P again every 64 steps.

A prior that is wide where the sensors look and narrow elsewhere makes the first downdate cancel all but 1e-8 of P, so its
rounding, 1e-16 of the prior, is 1e-8 of diag P. The Riccati recursion forgets such an error within a few steps if
B is formed from P; a B that never reads P keeps it. From step 128 on (two refreshes) 1e-11 of diag P is left
far above the rounding of either side (T m u = 1e-13) and far below the kept error.
"""
import numpy as np
import pytest

import oracle
from paper_1107_4192_amd import kfmeg as F
from _helpers import dev, eps_d, eps_x

pytestmark = pytest.mark.gpu


def wide_prior(N, m, T, seed=0):
    rng = np.random.default_rng(seed)
    X = np.zeros((m, N))
    X[:, :m] = np.linalg.qr(rng.normal(size=(m, m)))[0]
    P0 = np.diag(np.where(np.arange(N) < m, 1.0, 1e-8))
    r, q = 1e-10, 1e-12
    x = np.sqrt(np.diag(P0)) * rng.normal(size=N) + np.cumsum(np.sqrt(q) * rng.normal(size=(T, N)), axis=0)
    Y = x @ X.T + np.sqrt(r) * rng.normal(size=(T, m))
    return X, q * np.eye(N), r * np.eye(m), np.zeros(N), P0, Y


@pytest.mark.parametrize("N,m,T,stride", [(12, 2, 300, 0), (40, 8, 200, 0), (40, 8, 200, 7)])
def test_first_steps_rounding_is_forgotten(N, m, T, stride):
    p = wide_prior(N, m, T)
    _, _, dPf = oracle.kf_filter(*p)
    ks = F.KalmanSmoother(*(dev(v) for v in p[:5]), T_max=T, checkpoint_stride=stride)
    try:
        f = ks.filter(dev(p[5]))
    finally:
        ks.close()
    assert eps_d(f.Pdiag_filt[128:], dPf[128:]) <= 1e-11


@pytest.mark.parametrize("T,B", [(63, 1), (64, 1), (65, 1), (66, 3), (130, 1)])
def test_horizons_at_the_refresh_against_oracle(T, B):
    """The steps beside a refresh, with one data set and several; the float64 bar of every parity test, 1e-10."""
    from paper_1107_4192_amd import synth
    p = synth.small_random(T, 70, 20, T)
    Y = np.random.default_rng(T).normal(size=(B, T, p.m))
    ks = F.KalmanSmoother(dev(p.X), dev(p.Q), dev(p.R), dev(p.x0), dev(p.P0), T_max=T)
    try:
        res = ks.run_batch(dev(Y)) if B > 1 else ks.run(dev(Y[0]))
    finally:
        ks.close()
    for b in range(B):
        xf, Pf, dPf = oracle.kf_filter(p.X, p.Q, p.R, p.x0, p.P0, Y[b])
        xs, _, dPs = oracle.rts_smooth(xf, Pf, p.Q)
        got = (res.x_filt[b], res.x_smooth[b]) if B > 1 else (res.x_filt, res.x_smooth)
        assert eps_x(got[0], xf) <= 1e-10 and eps_x(got[1], xs) <= 1e-10
    assert eps_d(res.Pdiag_filt, dPf) <= 1e-10 and eps_d(res.Pdiag_smooth, dPs) <= 1e-10
