"""kf_smooth reports a P_{t+1|t} that is not positive definite in its m x m form too (float64, F = I, 2 m <= N), where
nothing else needs its factor: whatever the model's bounds say, with every P_{t|t} stored and with checkpoints, and with
the lowest failing step in the message.
"""
import numpy as np
import pytest
import torch

from paper_1107_4192_amd import kfmeg as F
from _helpers import dev

pytestmark = pytest.mark.gpu


def refused_at(X, Q, R, P0, T, step, **opt):
    N, m = X.shape[1], X.shape[0]
    Y = np.random.default_rng(T).normal(size=(T, m)) * 1e-3
    ks = F.KalmanSmoother(dev(X), dev(Q), dev(R), dev(np.zeros(N)), dev(P0), T_max=T, **opt)
    try:
        f = ks.filter(dev(Y))
        with pytest.raises(F.KFError) as ei:
            ks.smooth(f)
        with pytest.raises(F.KFError):            # and again: nothing is remembered from the first call
            ks.smooth(f)
    finally:
        ks.close()
    msg = str(ei.value)
    assert ei.value.status == F.KF_ENOTPD and "P_{t+1|t}" in msg and f"t={step} " in msg, msg


@pytest.mark.parametrize("seed", [0, 1, 2])
@pytest.mark.parametrize("stride", [0, 2])
def test_rounding_beyond_a_small_q(seed, stride):
    """P_0 = I and Q = 2e-12 I are as definite as can be, but at cond(S) = 1e10 the first update leaves -1e-9 or less."""
    N, m, T = 64, 12, 4
    rng = np.random.default_rng(seed)
    U, V = np.linalg.qr(rng.normal(size=(m, m)))[0], np.linalg.qr(rng.normal(size=(N, m)))[0]
    X = (U * np.geomspace(1.0, 1e-5, m)) @ V.T
    refused_at(X, 2e-12 * np.eye(N), 1e-18 * np.eye(m), np.eye(N), T, 1, checkpoint_stride=stride)


@pytest.mark.parametrize("N,m,T,stride", [(90, 20, 30, 0), (90, 20, 30, 4), (90, 20, 30, 7), (90, 20, 30, 30), (90, 20, 15, 2),
                                          (24, 12, 30, 5)])
def test_lowest_failing_step(N, m, T, stride):
    """Q's eigenvalue along an unseen direction is -0.07: P_{t+1|t} has 1 - 0.07 (t + 1) there, negative from t = 14 on."""
    rng = np.random.default_rng(N + T)
    X = rng.normal(size=(m, N)) / np.sqrt(N)
    v = np.linalg.svd(X)[2][-1]
    Q = 0.01 * np.eye(N) - 0.08 * np.outer(v, v)
    refused_at(X, (Q + Q.T) / 2, 1e-2 * np.eye(m), np.eye(N), T, 14, checkpoint_stride=stride)


def test_one_step_needs_no_prediction():
    """T = 1 has no P_{t+1|t}."""
    N, m = 24, 6
    X = np.random.default_rng(0).normal(size=(m, N))
    ks = F.KalmanSmoother(dev(X), dev(-2.0 * np.diag(np.arange(N) == N - 1.0)), dev(np.eye(m) * 1e3), dev(np.zeros(N)),
                          dev(4.0 * np.eye(N)), T_max=1)
    try:
        r = ks.run(dev(np.ones((1, m))))
        assert torch.equal(r.x_smooth, r.x_filt) and torch.equal(r.Pdiag_smooth, r.Pdiag_filt)
    finally:
        ks.close()
