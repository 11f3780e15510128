"""The sensor-space filter and smoother (float64, F = I, 2 m <= N) against the oracle's N x N recursions.

Horizons sit at the edges of its 16-step chunks, sizes at the edges of its shape rule (2 m = N; one
sensor more takes the gains instead) and of the 32-wide product tiles. Tolerance: the float64 bar of every
parity test, 1e-10 normwise per step; the problems have condition numbers of about 10, so both sides are
within about T * N * cond * 1e-16 = 3e-12 of the exact result.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_1107_4192_amd import kfmeg, synth
from _helpers import dev, eps_P, eps_d, eps_x, to_np

pytestmark = pytest.mark.gpu
TOL = 1e-10


def plan(p, **opt):
    return kfmeg.KalmanSmoother(dev(p.X), dev(p.Q), dev(p.R), dev(p.x0), dev(p.P0), T_max=p.T, **opt)


def reference(p):
    xf, Pf, dPf = oracle.kf_filter(p.X, p.Q, p.R, p.x0, p.P0, p.Y)
    xs, Ps, dPs = oracle.rts_smooth(xf, Pf, p.Q)
    return xf, Pf, dPf, xs, Ps, dPs


@pytest.mark.parametrize("N,m,T", [(2, 1, 3), (64, 32, 1), (64, 32, 2), (66, 33, 16), (66, 33, 17), (65, 33, 17),
                                   (130, 65, 18), (70, 7, 33), (70, 31, 34), (100, 17, 49)])
def test_against_oracle(N, m, T):
    p = synth.small_random(N + m + T, N, m, T)        # dense P0 and Q
    xf, Pf, dPf, xs, Ps, dPs = reference(p)
    ks = plan(p)
    try:
        res = ks.run(dev(p.Y))
        full = ks.run(dev(p.Y), want_full=True)       # P_{t|T} itself: another route to the variances
        P1 = ks.filtered_cov(T)
        only = torch.empty_like(res.x_smooth)
        kfmeg.kf_smooth(ks.plan, only)                # means alone
    finally:
        ks.close()
    assert eps_x(res.x_filt, xf) <= TOL and eps_d(res.Pdiag_filt, dPf) <= TOL
    assert eps_x(res.x_smooth, xs) <= TOL and eps_d(res.Pdiag_smooth, dPs) <= TOL
    assert eps_P(full.P_smooth, Ps) <= TOL and eps_d(full.Pdiag_smooth, dPs) <= TOL
    assert eps_P(P1, Pf[T - 1]) <= TOL
    assert torch.equal(full.P_smooth, full.P_smooth.transpose(1, 2))
    assert torch.equal(only, res.x_smooth) and torch.equal(full.x_smooth, res.x_smooth)


@pytest.mark.parametrize("stride", [2, 5, 40])
def test_checkpointed_bitwise(stride):
    p = synth.small_random(3, 90, 20, 37)
    a, b = plan(p), plan(p, checkpoint_stride=stride)
    try:
        ra, rb = a.run(dev(p.Y), want_full=True), b.run(dev(p.Y), want_full=True)
        for t in (1, 2, 20, 36, 37):
            assert torch.equal(a.filtered_cov(t), b.filtered_cov(t))
    finally:
        a.close()
        b.close()
    for k in ("x_filt", "Pdiag_filt", "x_smooth", "Pdiag_smooth", "P_smooth"):
        assert torch.equal(getattr(ra, k), getattr(rb, k))


def test_data_sets_means_only_and_shorter_calls():
    """Several data sets through one plan, then fewer, the mean-only smoother, and a horizon below T_max."""
    B, T = 5, 20
    p = synth.small_random(9, 80, 24, T)
    Y = np.random.default_rng(1).normal(size=(B, T, p.m))
    ks = plan(p, keep_gain_factors=True)
    try:
        r = ks.run_batch(dev(Y))
        means = torch.empty_like(r.x_filt)
        kfmeg.kf_smooth_means(ks.plan, means)
        for b in range(B):
            p.Y = Y[b]
            xf, _, dPf, xs, _, dPs = reference(p)
            assert eps_x(r.x_filt[b], xf) <= TOL and eps_x(r.x_smooth[b], xs) <= TOL
            assert eps_x(means[b], xs) <= TOL
        assert eps_d(r.Pdiag_smooth, dPs) <= TOL
        p.Y = Y[2][:11]                               # one data set again, 11 of 20 steps
        xf, _, dPf, xs, _, dPs = reference(p)
        s = ks.run(dev(p.Y))
        assert eps_x(s.x_smooth, xs) <= TOL and eps_d(s.Pdiag_smooth, dPs) <= TOL
        assert eps_x(ks.smooth_means(s).x_smooth, xs) <= TOL
    finally:
        ks.close()


def test_certified_and_factored_positive_definiteness_agree():
    """The bounds that replace the factorisation of P_{t+1|t} (diagonal P0) and the factorisation itself
    (dense P0: no bound) give the same results; a Q whose negative part the sensors never see is refused."""
    p = synth.tiny(T=9, N=120, m=20)
    xf, _, _, xs, _, dPs = reference(p)
    ks = plan(p)
    try:
        r = ks.run(dev(p.Y))
    finally:
        ks.close()
    assert eps_x(r.x_smooth, xs) <= TOL and eps_d(r.Pdiag_smooth, dPs) <= TOL
    p.Q = p.Q.copy()
    v = np.linalg.svd(p.X)[2][-1]
    p.Q -= 0.4 * np.outer(v, v)                       # diagonal P0, but Q has a negative eigenvalue
    p.Q = (p.Q + p.Q.T) / 2
    ks = plan(p)
    try:
        f = ks.filter(dev(p.Y))
        with pytest.raises(kfmeg.KFError) as ei:
            ks.smooth(f)
    finally:
        ks.close()
    assert ei.value.status == kfmeg.KF_ENOTPD and "P_{t+1|t}" in str(ei.value) and "t=2 " in str(ei.value)


def test_budget_without_room_for_the_factors_still_smooths():
    """A budget that holds the checkpointed plan but not every step's factors smooths through the gains."""
    p = synth.small_random(5, 60, 30, 120)
    ref = reference(p)
    lo, hi = 1 << 20, kfmeg.kf_plan_bytes(p.N, p.m, p.T)
    while hi - lo > 4096:                             # the smallest budget that is accepted
        mid = (lo + hi) // 2
        try:
            plan(p, hbm_budget_bytes=mid).close()
            hi = mid
        except kfmeg.KFError:
            lo = mid
    ks = plan(p, hbm_budget_bytes=hi)
    try:
        r = ks.run(dev(p.Y))
    finally:
        ks.close()
    assert eps_x(r.x_smooth, ref[3]) <= TOL and eps_d(r.Pdiag_smooth, ref[5]) <= TOL
    assert eps_d(to_np(r.Pdiag_filt), ref[2]) <= TOL
