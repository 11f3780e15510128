"""What a budget buys: a plan keeps every P_{t|t} wherever the store and the gains' workspace fit, also where the
sensor-space smoother's factors do not fit beside them."""
import pytest
import torch

import oracle
from paper_1107_4192_amd import kfmeg as F, synth
from _helpers import dev, eps_d, eps_x

pytestmark = pytest.mark.gpu


def plan(p, **opt):
    return F.KalmanSmoother(dev(p.X), dev(p.Q), dev(p.R), dev(p.x0), dev(p.P0), T_max=p.T, **opt)


@pytest.mark.parametrize("N,m,T", [(64, 10, 120), (96, 8, 200), (60, 30, 120)])
@pytest.mark.parametrize("extra", [0, 64 << 10])
def test_full_store_before_the_factors(N, m, T, extra):
    """The smallest budget that an explicit full store (stride 1) accepts is a full store without it too, so that
    kf_smooth_assoc runs (it is refused on checkpoints); the smoother agrees with the oracle at 1e-10."""
    p = synth.small_random(5, N, m, T)
    lo, hi = 1 << 20, 2 * F.kf_plan_bytes(N, m, T)
    while hi - lo > 4096:
        mid = (lo + hi) // 2
        try:
            plan(p, hbm_budget_bytes=mid, checkpoint_stride=1).close()
            hi = mid
        except F.KFError:
            lo = mid
    xf, Pf, _ = oracle.kf_filter(p.X, p.Q, p.R, p.x0, p.P0, p.Y)
    xs, _, dPs = oracle.rts_smooth(xf, Pf, p.Q)
    ks = plan(p, hbm_budget_bytes=hi + extra)
    try:
        r = ks.run(dev(p.Y))
        a = ks.smooth_assoc(ks.filter(dev(p.Y)))
    finally:
        ks.close()
    for got in (r, a):
        assert eps_x(got.x_smooth, xs) <= 1e-10 and eps_d(got.Pdiag_smooth, dPs) <= 1e-10
