"""Products with F where their work is divided: rows of none to 40 entries (batches of 8), N around the stripes
of 16 columns and around the 2048 up to which two rows of P share a workgroup. Filter and smoother against
the oracle with the same dense F, 1e-10 normwise as for every float64 path.
"""
import numpy as np
import pytest

import oracle
from paper_1107_4192_amd import kfmeg, synth
from _helpers import dev, eps_d, eps_x

pytestmark = pytest.mark.gpu


def run(p, F):
    n = p.N
    rp = np.concatenate([[0], np.cumsum((F != 0).sum(1))]).astype(np.int32)
    ci = np.concatenate([np.nonzero(F[i])[0] for i in range(n)]).astype(np.int32)
    v = np.concatenate([F[i][F[i] != 0] for i in range(n)])
    ks = kfmeg.KalmanSmoother(dev(p.X), dev(p.Q), dev(p.R), dev(p.x0), dev(p.P0), T_max=p.T, F=(rp, ci, v))
    try:
        res = ks.run(dev(p.Y))
    finally:
        ks.close()
    xf, Pf, _ = oracle.kf_filter(p.X, p.Q, p.R, p.x0, p.P0, p.Y, F=F)
    xs, _, dPs = oracle.rts_smooth(xf, Pf, p.Q, F=F)
    errs = (eps_x(res.x_filt, xf), eps_x(res.x_smooth, xs), eps_d(res.Pdiag_smooth, dPs))
    assert max(errs) <= 1e-10, errs


@pytest.mark.parametrize("N", [15, 16, 17, 33, 129, 143])
def test_rows_of_any_length(N):
    p = synth.small_random_F(N, N, 6, 4, 0.3)
    rng = np.random.default_rng(N)
    F = np.zeros((N, N))
    for i in range(N):
        k = min(N, [0, 1, 7, 8, 9, 16, 17, 40][i % 8])
        F[i, rng.choice(N, k, replace=False)] = rng.uniform(0.1, 0.9, k) / max(k, 1)
    run(p, F)


@pytest.mark.parametrize("N", [2047, 2049])
def test_two_rows_a_workgroup(N):
    p = synth.small_random_F(3, N, 8, 2, 0.002)
    run(p, p.F_dense())
