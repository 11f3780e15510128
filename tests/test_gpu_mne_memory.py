"""The allocating minimum-norm entry points give their workspace back: no more than 128 MiB stays with the library between
calls, whatever a call needed and however many ran at once."""
import threading

import pytest
import torch

from paper_1107_4192_amd import kfmeg as F

pytestmark = pytest.mark.gpu
KEEP, SLACK = 128 << 20, 8 << 20


def model(N, m, T):
    g = torch.Generator(device="cuda").manual_seed(N + m)
    X = torch.randn(m, N, generator=g, dtype=torch.float64, device="cuda")
    Y = torch.randn(T, m, generator=g, dtype=torch.float64, device="cuda")
    return X, torch.eye(N, dtype=torch.float64, device="cuda"), torch.eye(m, dtype=torch.float64, device="cuda"), Y


@pytest.mark.parametrize("T", [100_000, 400_000])      # workspaces of 98 and 392 MiB
def test_workspace_is_given_back(T):
    X, C, R, Y = model(32, 64, T)
    J = torch.empty(T, 32, dtype=torch.float64, device="cuda")
    F.mne_solve(X, C, R, Y[:10].contiguous())
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    F.mne_solve(X, C, R, Y, J)
    assert before - torch.cuda.mem_get_info()[0] <= KEEP + SLACK
    x0, Q = F.kf_init_from_mne(X, C, R, Y, 1e-3)
    assert before - torch.cuda.mem_get_info()[0] <= KEEP + SLACK
    assert bool(torch.isfinite(J).all()) and torch.equal(x0, J[0])


def test_workspaces_of_threads_are_given_back():
    X, C, R, Y = model(32, 64, 90_000)                 # 88 MiB each
    want = F.mne_solve(X, C, R, Y)
    torch.cuda.synchronize()
    outs = [torch.empty_like(want) for _ in range(4)]
    before = torch.cuda.mem_get_info()[0]

    def work(k):
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.default_stream())
        for _ in range(3):
            F.mne_solve(X, C, R, Y, outs[k], stream=s)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    F.mne_solve(X, C, R, Y[:10].contiguous())          # the next call finds the surplus, if any is left
    assert before - torch.cuda.mem_get_info()[0] <= KEEP + 4 * SLACK
    assert all(torch.equal(o, want) for o in outs)
