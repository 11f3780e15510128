"""The 128 x 128 GEMM tiles at a partial last k-tile (operands' rows padded with NaN, K on both sides of a
multiple of 16) and in the epilogue of tiles that lie inside C (in place, lower with mirror). Float64 bit for bit
against the kernel for small products, which adds in the same order; float32 against float64.
"""
import numpy as np
import pytest
import torch

from paper_1107_4192_amd import kfmeg as F

pytestmark = pytest.mark.gpu


def padded(rows, cols, g, dtype=torch.float64):
    """Rows of 16-byte multiples, NaN past the matrix, which must not reach a sum."""
    t = torch.full((rows, (cols + 3) // 4 * 4 + 4), float("nan"), dtype=dtype, device="cuda")
    t[:, :cols] = torch.randn((rows, cols), generator=g, dtype=torch.float64, device="cuda").to(dtype)
    return t


@pytest.mark.parametrize("lay", [0, 1, 2, 3])
@pytest.mark.parametrize("M,N", [(256, 128), (130, 257)])
@pytest.mark.parametrize("K", [1, 2, 3, 15, 16, 17, 31, 34, 65])
def test_partial_k_tile(lay, M, N, K):
    g = torch.Generator(device="cuda").manual_seed(K * 8 + lay)
    A = padded(K, M, g) if lay & 1 else padded(M, K, g)
    B = padded(N, K, g) if lay & 2 else padded(K, N, g)
    Cin = torch.randn((M, N), generator=g, dtype=torch.float64, device="cuda")
    for ks in (1, 2):
        want = F.kfd_gemm_small(A, B, M, N, K, lay, alpha=-0.5, beta=2.0, Cin=Cin, ksplit=ks)
        assert torch.equal(F.kfd_gemm(A, B, M, N, K, lay, alpha=-0.5, beta=2.0, Cin=Cin, ksplit=ks), want)


@pytest.mark.parametrize("lay", [0, 1, 2, 3])
@pytest.mark.parametrize("K", [1, 3, 5, 18, 35])
def test_partial_k_tile_float32(lay, K):
    """Tolerance: K products and sums of 24-bit numbers, each rounded once: 2^-23 K |A| |B| K."""
    M, N = 160, 128
    g = torch.Generator(device="cuda").manual_seed(K + 100 * lay)
    A = padded(K, M, g, torch.float32) if lay & 1 else padded(M, K, g, torch.float32)
    B = padded(N, K, g, torch.float32) if lay & 2 else padded(K, N, g, torch.float32)
    got = F.kfd_gemm(A, B, M, N, K, lay).cpu().numpy()
    a = (A[:, :M].T if lay & 1 else A[:, :K]).double().cpu().numpy()
    b = (B[:, :K].T if lay & 2 else B[:, :N]).double().cpu().numpy()
    assert np.abs(got - a @ b).max() <= 2.0 ** -23 * K * K * np.abs(a).max() * np.abs(b).max()


@pytest.mark.parametrize("n,ldc", [(256, 256), (256, 258), (256, 257), (300, 304), (384, 384)])
@pytest.mark.parametrize("flags", [0, F.G_LOWER, F.G_LOWER | F.G_MIRROR])
def test_inside_tiles_in_place(n, ldc, flags):
    """Even and odd rows of C (16-byte mirrored stores or not), C = Cin, nothing written past a row's end."""
    K = 50
    g = torch.Generator(device="cuda").manual_seed(n + ldc)
    A = padded(K, n, g)
    C0 = torch.full((n, ldc), float("nan"), dtype=torch.float64, device="cuda")
    C0[:, :n] = torch.randn((n, n), generator=g, dtype=torch.float64, device="cuda")
    C1 = C0.clone()
    F.kfd_gemm(A, A, n, n, K, 1 | flags, alpha=-1.0, beta=1.0, Cin=C0, C=C0)
    F.kfd_gemm_small(A, A, n, n, K, 1 | flags, alpha=-1.0, beta=1.0, Cin=C1, C=C1)
    assert torch.equal(C0[:, :n], C1[:, :n])
    assert torch.isnan(C0[:, n:]).all()
