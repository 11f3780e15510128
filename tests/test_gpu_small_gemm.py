"""The small-product GEMM kernel against the 128 x 128 tile kernels, bit for bit: both add the products of an
output in the order of k, so any difference is an indexing fault. Sizes sit at the edges of its
32 x 32 tiles and 32-wide k chunks, over all layouts, triangular operands, splits and odd leading
dimensions (unaligned loads)."""
import numpy as np
import pytest
import torch

from paper_1107_4192_amd import kfmeg as F

pytestmark = pytest.mark.gpu

TRI = {"A lower": F.G_ALOWER, "A upper": F.G_AUPPER, "B lower": F.G_BLOWER, "B upper": F.G_BUPPER}


def padded(rows, cols, pad, g):
    t = torch.full((rows, cols + pad), float("nan"), dtype=torch.float64, device="cuda")
    t[:, :cols] = torch.randn((rows, cols), generator=g, dtype=torch.float64, device="cuda")
    return t


@pytest.mark.parametrize("lay", [0, 1, 2, 3])
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (31, 33, 32), (33, 31, 31), (32, 32, 33), (64, 65, 64), (70, 5, 97),
                                   (8, 200, 130), (100, 100, 4)])
@pytest.mark.parametrize("pad", [0, 3])
def test_layouts_bitwise(lay, M, N, K, pad):
    g = torch.Generator(device="cuda").manual_seed(M * 7 + N * 3 + K + lay)
    A = padded(K, M, pad, g) if lay & 1 else padded(M, K, pad, g)
    B = padded(N, K, pad, g) if lay & 2 else padded(K, N, pad, g)
    Cin = torch.randn((M, N), generator=g, dtype=torch.float64, device="cuda")
    for ks in (1, 3):
        want = F.kfd_gemm(A, B, M, N, K, lay, alpha=-0.5, beta=2.0, Cin=Cin, ksplit=ks)
        got = F.kfd_gemm_small(A, B, M, N, K, lay, alpha=-0.5, beta=2.0, Cin=Cin, ksplit=ks)
        assert torch.equal(got, want)
    ref = -0.5 * (A[:, :M].T if lay & 1 else A[:, :K]).cpu().numpy() @ \
        (B[:, :K].T if lay & 2 else B[:, :N]).cpu().numpy() + 2.0 * Cin.cpu().numpy()
    # K + 2 roundings of terms of size at most |A| |B| row sums
    scale = float(A[:, :M if lay & 1 else K].abs().max() * B[:, :K if lay & 2 else N].abs().max()) * K + 10.0
    assert np.abs(got.cpu().numpy() - ref).max() <= 2.3e-16 * (K + 2) * scale


@pytest.mark.parametrize("tri", list(TRI))
@pytest.mark.parametrize("n", [31, 64, 100, 161])
def test_triangular_and_lower_bitwise(tri, n):
    g = torch.Generator(device="cuda").manual_seed(n)
    A, B = padded(n, n, 0, g), padded(n, n, 0, g)
    up = "upper" in tri
    if tri[0] == "A":
        A = torch.triu(A) if up else torch.tril(A)
    else:
        B = torch.triu(B) if up else torch.tril(B)
    for flags in (0, F.G_LOWER, F.G_LOWER | F.G_MIRROR):
        C0, C1 = (torch.zeros((n, n), dtype=torch.float64, device="cuda") for _ in range(2))
        F.kfd_gemm(A.contiguous(), B.contiguous(), n, n, n, TRI[tri] | flags, C=C0)
        F.kfd_gemm_small(A.contiguous(), B.contiguous(), n, n, n, TRI[tri] | flags, C=C1)
        assert torch.equal(C0, C1)
