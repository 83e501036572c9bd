"""X^T H at the edges of the tiles of 48, 80, 96 and 112 outputs and of short chunks, entry by entry against float64."""
import pytest
import torch

from paper_2308_12093_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [33, 97, 2048, 30011])
@pytest.mark.parametrize("M,N", [(128, 48), (129, 47), (256, 49), (128, 80), (127, 79), (260, 81), (96, 96), (95, 97), (192, 190),
                                 (128, 112), (250, 111), (256, 224), (300, 300), (512, 512), (17, 15), (64, 33)])
def test_tiles(M, N, K):
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    A, H = torch.randn(K, M, generator=gen, device="cuda"), torch.randn(K, N, generator=gen, device="cuda")
    C = torch.empty(M, N, device="cuda")
    B.gnn_gemm(1, 0, M, N, K, A, H, C, None, 0, B.alloc(B.gnn_gemm_workspace_bytes(1, 0, M, N, K)))
    ref = A.double().t() @ H.double()
    # products of two floats are exact in double: K roundings of the sums, here and in the reference, and that to float
    bound = 2.0 ** -24 * ref.abs() + 2 * K * 2.0 ** -53 * (A.double().abs().t() @ H.double().abs()) + 2.0 ** -150
    assert bool(((C.double() - ref).abs() <= bound).all())
