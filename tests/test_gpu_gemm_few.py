"""Small dense products whose tiles are shared by four wavefronts: reductions that do not divide by four steps, ragged tiles,
both sides of the lines at 64 indices and 512 tiles, bias and accumulation."""
import pytest
import torch

from paper_2308_12093_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tb", [0, 1])
@pytest.mark.parametrize("M,N,K", [(1, 1, 64), (33, 31, 65), (31, 7, 4000), (2048, 16, 512), (3001, 7, 203), (300, 300, 95),
                                   (16384, 32, 64), (16385, 32, 64), (64, 64, 63), (100, 40, 97), (100, 40, 129)])
def test_against_float64(M, N, K, tb):
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    A, Bm = torch.randn(M, K, generator=gen, device="cuda"), torch.randn(K, N, generator=gen, device="cuda")
    bias, held = torch.randn(N, generator=gen, device="cuda"), torch.randn(M, N, generator=gen, device="cuda")
    ws = B.alloc(B.gnn_gemm_workspace_bytes(0, tb, M, N, K))
    ref = A.double() @ Bm.double()
    # one rounding per pair of indices at the most, three for the four sums, two for bias and held value
    bound = (K // 2 + 8) * 2.0 ** -24 * (A.abs().double() @ Bm.abs().double() + bias.abs() + held.abs())
    for C, b, flags, want in ((torch.empty(M, N, device="cuda"), None, 0, ref), (held.clone(), bias, 4, ref + bias + held)):
        B.gnn_gemm(0, tb, M, N, K, A, Bm.t().contiguous() if tb else Bm, C, b, flags, ws)
        assert bool(((C.double() - want).abs() <= bound).all())
