"""Products on split parts around the lines between blocks that keep the parts of their columns and blocks that do not (which is which
is tested in test_gpu_gemm_routes.py): several tiles a wavefront, ragged ends, several column tiles, values that the parts cannot
hold, two operand pairs."""
import pytest
import torch

from paper_2308_12093_amd import binding as B

pytestmark = pytest.mark.gpu
BIG = (1 << 19) + 37


def product(M, N, K, A, Bm, tb, bias=None, relu=0, C=None):
    C = torch.empty(M, N, device="cuda") if C is None else C
    B.gnn_gemm(0, tb, M, N, K, A, Bm.t().contiguous() if tb else Bm, C, bias, relu, B.alloc(B.gnn_gemm_workspace_bytes(0, tb, M, N, K)))
    return C


@pytest.mark.parametrize("tb", [0, 1])
@pytest.mark.parametrize("M,N,K", [(BIG, 64, 64), (BIG, 47, 130), (BIG, 33, 200), (BIG, 128, 50), (BIG, 200, 90), (BIG, 65, 190),
                                   (BIG, 300, 20), (1 << 21, 128, 4), (1 << 20, 256, 32), (65536, 64, 16), (65536, 64, 20),
                                   (33000, 128, 32), (40001, 70, 4), (66001, 30, 64), (1 << 18, 64, 33)])
def test_against_float64(M, N, K, tb):
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    A, Bm = torch.randn(M, K, generator=gen, device="cuda"), torch.randn(K, N, generator=gen, device="cuda")
    bias, held = torch.randn(N, generator=gen, device="cuda"), torch.randn(M, N, generator=gen, device="cuda")
    ref = A.double() @ Bm.double()
    # at most eight roundings of the sum per 16 indices, the dropped products (2^-26) and the rounding of bias and held value
    bound = (8 * ((K + 15) // 16) + 4) * 2.0 ** -24 * (A.abs().double() @ Bm.abs().double())
    assert bool(((product(M, N, K, A, Bm, tb).double() - ref).abs() <= bound).all())
    bound += 2.0 ** -22 * (ref.abs() + bias.abs() + held.abs())
    # a ReLU decides signs: the same shape on the fp32 instruction
    assert bool(((product(M, N, K, A, Bm, tb, bias, 1).double() - torch.relu(ref + bias)).abs() <= bound).all())
    assert bool(((product(M, N, K, A, Bm, tb, bias, 4, held.clone()).double() - (ref + bias + held)).abs() <= bound).all())


@pytest.mark.parametrize("M,N,K", [(BIG, 64, 70), (BIG, 130, 40), (70000, 40, 60), (60000, 40, 60), (BIG, 160, 100), (BIG, 47, 300)])
def test_values_the_parts_cannot_hold(M, N, K):
    gen = torch.Generator(device="cuda").manual_seed(N)
    A, Bm = torch.randn(M, K, generator=gen, device="cuda"), torch.randn(K, N, generator=gen, device="cuda").abs() + 0.5
    A[::3] *= 2.0 ** -(85.0 + torch.arange(A[::3].shape[0], device="cuda") % 65)[:, None]       # rows of tiny values
    A[1::21] = 0.0
    A[2::33, :32] *= 2.0 ** -140
    Bm[:, 33] *= 1e-34                                      # third parts below the bf16 range
    A[5::1000, 0], A[7::1000, 1] = float("inf"), float("nan")
    C, ref = product(M, N, K, A, Bm, 0).double(), A.double() @ Bm.double()
    bound = (8 * ((K + 15) // 16) + 4) * 2.0 ** -24 * (A.abs().double() @ Bm.abs().double()) + K * 2.0 ** -149
    fine = torch.isfinite(ref)
    assert bool(((C - ref).abs() <= bound)[fine].all())
    assert bool((C[5::1000] == ref[5::1000])[torch.isinf(ref[5::1000])].all()) and bool(torch.isnan(C[7::1000]).all())


def test_two_operand_pairs():
    """GraphSAGE over the identity: Y = X (Ws + Wn)."""
    n, m, k = BIG, 40, 70
    gen = torch.Generator(device="cuda").manual_seed(3)
    ids = torch.arange(n + 1, dtype=torch.int32, device="cuda")
    g = B.Graph(n, ids, ids[:n].clone(), torch.ones(n, device="cuda"), ids[:n].clone(), symmetric=True)
    plan = B.Plan(B.GNN_LAYER_SAGE, n, n, m, k, order=B.GNN_ORDER_PROPAGATE_FIRST)
    X, Ws, Wn = (torch.randn(*s, generator=gen, device="cuda") for s in ((n, m), (m, k), (m, k)))
    Y = torch.empty(n, k, device="cuda")
    B.sage_layer_fwd(plan, g, X, Ws, Wn, None, Y, B.alloc(plan.info.cache_bytes), B.alloc(plan.info.workspace_bytes))
    ref = X.double() @ Ws.double() + X.double() @ Wn.double()
    bound = (8 * 6 + 4) * 2.0 ** -24 * (X.abs().double() @ (Ws.abs() + Wn.abs()).double())
    assert bool(((Y.double() - ref).abs() <= bound).all())
