"""X^T H of long reductions on five digits per float, against float64: tile, step and chunk edges, growing and sparse
columns, scales far apart, and values that no exponent holds."""
import numpy as np
import pytest
import torch

from paper_2308_12093_amd import binding as B

pytestmark = pytest.mark.gpu


def product(A, H):
    (K, M), N = A.shape, H.shape[1]
    C = torch.empty(M, N, device="cuda")
    B.gnn_gemm(1, 0, M, N, K, A, H, C, None, 0, B.alloc(B.gnn_gemm_workspace_bytes(1, 0, M, N, K)))
    return C


def check(C, A, H, name=""):
    ref = A.double().t() @ H.double()
    # the rounding to float, and per product of two columns' largest magnitudes: an exponent is at most 2^4 above the
    # largest magnitude, so the fifth digit rounds by 2^-35 (both operands), and the digit products left out
    # (i + j >= 7, four of 2^14 * 256 * 2^-60 * 2^8 and their tail) stay below 2^-27
    top = A.double().abs().amax(0)[:, None] * H.double().abs().amax(0)[None, :]
    bound = 2.0 ** -23.9 * ref.abs() + A.shape[0] * 2.0 ** -27 * top
    assert bool(((C.double() - ref).abs() <= bound).all()), name
    # in the mean the digits leave nothing beyond the rounding to float, at most 2^-24 / sqrt(3) = 3.4e-8
    assert float((C.double() - ref).norm() / ref.norm()) < 4e-8, name


def normal(seed, *shape):
    return torch.randn(*shape, generator=torch.Generator(device="cuda").manual_seed(seed), device="cuda")


# the last two: several folds of 512 steps in a chunk; one chunk per tile
@pytest.mark.parametrize("M,N,K", [(65, 65, 8192), (128, 128, 8193), (129, 200, 8223), (100, 256, 20001), (256, 96, 16415),
                                   (70, 68, 140000), (512, 300, 9000), (1024, 1024, 70003), (2100, 2050, 8200)])
def test_edges(M, N, K):
    A, H = normal(M, K, M), normal(N, K, N)
    check(product(A, H), A, H)


@pytest.mark.parametrize("by", [1, 2])
def test_unaligned_operands(by):
    K, M, N = 9001, 72, 132
    A = torch.empty(K * M + by, device="cuda")[by:].view(K, M).copy_(normal(1, K, M))
    H = torch.empty(K * N + by, device="cuda")[by:].view(K, N).copy_(normal(2, K, N))
    check(product(A, H), A, H)


@pytest.mark.parametrize("kind", ["growing", "sparse", "scales", "positive", "bursts"])
def test_exponents(kind):
    K, M, N = 20000, 100, 130
    A, H = normal(3, K, M), normal(4, K, N)
    at = torch.arange(K, device="cuda", dtype=torch.float32)[:, None]
    if kind == "growing":
        A *= 2.0 ** (at / 400)
    elif kind == "sparse":                                  # most columns begin with zeros, some hold nothing
        A *= (normal(5, K, M) > 3).float()
        A[:, 7] = 0
        H[:, 11] = 0
    elif kind == "scales":
        A *= 10.0 ** torch.linspace(-12, 12, M, device="cuda")
        H *= 10.0 ** torch.linspace(14, -14, N, device="cuda")
    elif kind == "positive":
        A.abs_(), H.abs_()
    else:
        A[K // 3:K // 3 + 5] *= 1e4
        H[::997] *= 1e3
    C = product(A, H)
    if kind == "scales":                                    # column by column, on one scale
        a, h = A.abs().amax(0), H.abs().amax(0)
        C, A, H = C.double() / a.double()[:, None] / h.double()[None, :], A.double() / a.double(), H.double() / h.double()
    check(C, A, H, kind)


def test_values_without_an_exponent():
    K, M, N = 9000, 70, 80
    A, H = normal(6, K, M), normal(7, K, N).abs() + 0.5
    A[4000, 3] = float("inf")
    A[8999, 5] = float("nan")
    A[:, 9] *= 1e-36
    C = product(A, H)
    ref = A.double().t() @ H.double()
    assert bool((C[3] == float("inf")).all()) and bool(torch.isnan(C[5]).all())
    fine = [i for i in range(M) if i not in (3, 5)]
    assert bool(((C.double() - ref)[fine].abs() <= 2.0 ** -23 * ref[fine].abs() + 1e-12 * A.double().abs().amax(0)[fine][:, None]).all())


@pytest.mark.parametrize("n", [8192, 9001])
def test_masked_gradient(n):
    """First layer of a network: the ReLU mask goes with the gradient; A' is the identity."""
    m, k = 70, 300
    ids = torch.arange(n + 1, dtype=torch.int32, device="cuda")
    g = B.Graph(n, ids, ids[:n].clone(), torch.ones(n, device="cuda"), ids[:n].clone(), symmetric=True)
    plan = B.Plan(B.GNN_LAYER_GCN, n, n, m, k, need_input_grad=False, fuse_relu=True,
                  order=B.GNN_ORDER_PROPAGATE_FIRST, bwd=B.GNN_BWD_SPLIT_PROPAGATE)
    X, W, dY = normal(8, n, m), normal(9, m, k) * 0.1, normal(10, n, k)
    Y, dW = torch.empty(n, k, device="cuda"), torch.empty(m, k, device="cuda")
    cache, ws = B.alloc(plan.info.cache_bytes), B.alloc(plan.info.workspace_bytes)
    B.gcn_layer_fwd(plan, g, X, W, None, Y, cache, ws)
    B.gcn_layer_bwd(plan, g, X, W, Y, dY, dW, None, None, cache, ws)
    check(dW, X, dY * (Y > 0))
