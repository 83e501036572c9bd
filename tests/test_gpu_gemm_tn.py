"""X^T H of long reductions against float64, entry by entry: tile and chunk edges, scales far apart within a column and
between columns, outliers that meet zeros, and values that are not finite."""
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
    A, H = A.double(), H.double()
    ref = A.t() @ H
    # products of two floats are exact in double: K roundings of the sums, here and in the reference, and the rounding to float
    bound = 2.0 ** -24 * ref.abs() + 2 * A.shape[0] * 2.0 ** -53 * (A.abs().t() @ H.abs()) + 2.0 ** -150
    assert bool(((C.double() - ref).abs() <= bound).all()), name


def normal(seed, *shape):
    return torch.randn(*shape, generator=torch.Generator(device="cuda").manual_seed(seed), device="cuda")


@pytest.mark.parametrize("M,N,K", [(65, 65, 8192), (128, 128, 8193), (129, 200, 8223), (100, 256, 20001), (256, 96, 16415),
                                   (70, 68, 140000), (512, 300, 9000), (1024, 1024, 70003), (2100, 2050, 8200),
                                   (2100, 2050, 100), (64, 40000, 512)])
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
    check(product(A, H), A, H, kind)


@pytest.mark.parametrize("by", [1e3, 1e6, 2.0 ** 40])
@pytest.mark.parametrize("kind", ["one row", "hubs", "both halves", "later rows"])
def test_outliers_that_meet_zeros(kind, by):
    """Rows that are large in one operand and zero in the other must not cost the rest of the sum a bit."""
    K, M, N = 16384, 80, 72
    A, H = normal(11, K, M), normal(12, K, N)
    if kind == "one row":
        A[100] *= by
        H[100] = 0
    elif kind == "hubs":
        A[5::256] *= by
        H[5::256] = 0
        H[77::256] *= by
        A[77::256] = 0
    elif kind == "both halves":                             # half of each operand masked, one outlier row in each
        A[normal(13, K, M) < 0] = 0
        H[normal(14, K, N) < 0] = 0
        A[3000] *= by
        H[3001] *= by
    else:                                                   # small rows first, larger ones where the other operand is zero
        A[:K // 2] /= by
        H[K // 2:] = 0
    check(product(A, H), A, H, kind)


@pytest.mark.parametrize("kind", ["student", "lognormal"])
def test_heavy_tails(kind):
    K, M, N = 16384, 100, 72
    A, H = normal(15, K, M), normal(16, K, N)
    if kind == "student":                                   # two degrees of freedom
        A /= ((normal(17, K, M) ** 2 + normal(18, K, M) ** 2) / 2).sqrt()
        H /= ((normal(19, K, N) ** 2 + normal(20, K, N) ** 2) / 2).sqrt()
    else:                                                   # a standard deviation of a decade
        A *= 10.0 ** normal(17, K, M)
        H *= 10.0 ** normal(18, K, N)
    check(product(A, H), A, H, kind)


def test_values_that_are_not_finite():
    K, M, N = 9000, 70, 80
    A, H = normal(6, K, M), normal(7, K, N).abs() + 0.5
    A[4000, 3] = float("inf")
    A[8999, 5] = float("nan")
    A[:, 9] *= 1e-36
    C = product(A, H)
    assert bool((C[3] == float("inf")).all()) and bool(torch.isnan(C[5]).all())
    fine = [i for i in range(M) if i not in (3, 5)]
    check(C[fine], A[:, fine], H)


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


@pytest.mark.parametrize("M,N", [(1, 1), (5, 7), (16, 3), (300, 500)])
def test_no_rows_need_no_room(M, N):
    """Zero rows: zeros, and nothing written behind the workspace that the query asks for."""
    need = B.gnn_gemm_workspace_bytes(1, 0, M, N, 0)
    memory = torch.full((need + 16 * M * N + 256,), 7, dtype=torch.uint8, device="cuda")
    A, H, C = torch.empty(1, M, device="cuda"), torch.empty(1, N, device="cuda"), torch.full((M, N), float("nan"), device="cuda")
    B.gnn_gemm(1, 0, M, N, 0, A, H, C, None, 0, memory[:need])
    assert bool((C == 0).all()) and bool((memory[need:] == 7).all())
