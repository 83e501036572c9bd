"""SpMM of graphs large enough for long rows to be cut into pieces: row lengths at the edges of pieces and classes, columns
in any order, ragged and wide operands, values that are not finite, and the products that stay with the segments."""
import pytest
import torch

from paper_2308_12093_amd import binding as B

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 2, 8, 9, 16, 17, 33, 64, 65, 127, 128, 129, 143, 144, 191, 192, 193, 255, 256, 1000, 4097, 65535, 65600, 200000]


def matrix(seed, n, nnz, hubs=True, ordered=True):
    """CSR on the device: the lengths of EDGES first and last, the others alike but a few thousand long ones."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    d = torch.full((n,), 3, dtype=torch.int64, device="cuda")
    if hubs:
        d[torch.randperm(n, generator=gen, device="cuda")[:4000]] = max(128, (nnz - 3 * n - 2 * sum(EDGES)) // 4000)
        edges = torch.tensor(EDGES, device="cuda")
        d[:len(EDGES)], d[n - len(EDGES):] = edges, edges.flip(0)
    else:
        d[:] = nnz // n
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    rowptr[1:] = d.cumsum(0)
    q = int(rowptr[-1])
    row = torch.repeat_interleave(torch.arange(n, device="cuda"), d)
    col = torch.randint(0, n, (q,), generator=gen, device="cuda")
    if ordered:
        col = (torch.sort(row * n + col).values - row * n)
    val = torch.randn(q, generator=gen, device="cuda")
    return rowptr.int(), col.int(), val, row.int(), gen


def run(n, rowptr, col, val, erow, X, bias=None, relu=False):
    f, q = X.shape[1], col.numel()
    C = torch.full((n, f), float("nan"), device="cuda")
    B.gnn_spmm_csr(n, q, rowptr, col, val, erow, X, f, C, bias, relu,
                   workspace=B.alloc(B.gnn_spmm_workspace_bytes(n, q, f)))
    return C


def check(C, n, col, val, erow, X, bias=None, relu=False):
    ref = torch.zeros(n, X.shape[1], dtype=torch.float64, device="cuda")
    mag = torch.zeros_like(ref)
    X = X.double()
    piece = max(1, (1 << 28) // X.shape[1])
    for lo in range(0, col.numel(), piece):
        t = X[col[lo:lo + piece].long()] * val[lo:lo + piece, None].double()
        ref.index_add_(0, erow[lo:lo + piece].long(), t)
        mag.index_add_(0, erow[lo:lo + piece].long(), t.abs_())
    if bias is not None:
        ref += bias.double()
        mag += bias.double().abs()
    if relu:
        ref.clamp_(min=0)
    # roundings on the way of a product: its chain in a piece (fewer than 160), the partials of one of four sums of a slot
    # (1024 / 4 at most), the tree, the bias
    assert bool(((C.double() - ref).abs() <= 430 * 2.0 ** -24 * mag).all())


@pytest.mark.parametrize("f,nnz,ordered,relu", [(64, 32_000_000, True, True), (47, 43_000_000, True, False),
                                                (17, 120_000_000, True, True), (100, 21_000_000, False, False),
                                                (260, 8_000_000, True, True), (601, 4_000_000, False, False)])
def test_row_lengths(f, nnz, ordered, relu):
    n = 70001
    rowptr, col, val, erow, gen = matrix(f, n, nnz, ordered=ordered)
    assert col.numel() * f >= 2_000_000_000
    X, bias = torch.randn(n, f, generator=gen, device="cuda"), torch.randn(f, generator=gen, device="cuda")
    C = run(n, rowptr, col, val, erow, X, bias, relu)
    check(C, n, col, val, erow, X, bias, relu)
    assert torch.equal(C, run(n, rowptr, col, val, erow, X, bias, relu))


def test_operand_beyond_32_bit_offsets():
    n, f = (1 << 22) + 3, 260
    rowptr, col, val, erow, gen = matrix(1, n, 24_000_000)
    X = torch.randn(n, f, generator=gen, device="cuda")
    check(run(n, rowptr, col, val, erow, X), n, col, val, erow, X)


def test_not_finite_only_where_it_is_stored():
    n, f = 70001, 64
    rowptr, col, val, erow, gen = matrix(2, n, 32_000_000)
    X = torch.randn(n, f, generator=gen, device="cuda")
    X[0], X[123], X[n - 1] = float("inf"), float("nan"), float("inf")
    C = run(n, rowptr, col, val, erow, X)
    held = torch.zeros(n, dtype=torch.bool, device="cuda")
    held[erow[(col == 0) | (col == 123) | (col == n - 1)].long()] = True
    assert torch.equal(~torch.isfinite(C).all(1), held)


def test_without_long_rows_the_segments_do_it():
    n, f = 300_000, 100
    rowptr, col, val, erow, gen = matrix(3, n, 21_000_000, hubs=False)
    X = torch.randn(n, f, generator=gen, device="cuda")
    C, S = run(n, rowptr, col, val, erow, X), torch.empty(n, f, device="cuda")
    B.gnn_spmm_csr_static(n, col.numel(), rowptr, col, val, erow, X, f, S)
    assert torch.equal(C, S)
    check(C, n, col, val, erow, X)


def test_capture():
    n, f = 70001, 64
    rowptr, col, val, erow, gen = matrix(4, n, 32_000_000)
    X, C = torch.randn(n, f, generator=gen, device="cuda"), torch.empty(n, f, device="cuda")
    ws = B.alloc(B.gnn_spmm_workspace_bytes(n, col.numel(), f))
    want = run(n, rowptr, col, val, erow, X)
    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            B.gnn_spmm_csr(n, col.numel(), rowptr, col, val, erow, X, f, C, None, False, workspace=ws)
    for _ in range(3):
        C.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(C, want)


def test_weights_through_the_permutation():
    """Backward of a layer whose graph holds no weights in column order."""
    n, m = 70001, 256
    rowptr, col, val, erow, gen = matrix(5, n, 8_000_000)
    q = col.numel()
    key, perm = torch.sort(col.long() * n + erow)
    row, ecol = (key % n).int(), (key // n).int()
    colptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    colptr[1:] = torch.bincount(ecol.long(), minlength=n).cumsum(0)
    g = B.Graph(n, rowptr, col, val, erow, colptr.int(), row, perm.int(), None, ecol, symmetric=False)
    plan = B.Plan(B.GNN_LAYER_GCN, n, q, m, m, order=B.GNN_ORDER_PROPAGATE_FIRST, bwd=B.GNN_BWD_SPLIT_PROPAGATE)
    X, dY = torch.randn(n, m, generator=gen, device="cuda"), torch.randn(n, m, generator=gen, device="cuda")
    W = torch.eye(m, device="cuda")
    Y, dW, dX = torch.empty_like(X), torch.empty_like(W), torch.empty_like(X)
    cache, ws = B.alloc(plan.info.cache_bytes), B.alloc(plan.info.workspace_bytes)
    B.gcn_layer_fwd(plan, g, X, W, None, Y, cache, ws)
    B.gcn_layer_bwd(plan, g, X, W, None, dY, dW, None, dX, cache, ws)
    check(Y, n, col, val, erow, X)
    check(dX, n, row, val[perm], ecol, dY)
