"""SpMM of graphs large enough for long rows to be cut into pieces: row lengths at the edges of pieces and classes, columns
in any order, ragged and wide operands, values that are not finite, and the products that stay with the segments."""
import pytest
import torch

from paper_2308_12093_amd import binding as B

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 2, 8, 9, 16, 17, 33, 64, 65, 127, 128, 129, 143, 144, 191, 192, 193, 255, 256, 1000, 4097, 65535, 65600, 200000]


def matrix(seed, n, nnz, hubs=True, ordered=True, more=(), by_length=False):
    """CSR on the device: the lengths of EDGES first and last, `more` behind the first ones, the others alike but a few
    thousand long ones; by_length: rows in descending order of their length."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    d = torch.full((n,), 3, dtype=torch.int64, device="cuda")
    if hubs:
        d[torch.randperm(n, generator=gen, device="cuda")[:4000]] = max(128, (nnz - 3 * n - 2 * sum(EDGES)) // 4000)
        edges = torch.tensor(EDGES, device="cuda")
        d[:len(EDGES)], d[n - len(EDGES):] = edges, edges.flip(0)
        d[len(EDGES):len(EDGES) + len(more)] = torch.tensor(more, dtype=torch.int64, device="cuda")
        if by_length:
            d = d.sort(descending=True).values
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
        rows = erow[lo:lo + piece].long()
        t = X[col[lo:lo + piece].long()] * val[lo:lo + piece, None].double()
        # runs of one row, of 512 entries at most: millions of entries added to one row at once wait for each other for hours
        first = torch.arange(rows.numel(), device="cuda") % 512 == 0
        first[1:] |= rows[1:] != rows[:-1]
        first = first.nonzero().squeeze(1)
        lengths = torch.diff(first, append=first.new_tensor([rows.numel()]))
        ref.index_add_(0, rows[first], torch.segment_reduce(t, "sum", lengths=lengths, axis=0))
        mag.index_add_(0, rows[first], torch.segment_reduce(t.abs_(), "sum", lengths=lengths, axis=0))
    if bias is not None:
        ref += bias.double()
        mag += bias.double().abs()
    if relu:
        ref.clamp_(min=0)
    most = roundings(torch.bincount(erow, minlength=n), X.shape[1])
    assert bool(((C.double() - ref).abs() <= most[:, None] * 2.0 ** -24 * 1.001 * mag).all())


def roundings(d, f):
    """Roundings on the way of a product into a row of d entries.  A row below 128 entries: one for each and six for the
    bias and for where segments meet.  A longer one: at most 111 in a piece; then 512 partials at a time, in four rotating
    sums of each slot (three more for the rest), two to join those and a tree over the slots; the same over the shares of
    512; the bias."""
    lanes = 4
    while lanes < 64 and 4 * lanes < f:
        lanes *= 2
    slots = 64 // lanes
    level = lambda n: (n / (4 * slots)).ceil() + 5 + slots.bit_length() - 1  # noqa: E731
    pieces = (d.double() / 64).floor()
    shares = (pieces / 512).ceil()
    return torch.where(d < 128, d + 6.0, 111 + level(pieces.clamp(max=512)) + torch.where(pieces > 512, level(shares), 0.0) + 1)


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


@pytest.mark.parametrize("f,more", [(64, [5_000_000, 300_000, 32_767, 32_768, 32_784, 32_832, 65_600]), (47, [16_000_000]),
                                    (260, [2_100_000, 32_831, 98_368])])
@pytest.mark.parametrize("by_length", [False, True])
def test_a_row_with_much_of_the_graph(f, more, by_length):
    """Equal products: every addition of a long chain rounds the same way, so that its length shows in the result."""
    n = 70001
    rowptr, col, val, erow, gen = matrix(f, n, 28_000_000, ordered=False, more=more, by_length=by_length)
    val.fill_(1.0)
    X = torch.rand(f, generator=gen, device="cuda").expand(n, f).contiguous()
    C = run(n, rowptr, col, val, erow, X)
    check(C, n, col, val, erow, X)
    assert torch.equal(C, run(n, rowptr, col, val, erow, X))


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


def test_sums_that_underflow_keep_the_sign_of_zero():
    n, d, f = 110_000, 300, 64
    rowptr = torch.arange(0, n * d + 1, d, dtype=torch.int32, device="cuda")
    erow = torch.arange(n, dtype=torch.int32, device="cuda").repeat_interleave(d)
    col = torch.randint(0, n, (n * d,), dtype=torch.int32, device="cuda")
    X = torch.full((n, f), 1e-30, device="cuda")
    X[:, ::2] = -1e-30
    C = run(n, rowptr, col, torch.full((n * d,), 1e-30, device="cuda"), erow, X)
    assert bool((C == 0).all()) and bool(torch.signbit(C[:, ::2]).all()) and not bool(torch.signbit(C[:, 1::2]).any())


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
