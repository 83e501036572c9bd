"""Small products with long rows side by side: sums against float64 on both sides of the lines between the kernels, and the
time of a call, which hangs neither on a ragged width nor on where the long rows are.  Times of a graph of twenty calls, the least
of several replays, against another call of the same size: the bounds leave a factor of about two."""
import pytest
import torch

from paper_2308_12093_amd import binding as B

pytestmark = pytest.mark.gpu


def hub_graph(n, hubs):
    """`hubs` nodes, numbered first, joined to every node, and a loop at each."""
    a, h = torch.arange(n, device="cuda"), torch.arange(hubs, device="cuda")
    key = torch.unique(torch.cat([a * n + a, h.repeat_interleave(n) * n + a.repeat(hubs), a.repeat(hubs) * n + h.repeat_interleave(n)]))
    return csr(n, key)


def csr(n, key):
    row, col = torch.div(key, n, rounding_mode="floor"), key % n
    rowptr = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    rowptr[1:] = torch.bincount(row, minlength=n).cumsum(0).int()
    return rowptr, col.int(), row.int()


def uniform_graph(n, q, seed=1):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return csr(n, torch.randint(0, n * n, (q,), generator=gen, device="cuda").sort().values)


def operands(n, f, q, seed=1):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(q, generator=gen, device="cuda"), torch.randn(n, f, generator=gen, device="cuda")


def call(n, f, graph):
    rowptr, col, erow = graph
    q = col.numel()
    val, X = operands(n, f, q)
    C, ws = torch.empty(n, f, device="cuda"), B.alloc(B.gnn_spmm_workspace_bytes(n, q, f))
    return lambda: B.gnn_spmm_csr(n, q, rowptr, col, val, erow, X, f, C, workspace=ws)


def without_expanded_rows(n, f, graph):
    rowptr, col, _ = graph
    val, X = operands(n, f, col.numel())
    C = torch.empty(n, f, device="cuda")
    return lambda: B.gnn_spmm_csr(n, col.numel(), rowptr, col, val, None, X, f, C)


def check(n, f, graph, expanded=True):
    rowptr, col, erow = graph
    q = col.numel()
    val, X = operands(n, f, q)
    C, ws = torch.full((n, f), float("nan"), device="cuda"), B.alloc(B.gnn_spmm_workspace_bytes(n, q, f))
    B.gnn_spmm_csr(n, q, rowptr, col, val, erow if expanded else None, X, f, C, workspace=ws)
    A = torch.zeros(n, n, dtype=torch.float64, device="cuda").index_put_((erow.long(), col.long()), val.double(), accumulate=True)
    size = torch.zeros_like(A).index_put_((erow.long(), col.long()), val.double().abs(), accumulate=True) @ X.double().abs()
    length = (rowptr[1:] - rowptr[:-1]).double()[:, None]
    # a rounding per entry at the most, and a few for the sums of the slots
    assert bool(((C.double() - A @ X.double()).abs() <= (length + 16) * 2.0 ** -24 * size).all())


def least_us(run, calls=20, replays=8):
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        run()
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for _ in range(calls):
            run()
    least = float("inf")
    for _ in range(replays):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        graph.replay()
        b.record()
        b.synchronize()
        least = min(least, a.elapsed_time(b) * 1e3 / calls)
    return least


@pytest.mark.parametrize("n,f,aligned", [(1024, 23, 32), (512, 17, 32), (512, 47, 64)])
def test_ragged_width(n, f, aligned):
    """Takes about what the next aligned width takes (1024 x 23: 2.3 times that with one feature a lane)."""
    graph = hub_graph(n, 8)
    assert least_us(call(n, f, graph)) <= 1.6 * least_us(call(n, aligned, graph))


@pytest.mark.parametrize("n,f", [(1024, 16), (4096, 32), (2048, 23), (8192, 16)])
def test_hubs_side_by_side(n, f):
    """Eight rows of n entries take about what as many entries take in rows of one length (one block for the eight: 6 to 30 times)."""
    graph = hub_graph(n, 8)
    assert least_us(call(n, f, graph)) <= 4 * least_us(call(n, f, uniform_graph(n, graph[1].numel())))


@pytest.mark.parametrize("n,f", [(1500, 128), (4096, 23), (8192, 16), (1500, 64)])
def test_no_long_rows(n, f):
    """Small products without long rows are not held back by those with them: what calls without expanded rows take, which always go by
    rows (in segments 1.6 to 4 times that)."""
    graph = uniform_graph(n, 9 * n)
    assert least_us(call(n, f, graph)) <= 1.35 * least_us(without_expanded_rows(n, f, graph))


@pytest.mark.parametrize("n,f", [(4096, 31), (4097, 31), (10240, 16), (10241, 16), (2048, 64), (2049, 64), (1536, 100), (4096, 127), (2048, 112),
                                 (2048, 32), (2049, 32), (2047, 17), (4096, 16), (4097, 13), (8191, 8), (8192, 5), (8193, 8), (512, 64),
                                 (513, 64), (511, 33), (512, 65), (16, 64), (9, 3), (8193, 3)])
@pytest.mark.parametrize("expanded", [True, False])
def test_hubs_against_float64(n, f, expanded):
    check(n, f, hub_graph(n, 8), expanded)


@pytest.mark.parametrize("n,f,q", [(512, 16, 98304), (512, 16, 98305), (512, 64, 24576), (512, 64, 24577), (469, 28, 70182), (469, 99, 52000),
                                   (512, 32, 163840), (512, 32, 163841), (2048, 8, 700000), (2048, 8, 700001)])
def test_entries_against_float64(n, f, q):
    check(n, f, uniform_graph(n, q))


@pytest.mark.parametrize("f", [256 * 65535, 256 * 65535 + 5])
def test_more_feature_tiles_than_a_grid_has(f):
    rowptr, col = (torch.tensor(x, dtype=torch.int32, device="cuda") for x in ([0, 2, 3], [0, 1, 1]))
    val, X = torch.tensor([1.5, -2.0, 0.5], device="cuda"), torch.randn(2, f, device="cuda")
    C = torch.full((2, f), float("nan"), device="cuda")
    B.gnn_spmm_csr(2, 3, rowptr, col, val, None, X, f, C)
    assert torch.equal(C[1], 0.5 * X[1])
    assert bool(((C[0] - (1.5 * X[0] - 2.0 * X[1])).abs() <= 2.0 ** -22 * (1.5 * X[0].abs() + 2.0 * X[1].abs())).all())


@pytest.mark.parametrize("f", [3, 16, 23, 60, 100])
@pytest.mark.parametrize("lengths", [[2000] + [150] * 7, [150] * 6 + [3000, 3000], [129, 128, 127, 1025, 1024, 1023, 0, 5], [700] * 8, [0] * 7 + [4000]])
def test_long_and_short_rows_of_a_block(f, lengths):
    """Seven rows that are not long between a block's eight, so that it has these."""
    n = 8 * 64
    rows = torch.zeros(n, dtype=torch.long)
    rows[::64] = torch.tensor(lengths)
    rows[5::64] = 3
    gen = torch.Generator(device="cuda").manual_seed(f)
    row = torch.repeat_interleave(torch.arange(n), rows).cuda()
    check(n, f, csr(n, (row * n + torch.randint(0, n, row.shape, generator=gen, device="cuda")).sort().values))
