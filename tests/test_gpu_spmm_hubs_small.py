"""Small products with long rows side by side: the time of a call does not hang on a ragged width.  Times of a graph of twenty
calls, the least of several replays, against another call of the same kernel: the bounds leave a factor of about two."""
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


def call(n, f, graph, seed=1):
    rowptr, col, erow = graph
    q = col.numel()
    gen = torch.Generator(device="cuda").manual_seed(seed)
    val, X = torch.randn(q, generator=gen, device="cuda"), torch.randn(n, f, generator=gen, device="cuda")
    C, ws = torch.empty(n, f, device="cuda"), B.alloc(B.gnn_spmm_workspace_bytes(n, q, f))
    return lambda: B.gnn_spmm_csr(n, q, rowptr, col, val, erow, X, f, C, workspace=ws)


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
