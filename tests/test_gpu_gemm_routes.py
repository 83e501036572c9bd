"""Which products go to blocks that keep the parts of their columns, told from the launches that a call records, and the whole-tile
stores of these blocks with bias and ReLU.  A kept product is one launch; the other has the launch that makes the parts before it."""
import ctypes

import pytest
import torch

from paper_2308_12093_amd import binding as B

pytestmark = pytest.mark.gpu
BIG = (1 << 19) + 37


def launches(call):
    """Nodes of the graph that `call` records; nothing runs."""
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        call()
    count = ctypes.c_size_t(0)
    nodes = ctypes.CDLL("libamdhip64.so").hipGraphGetNodes
    assert nodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(count)) == 0
    return count.value


def gemm(tb, M, N, K):
    A, Bm, C = (torch.empty(s, device="cuda") for s in (M * K, N * K, M * N))
    ws = B.alloc(B.gnn_gemm_workspace_bytes(0, tb, M, N, K))
    return lambda: B.gnn_gemm(0, tb, M, N, K, A, Bm, C, None, 0, ws)


@pytest.mark.parametrize("tb,M,N,K", [
    (0, 1 << 18, 400, 4), (1, 1 << 20, 300, 4), (0, 1 << 20, 336, 20), (1, 1 << 20, 200, 32), (0, 1 << 20, 100, 32),   # shared lines
    (0, 420000, 83, 16), (1, 1 << 19, 176, 24), (1, 1 << 20, 47, 30), (0, 1 << 21, 30, 20), (0, 1 << 20, 60, 16),
    (1, 1 << 17, 128, 32), (1, 90000, 100, 32),                                               # B in rows of 32 floats
    (0, 1 << 20, 128, 32), (0, 1 << 21, 64, 20),                                              # one step, much of C
    (1, 1 << 17, 64, 48), (0, 1 << 20, 30, 48), (0, 1 << 20, 100, 48), (0, 1 << 19, 128, 64),  # two
    (0, 1 << 20, 100, 90), (0, 1 << 20, 259, 128), (0, 1 << 20, 117, 112), (1, 1 << 20, 30, 301), (0, 1 << 18, 256, 100)])
def test_step_by_step(tb, M, N, K):
    assert launches(gemm(tb, M, N, K)) == 2


@pytest.mark.parametrize("tb,M,N,K", [
    (0, 60000, 128, 16), (1, 60000, 336, 20), (0, 1 << 17, 128, 32), (1, 60000, 30, 50), (0, 60000, 64, 64), (0, 1 << 20, 96, 16),
    (0, 400000, 83, 16), (0, 1 << 19, 80, 16), (1, 1 << 20, 47, 10), (0, 1 << 22, 16, 30), (1, 1 << 21, 30, 15), (0, 1 << 18, 16, 48),
    (0, 1 << 20, 192, 48), (0, 1 << 20, 256, 100), (1, 1 << 20, 352, 190), (0, 1 << 20, 352, 96), (0, 1 << 19, 64, 400),
    (1, 1 << 20, 60, 160), (0, 1 << 20, 100, 160)])
def test_kept(tb, M, N, K):
    assert launches(gemm(tb, M, N, K)) == 1


# (BIG, 64, 80) and so on: all block shapes that keep parts, of every width
SHAPES = [(66001, 24, 20), (60001, 30, 42), (BIG, 64, 80), (BIG, 47, 250), (131100, 128, 16), (BIG, 160, 48), (BIG, 256, 100),
          (BIG, 100, 170), (70001, 130, 25)]


@pytest.mark.parametrize("M,N,K", SHAPES)
@pytest.mark.parametrize("tb", [0, 1])
def test_bias(M, N, K, tb):
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    A, Bm = torch.randn(M, K, generator=gen, device="cuda"), torch.randn(K, N, generator=gen, device="cuda")
    bias, C = torch.randn(N, generator=gen, device="cuda"), torch.full((M, N), float("nan"), device="cuda")
    ws, Bt = B.alloc(B.gnn_gemm_workspace_bytes(0, tb, M, N, K)), Bm.t().contiguous() if tb else Bm
    run = lambda: B.gnn_gemm(0, tb, M, N, K, A, Bt, C, bias, 0, ws)  # noqa: E731
    assert launches(run) == 1
    run()
    ref = A.double() @ Bm.double()
    # at most eight roundings of the sum per 16 indices, the dropped products (2^-26), the rounding of the bias
    bound = (8 * ((K + 15) // 16) + 4) * 2.0 ** -24 * (A.abs().double() @ Bm.abs().double()) + 2.0 ** -22 * (ref.abs() + bias.abs())
    assert bool(((C.double() - (ref + bias)).abs() <= bound).all())


@pytest.mark.parametrize("M,N,K", SHAPES + [(50021, 256, 100), (33000, 47, 70), (20011, 130, 65)])
@pytest.mark.parametrize("order", [B.GNN_ORDER_PROPAGATE_FIRST, B.GNN_ORDER_TRANSFORM_FIRST])
def test_bias_and_relu(M, N, K, order):
    """A layer without input gradient over the identity, Y = relu(X W + b): kept parts, and from 1024 tiles on the others."""
    gen = torch.Generator(device="cuda").manual_seed(M + N)
    ids = torch.arange(M + 1, dtype=torch.int32, device="cuda")
    g = B.Graph(M, ids, ids[:M].clone(), torch.ones(M, device="cuda"), ids[:M].clone(), symmetric=True)
    plan = B.Plan(B.GNN_LAYER_GCN, M, M, K, N, need_input_grad=False, has_bias=True, fuse_relu=True, order=order)
    X, W, b = (torch.randn(*s, generator=gen, device="cuda") for s in ((M, K), (K, N), (N,)))
    Y = torch.full((M, N), float("nan"), device="cuda")
    B.gcn_layer_fwd(plan, g, X, W, b, Y, B.alloc(plan.info.cache_bytes), B.alloc(plan.info.workspace_bytes))
    ref = X.double() @ W.double()
    bound = (8 * ((K + 15) // 16) + 4) * 2.0 ** -24 * (X.abs().double() @ W.abs().double()) + 2.0 ** -22 * (ref.abs() + b.abs())
    assert bool(((Y.double() - torch.relu(ref + b)).abs() <= bound).all())
