"""Backward from cached edge weights, which the row pass leaves signed for the column pass where they are larger than an L2 (4 bytes
and the mask's one per entry and head): against the variant that rebuilds them and, on both sides of that line, entry by entry against
float64 from the cache's own arrays.  Heads of one lane, of two and more, several feature tiles, lists that end inside a batch."""
import numpy as np
import pytest
import torch

import oracle
from paper_2308_12093_amd import binding as B, graphs
from tests._util import assert_close, host

pytestmark = pytest.mark.gpu
LINE = 4 << 20


def pattern(n, extra, h, k):
    gen = np.random.Generator(np.random.PCG64(n + h + k))
    key = np.unique(gen.integers(0, n, n * extra) * n + gen.integers(0, n, n * extra) // 3)
    row, col = key // n, key % n
    return np.concatenate([[0], np.cumsum(np.bincount(row, minlength=n))]).astype(np.int32), col.astype(np.int32)


def tensors(n, m, h, k):
    tg = torch.Generator(device="cuda").manual_seed(n)
    X, W, dY = (torch.randn(*s, generator=tg, device="cuda") for s in ((n, m), (m, h * k), (n, h * k)))
    return X, W * 0.2, dY, [torch.randn(h, k, generator=tg, device="cuda") * 0.3 for _ in range(2)]


@pytest.mark.parametrize("n,extra,h,k", [(9000, 25, 8, 4), (9001, 11, 8, 4), (9000, 12, 8, 16), (5003, 20, 10, 32), (60001, 15, 1, 8), (3001, 80, 4, 64)])
def test_variants_agree(n, extra, h, k):
    g = graphs.gat_graph(*pattern(n, extra, h, k), "cuda:0")
    assert g.nnz * h * 5 > LINE
    m, f = 24, h * k
    X, W, dY, a = tensors(n, m, h, k)
    results = []
    for cache in (B.GNN_CACHE_GAT_FEAT_EDGE, B.GNN_CACHE_GAT_FEAT_NODEATT):
        plan = B.Plan(B.GNN_LAYER_GAT, g.n, g.nnz, m, k, heads=h, cache=cache)
        ws, held = B.alloc(plan.info.workspace_bytes), B.alloc(plan.info.cache_bytes)
        Y, dW, dX = torch.empty(n, f, device="cuda"), torch.empty(m, f, device="cuda"), torch.empty(n, m, device="cuda")
        da = [torch.empty(h, k, device="cuda") for _ in range(2)]
        B.gat_layer_fwd(plan, g, X, W, *a, None, Y, held, ws)
        for _ in range(2):                                  # the cache serves a second call
            B.gat_layer_bwd(plan, g, X, W, *a, dY, dW, *da, None, dX, held, ws)
        results.append([Y, dW, dX, *da])
    for x, y in zip(*results):
        # both take the LeakyReLU signs from the same floats; float sums of a few hundred terms, da from sums that cancel
        assert float((x.double() - y.double()).norm() / y.double().norm()) < 2e-5


@pytest.mark.parametrize("n,extra,h,k,signed", [(9001, 10, 8, 4, False), (9001, 11, 8, 4, True), (5003, 14, 10, 32, False),
                                                (5003, 16, 10, 32, True), (60001, 12, 1, 8, False), (60001, 13, 1, 8, True),
                                                (6000, 16, 8, 8, False), (6000, 18, 8, 8, True), (3001, 80, 4, 64, True)])
def test_against_float64(n, extra, h, k, signed):
    rowptr, col = pattern(n, extra, h, k)
    g = graphs.gat_graph(rowptr, col, "cuda:0")
    assert (g.nnz * h * 5 > LINE) == signed
    m, f, q = 24, h * k, g.nnz
    X, W, dY, a = tensors(n, m, h, k)
    plan = B.Plan(B.GNN_LAYER_GAT, n, q, m, k, heads=h, cache=B.GNN_CACHE_GAT_FEAT_EDGE)
    ws, held = B.alloc(plan.info.workspace_bytes), B.alloc(plan.info.cache_bytes)
    Y, dW, dX = torch.empty(n, f, device="cuda"), torch.empty(m, f, device="cuda"), torch.empty(n, m, device="cuda")
    da = [torch.empty(h, k, device="cuda") for _ in range(2)]
    B.gat_layer_fwd(plan, g, X, W, *a, None, Y, held, ws)
    # the cache holds M, alpha and mask, each from a multiple of 256 bytes on
    at_alpha = (4 * n * f + 255) // 256 * 256
    at_mask = at_alpha + (4 * q * h + 255) // 256 * 256
    M, alpha = held[:4 * n * f].view(torch.float32), held[at_alpha:at_alpha + 4 * q * h].view(torch.float32)
    mask = held[at_mask:at_mask + q * h]
    rp, c, _ = oracle.add_self_loops_degree(rowptr, col)
    ref = oracle.gat_backward_from(rp, c, host(X), host(W), host(a[0]), host(a[1]), host(dY), host(M).reshape(n, h, k),
                                   host(alpha).reshape(q, h), host(mask).reshape(q, h), plan.desc.leaky_slope)
    for _ in range(2):
        for t in (dW, dX, *da):
            t.fill_(float("nan"))
        ws.fill_(0xFF)                                      # nothing of an earlier call may be read
        B.gat_layer_bwd(plan, g, X, W, *a, dY, dW, *da, None, dX, held, ws)
        for name, got in (("dW", dW), ("dX", dX), ("da_src", da[0]), ("da_dst", da[1])):
            assert_close(host(got), ref[name].reshape(got.shape), name)
