"""Backward from cached edge weights where the row pass leaves them signed for the column pass, against the variant that rebuilds
them: heads of one lane, of two and more, several feature tiles, lists that end inside a batch, both sides of the line."""
import numpy as np
import pytest
import torch

from paper_2308_12093_amd import binding as B, graphs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,extra,h,k", [(9000, 25, 8, 4), (9001, 11, 8, 4), (9000, 12, 8, 16), (5003, 20, 10, 32), (60001, 15, 1, 8), (3001, 80, 4, 64)])
def test_variants_agree(n, extra, h, k):
    gen = np.random.Generator(np.random.PCG64(n + h + k))
    key = np.unique(gen.integers(0, n, n * extra) * n + gen.integers(0, n, n * extra) // 3)
    row, col = key // n, key % n
    rowptr = np.concatenate([[0], np.cumsum(np.bincount(row, minlength=n))]).astype(np.int32)
    g = graphs.gat_graph(rowptr, col.astype(np.int32), "cuda:0")
    m, f = 24, h * k
    tg = torch.Generator(device="cuda").manual_seed(n)
    X, W, dY = (torch.randn(*s, generator=tg, device="cuda") for s in ((n, m), (m, f), (n, f)))
    W *= 0.2
    a = [torch.randn(h, k, generator=tg, device="cuda") * 0.3 for _ in range(2)]
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
