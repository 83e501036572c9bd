"""Products before a fused ReLU on both sides of the line at 2^17 outputs, with and without dX, against float64."""
import pytest
import torch

from paper_2308_12093_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dx", [False, True])
@pytest.mark.parametrize("n,m,k", [(33, 64, 5), (3001, 203, 7), (8192, 70, 16), (8193, 70, 16), (2048, 95, 64), (2049, 96, 64)])
def test_forward(n, m, k, dx):
    """A' is the identity, so that Y = relu(X W + b)."""
    gen = torch.Generator(device="cuda").manual_seed(n + m + k)
    ids = torch.arange(n + 1, dtype=torch.int32, device="cuda")
    g = B.Graph(n, ids, ids[:n].clone(), torch.ones(n, device="cuda"), ids[:n].clone(), symmetric=True)
    for order in (B.GNN_ORDER_PROPAGATE_FIRST, B.GNN_ORDER_TRANSFORM_FIRST):
        plan = B.Plan(B.GNN_LAYER_GCN, n, n, m, k, need_input_grad=dx, has_bias=True, fuse_relu=True, order=order)
        X, W, b = (torch.randn(*s, generator=gen, device="cuda") for s in ((n, m), (m, k), (k,)))
        Y = torch.empty(n, k, device="cuda")
        B.gcn_layer_fwd(plan, g, X, W, b, Y, B.alloc(plan.info.cache_bytes), B.alloc(plan.info.workspace_bytes))
        ref = torch.relu(X.double() @ W.double() + b.double())
        # one rounding per pair of indices at the most, three for the four sums, one each for the bias and the result
        bound = (m // 2 + 6) * 2.0 ** -24 * (X.abs().double() @ W.abs().double() + b.abs())
        assert bool(((Y.double() - ref).abs() <= bound).all())
