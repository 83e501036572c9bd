"""Layers with bias and ReLU in the split-propagate scheme: the forward product on both sides of the node count from which it
runs on split parts (without dX), and backward: bias gradient and mask formed beside X^T G, the mask
taken by the products with the weights.  A' is the identity, so that every gradient is a dense product."""
import pytest
import torch

from paper_2308_12093_amd import binding as B

pytestmark = pytest.mark.gpu


def normal(gen, *shape):
    return torch.randn(*shape, generator=gen, device="cuda")


def close(got, want, most):
    assert bool(((got.double() - want).abs() <= most).all())


# ragged and whole tiles of one, two and four times 32 columns, reductions that end inside a step, outputs beyond 64 MB
@pytest.mark.parametrize("sage", [False, True])
@pytest.mark.parametrize("order", [B.GNN_ORDER_PROPAGATE_FIRST, B.GNN_ORDER_TRANSFORM_FIRST])
@pytest.mark.parametrize("n", [65535, 65536, 70001])
@pytest.mark.parametrize("m,k", [(64, 64), (16, 5), (100, 33), (130, 47), (70, 200), (128, 512), (33, 96), (4, 17), (40, 259)])
def test_forward(n, m, k, order, sage):
    gen = torch.Generator(device="cuda").manual_seed(n + m + k)
    ids = torch.arange(n + 1, dtype=torch.int32, device="cuda")
    g = B.Graph(n, ids, ids[:n].clone(), torch.ones(n, device="cuda"), ids[:n].clone(), symmetric=True)
    plan = B.Plan(B.GNN_LAYER_SAGE if sage else B.GNN_LAYER_GCN, n, n, m, k, need_input_grad=False, has_bias=True,
                  fuse_relu=True, order=order)
    X, Ws, Wn, b = normal(gen, n, m), normal(gen, m, k) * 0.1, normal(gen, m, k) * 0.1, normal(gen, k)
    X[::7] *= 2.0 ** -100                                   # rows that are taken times a power of two
    Y, cache, ws = torch.empty(n, k, device="cuda"), B.alloc(plan.info.cache_bytes), B.alloc(plan.info.workspace_bytes)
    if sage:
        B.sage_layer_fwd(plan, g, X, Ws, Wn, b, Y, cache, ws)
    else:
        B.gcn_layer_fwd(plan, g, X, Wn, b, Y, cache, ws)
    W, Wabs = (Ws.double() + Wn.double(), Ws.abs().double() + Wn.abs().double()) if sage else (Wn.double(), Wn.abs().double())
    ref, mag = X.double() @ W + b.double(), X.abs().double() @ Wabs + b.abs().double()
    # sums in float: at most eight roundings per 16 indices of each operand pair, then those of the aggregation, the
    # accumulated product and the bias
    close(Y, ref.clamp(min=0), (8 * ((m + 15) // 16) * (2 if sage else 1) + 8) * 2.0 ** -24 * mag)
    assert bool((Y >= 0).all())


# widths at the edges of tiles and of 16-column words; 2100 columns, few rows and long input features take the mask no
# product's way
@pytest.mark.parametrize("sage", [False, True])
@pytest.mark.parametrize("relu,dx", [(True, True), (True, False), (False, True)])
@pytest.mark.parametrize("n,m,k", [(40007, 64, 64), (33000, 100, 33), (40000, 130, 47), (36000, 70, 200), (65536, 128, 512),
                                   (35001, 96, 80), (34000, 300, 17), (3000, 40, 50), (40000, 40, 2100), (70001, 16, 5),
                                   (33000, 64, 1000), (33000, 40, 2048), (33001, 130, 519),
                                   (33000, 515, 300), (35000, 200, 130)])
def test_gradients(n, m, k, relu, dx, sage):
    gen = torch.Generator(device="cuda").manual_seed(n + m + k)
    ids = torch.arange(n + 1, dtype=torch.int32, device="cuda")
    g = B.Graph(n, ids, ids[:n].clone(), torch.ones(n, device="cuda"), ids[:n].clone(), symmetric=True)
    plan = B.Plan(B.GNN_LAYER_SAGE if sage else B.GNN_LAYER_GCN, n, n, m, k, need_input_grad=dx, has_bias=True, fuse_relu=relu,
                  order=B.GNN_ORDER_PROPAGATE_FIRST, bwd=B.GNN_BWD_SPLIT_PROPAGATE)
    X, Ws, Wn, b, dY = normal(gen, n, m), normal(gen, m, k) * 0.1, normal(gen, m, k) * 0.1, normal(gen, k), normal(gen, n, k)
    dY[normal(gen, n, k) > 1.5] = 0.0
    Y, dWs, dWn = torch.empty(n, k, device="cuda"), torch.empty(m, k, device="cuda"), torch.empty(m, k, device="cuda")
    db, dX = torch.empty(k, device="cuda"), torch.empty(n, m, device="cuda") if dx else None
    cache, ws = B.alloc(plan.info.cache_bytes), B.alloc(plan.info.workspace_bytes)
    for _ in range(2):                                      # the second over what the first left
        if sage:
            B.sage_layer_fwd(plan, g, X, Ws, Wn, b, Y, cache, ws)
            B.sage_layer_bwd(plan, g, X, Ws, Wn, Y, dY, dWs, dWn, db, dX, cache, ws)
        else:
            B.gcn_layer_fwd(plan, g, X, Wn, b, Y, cache, ws)
            B.gcn_layer_bwd(plan, g, X, Wn, Y, dY, dWn, db, dX, cache, ws)
    G = dY.double() * (Y > 0) if relu else dY.double()
    # sums in double, and the rounding to float
    double = lambda ref, mag, terms: 2.0 ** -24 * ref.abs() + 2 * terms * 2.0 ** -53 * mag  # noqa: E731
    Xd = X.double()
    ref, mag = Xd.t() @ G, Xd.abs().t() @ G.abs()
    for d in (dWs, dWn) if sage else (dWn,):
        close(d, ref, double(ref, mag, n))
    close(db, G.sum(0), double(G.sum(0), G.abs().sum(0), n))
    if dx:
        # sums in float: at most eight roundings per 16 indices, and those of the two products and the aggregation
        W, Wabs = (Ws.double() + Wn.double(), Ws.abs().double() + Wn.abs().double()) if sage else (Wn.double(), Wn.abs().double())
        close(dX, G @ W.t(), (8 * ((k + 15) // 16) + 8) * 2.0 ** -24 * (G.abs() @ Wabs.t()))


@pytest.mark.parametrize("sage", [False, True])
@pytest.mark.parametrize("offset", [0, 128])
@pytest.mark.parametrize("n,m", [(40007, 64), (33000, 100), (3000, 40)])
def test_input_gradient_over_the_output_gradient(n, m, offset, sage):
    """dX in the memory of dY, the same rows or some floats before them."""
    gen = torch.Generator(device="cuda").manual_seed(n + m)
    ids = torch.arange(n + 1, dtype=torch.int32, device="cuda")
    g = B.Graph(n, ids, ids[:n].clone(), torch.ones(n, device="cuda"), ids[:n].clone(), symmetric=True)
    plan = B.Plan(B.GNN_LAYER_SAGE if sage else B.GNN_LAYER_GCN, n, n, m, m, has_bias=True, fuse_relu=True,
                  order=B.GNN_ORDER_PROPAGATE_FIRST, bwd=B.GNN_BWD_SPLIT_PROPAGATE)
    X, Ws, Wn, b = normal(gen, n, m), normal(gen, m, m) * 0.1, normal(gen, m, m) * 0.1, normal(gen, m)
    memory = normal(gen, n * m + offset)
    dY, dX = memory[offset:].view(n, m), memory[:n * m].view(n, m)
    G = dY.double()
    Y, cache, ws = torch.empty(n, m, device="cuda"), B.alloc(plan.info.cache_bytes), B.alloc(plan.info.workspace_bytes)
    dWs, dWn, db = torch.empty(m, m, device="cuda"), torch.empty(m, m, device="cuda"), torch.empty(m, device="cuda")
    if sage:
        B.sage_layer_fwd(plan, g, X, Ws, Wn, b, Y, cache, ws)
        B.sage_layer_bwd(plan, g, X, Ws, Wn, Y, dY, dWs, dWn, db, dX, cache, ws)
    else:
        B.gcn_layer_fwd(plan, g, X, Wn, b, Y, cache, ws)
        B.gcn_layer_bwd(plan, g, X, Wn, Y, dY, dWn, db, dX, cache, ws)
    G *= Y > 0
    # bounds as above
    double = lambda ref, mag: 2.0 ** -24 * ref.abs() + 2 * n * 2.0 ** -53 * mag  # noqa: E731
    Xd = X.double()
    ref, mag = Xd.t() @ G, Xd.abs().t() @ G.abs()
    for d in (dWs, dWn) if sage else (dWn,):
        close(d, ref, double(ref, mag))
    close(db, G.sum(0), double(G.sum(0), G.abs().sum(0)))
    W, Wabs = (Ws.double() + Wn.double(), Ws.abs().double() + Wn.abs().double()) if sage else (Wn.double(), Wn.abs().double())
    close(dX, G @ W.t(), (8 * ((m + 15) // 16) + 8) * 2.0 ** -24 * (G.abs() @ Wabs.t()))
