"""The workloads this library is timed on, each as a user's program runs it through the public entry points.

A case is a dict of plain values.  ``kind`` names what one pass does:

  gcn      one GCN layer: forward, and (``step``) backward, as in training; without ``step`` the pass is inference
  gcn2     a two-layer GCN with ReLU between the layers and softmax cross-entropy: forward, loss, backward
  gat      one multi-head GAT layer, forward and (``step``) backward
  gat2     a two-layer GAT with ELU between the layers and squared error: forward, loss, backward
  sage     one GraphSAGE layer with mean aggregation (a directed operator: backward reads the CSC arrays)
  spmm     the sparse-dense product on its own
  setup    what a program does once for every new graph: self-loops, degrees, weights, transpose, expanded indices

Graphs are R-MAT (the hub-heavy case of citation and social graphs) or uniform random, made on the GPU from the seed;
``degree`` is the mean number of stored neighbours per node, self-loops not counted.  Dense inputs are N(0, 1),
weights Glorot-uniform.  The sizes follow the five configurations and the tests of this repository.
"""
import math

import torch

from paper_2308_12093_amd import binding as B
from paper_2308_12093_amd import graphs

RMAT = (0.57, 0.19, 0.19)            # the fourth quadrant has the rest


def listed():
    return [
        # a citation graph of a few thousand nodes with long input features: every kernel is short, launches count
        dict(name="gcn_small_step", kind="gcn", graph="uniform", n=2048, degree=8, f_in=512, f_out=16, step=True,
             bias=False, relu=False),
        # inference on a small graph with sizes that are multiples of nothing
        dict(name="gcn_small_forward", kind="gcn", graph="uniform", n=3001, degree=9, f_in=203, f_out=7, step=False,
             bias=True, relu=True),
        # a mid-sized graph, narrow output: the product first, then a narrow aggregation
        dict(name="gcn_narrow_step", kind="gcn", graph="rmat", n=1 << 17, degree=14, f_in=128, f_out=16, step=True,
             bias=False, relu=False),
        # the same graph with a wide hidden layer, bias and ReLU: the dense products weigh as much as the aggregation
        dict(name="gcn_wide_step", kind="gcn", graph="rmat", n=1 << 17, degree=14, f_in=128, f_out=512, step=True,
             bias=True, relu=True),
        # full-batch training of a two-layer network on a million nodes with 47 classes
        dict(name="gcn_network_step", kind="gcn2", graph="rmat", n=1 << 20, degree=50, f_in=100, hidden=256, f_out=47),
        # the largest graph of the benchmark: aggregation over 132 million entries
        dict(name="gcn_large_step", kind="gcn", graph="rmat", n=1 << 22, degree=32, f_in=64, f_out=256, step=True,
             bias=False, relu=False),
        # attention layer with eight narrow heads and the default caching variant
        dict(name="gat_step", kind="gat", graph="rmat", n=1 << 17, degree=14, f_in=256, heads=8, f_out=8, step=True,
             bias=False, elu=False, calibrated=False),
        # two attention layers, 256 features each, the caching variant that is fastest here
        dict(name="gat_network_step", kind="gat2", graph="rmat", n=1 << 17, degree=14, f_in=256, heads=8, f_out=32,
             calibrated=True),
        # attention inference on a graph with an odd node count
        dict(name="gat_forward", kind="gat", graph="rmat", n=50021, degree=11, f_in=96, heads=4, f_out=16, step=False,
             bias=True, elu=True, calibrated=True),
        # GraphSAGE with mean aggregation: two weights, a transpose that is not the matrix itself
        dict(name="sage_step", kind="sage", graph="rmat", n=1 << 17, degree=14, f_in=128, f_out=128, step=True,
             bias=True, relu=True),
        # the operator on its own with a class count that is no multiple of four
        dict(name="spmm_ragged", kind="spmm", graph="rmat", n=1 << 17, degree=14, f_in=47),
        # preparing a directed graph of a million nodes
        dict(name="graph_setup", kind="setup", graph="rmat", n=1 << 20, degree=16),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi):
    """A feature width: half of them multiples of 16, the others any number."""
    w = _log_int(rng, lo, hi)
    return max(16, w // 16 * 16) if rng.random() < 0.5 else w


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        kind = rng.choice(["gcn", "gcn", "gcn", "gcn2", "gat", "gat", "gat2", "sage", "spmm", "setup"])
        c = dict(kind=kind, graph="uniform" if rng.random() < 0.3 else "rmat", n=_log_int(rng, 2000, 1 << 22),
                 degree=rng.randint(4, 50))
        if kind in ("gcn", "sage"):
            c.update(f_in=_width(rng, 16, 512), f_out=_width(rng, 7, 512), step=rng.random() < 0.75,
                     bias=rng.random() < 0.5, relu=rng.random() < 0.5)
        elif kind == "gcn2":
            c.update(f_in=_width(rng, 16, 512), hidden=_width(rng, 16, 256), f_out=rng.randint(3, 64))
        elif kind in ("gat", "gat2"):
            c.update(f_in=_width(rng, 16, 256), heads=rng.choice([1, 2, 4, 8]), f_out=rng.choice([8, 8, 16, 32, 64, 12]),
                     calibrated=rng.random() < 0.5)
            if kind == "gat":
                c.update(step=rng.random() < 0.75, bias=rng.random() < 0.5, elu=rng.random() < 0.5)
        elif kind == "spmm":
            c.update(f_in=_width(rng, 7, 512))
        # not more than the largest listed case, and at most 150 million entries
        if _cost(c) <= most and c["n"] * (c["degree"] + 1) <= 150_000_000 and _largest_tensor(c) <= 5 << 30:
            return c


# ---- sizes ---------------------------------------------------------------------------------------
def _entries(c):
    return c["n"] * (c["degree"] + 1)


def _layers(c):
    """(f_in, f_out, backward, input gradient) of every layer of one pass; f_out over all heads."""
    k = c["kind"]
    if k in ("gcn", "sage"):
        return [(c["f_in"], c["f_out"], c["step"], c["step"])]
    if k == "gcn2":
        return [(c["f_in"], c["hidden"], True, False), (c["hidden"], c["f_out"], True, True)]
    if k == "gat":
        return [(c["f_in"], c["heads"] * c["f_out"], c["step"], c["step"])]
    if k == "gat2":
        f = c["heads"] * c["f_out"]
        return [(c["f_in"], f, True, False), (f, f, True, True)]
    return []


def work(case):
    """Each input read once and each output written once; the flops of the products in the cheaper order."""
    n, q = case["n"], _entries(case)
    if case["kind"] == "setup":      # raw CSR in; CSR, CSC, perm, both expanded indices and the weights in both orders out
        return {"bytes": 4.0 * (2 * n + q) + 4.0 * (3 * n + 7 * q), "flops": 0.0}
    if case["kind"] == "spmm":
        f = case["f_in"]
        return {"bytes": 4.0 * (n + 2 * q + 2 * n * f), "flops": 2.0 * q * f}
    gat = case["kind"] in ("gat", "gat2")
    byts, flops = 4.0 * (n + (1 if gat else 2) * q), 0.0
    for i, (m, k, bwd, dx) in enumerate(_layers(case)):
        w = k if gat else min(m, k)
        pairs = 2 if case["kind"] == "sage" else 1
        if i == 0:
            byts += 4.0 * n * m
        byts += 4.0 * (n * k + pairs * m * k)
        flops += 2.0 * pairs * n * m * k + 2.0 * q * w
        if bwd:
            byts += 4.0 * (n * k + pairs * m * k + (n * m if dx else 0))
            flops += 2.0 * pairs * n * m * k * (2 if dx else 1) + (4.0 if gat else 2.0) * q * w
    return {"bytes": byts, "flops": flops}


def _cost(c):
    """Seconds, roughly: gathered rows at 7 TB/s, products at 60 TFLOP/s, streams at 4 TB/s."""
    q = _entries(c)
    if c["kind"] == "setup":
        return q * 100e-12
    gathered = 0.0
    for m, k, bwd, dx in _layers(c):
        gat = c["kind"] in ("gat", "gat2")
        w = k if gat else min(m, k)
        gathered += 4.0 * q * max(w, 32) * (1 + (2 if gat else 1) * bool(bwd))
    if c["kind"] == "spmm":
        gathered = 4.0 * q * max(c["f_in"], 32)
    w = work(c)
    return gathered / 7e12 + w["flops"] / 60e12 + w["bytes"] / 4e12


def _largest_tensor(c):
    widths = [max(m, k) for m, k, _, _ in _layers(c)] or [c.get("f_in", 1)]
    return 4 * c["n"] * max(widths)


def tolerance(case):
    """Largest relative error of a tensor against the same path in 64 bits, times about four.

    Chains of fp32 products and sums show up to 4e-7 (gradients of the long reductions 1e-7).  A pre-activation within
    rounding of zero may take the other branch of ReLU, which changes one entry of the masked gradient by its full size:
    up to 5e-4 seen.  The same for LeakyReLU on the attention logits and for the ELU between two layers: 5e-5.
    """
    backward = case["kind"] in ("gcn2", "gat2") or case.get("step")
    if case["kind"] == "setup":
        return {"rel": 1e-6}                           # the weights; every other output is whole numbers
    if backward and (case.get("relu") or case["kind"] == "gcn2"):
        return {"rel": 2e-3}
    if backward and case["kind"] in ("gat", "gat2"):
        return {"rel": 2e-4}
    return {"rel": 2e-6}


# ---- inputs --------------------------------------------------------------------------------------
def _arcs(kind, n, count, gen):
    """`count` node pairs; R-MAT ids are drawn on the next power of two, relabelled and scaled down to n."""
    dev = "cuda"
    if kind == "uniform":
        return (torch.randint(0, n, (count,), generator=gen, device=dev, dtype=torch.int64),
                torch.randint(0, n, (count,), generator=gen, device=dev, dtype=torch.int64))
    scale = max(1, (n - 1).bit_length())
    a, b, c = RMAT
    relabel = torch.randperm(1 << scale, generator=gen, device=dev, dtype=torch.int32)
    us, vs, chunk = [], [], 1 << 24
    for lo in range(0, count, chunk):
        m = min(chunk, count - lo)
        u = torch.zeros(m, dtype=torch.int32, device=dev)
        v = torch.zeros(m, dtype=torch.int32, device=dev)
        for _ in range(scale):
            r = torch.rand(m, generator=gen, device=dev)
            ub = r >= a + b
            vb = ((r >= a) & ~ub) | (r >= a + b + c)
            u = u * 2 + ub
            v = v * 2 + vb
        us.append((relabel[u.long()].long() * n) >> scale)
        vs.append((relabel[v.long()].long() * n) >> scale)
    return torch.cat(us), torch.cat(vs)


def _pattern(case, gen, directed):
    """Raw CSR pattern on the device: sorted rows, no duplicates, no diagonal, exactly `degree` entries a row on average.

    Directed: n * degree distinct arcs.  Undirected: half as many distinct pairs, each stored in both directions."""
    n = case["n"]
    need = n * case["degree"] if directed else n * case["degree"] // 2
    key, more = None, need + need // 8
    while key is None or key.numel() < need:
        u, v = _arcs(case["graph"], n, more, gen)
        if not directed:
            u, v = torch.minimum(u, v), torch.maximum(u, v)
        new = torch.unique((v * n + u)[u != v])
        del u, v
        key, more = new if key is None else torch.unique(torch.cat([key, new])), need
        del new
    surplus = key.numel() - need
    if surplus:                                        # drop evenly spaced ones
        keep = torch.ones(key.numel(), dtype=torch.bool, device="cuda")
        keep[torch.arange(surplus, device="cuda") * key.numel() // surplus] = False
        key = key[keep]
    row = torch.div(key, n, rounding_mode="floor")
    col = key - row * n
    if not directed:
        key = torch.cat([key, col * n + row]).sort().values
        row = torch.div(key, n, rounding_mode="floor")
        col = key - row * n
    del key
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    rowptr[1:] = torch.bincount(row, minlength=n).cumsum(0)
    return rowptr.int(), col.int()


def _graph(case, gen, kind):
    """kind: "sym" (GCN weights, undirected), "mean" (mean weights with CSC arrays), "gat" (pattern with CSC arrays)."""
    n = case["n"]
    rp, col, deg = graphs.add_self_loops(n, *_pattern(case, gen, directed=kind != "sym"))
    col = col.clone()
    q = int(col.numel())
    erow = graphs.expand(n, rp, q)
    if kind == "sym":
        val = torch.empty(q, device="cuda")
        B.gnn_gcn_normalize(n, rp, col, deg, val)
        return B.Graph(n, rp, col, val, erow, symmetric=True)
    colptr, row, perm = graphs.transpose(n, rp, col)
    ecol = graphs.expand(n, colptr, q)
    val = csc_val = None
    if kind == "mean":
        val, csc_val = torch.empty(q, device="cuda"), torch.empty(q, device="cuda")
        B.gnn_aggregator_weights(B.GNN_AGG_MEAN, 0.0, n, rp, col, deg, val)
        B.gnn_gather_f32(q, val, perm, csc_val)
    return B.Graph(n, rp, col, val, erow, colptr, row, perm, csc_val, ecol, symmetric=False)


def _normal(gen, *shape):
    return torch.randn(*shape, generator=gen, device="cuda")


def _glorot(gen, a, b):
    lim = math.sqrt(6.0 / (a + b))
    return (torch.rand(a, b, generator=gen, device="cuda") * 2 - 1) * lim


class _Layer:
    """What a program keeps for one layer: the plan, its buffers, the weights and the gradients' places."""

    def __init__(self, gen, layer, g, m, k, dx, bwd, heads=1, bias=False, relu=False, elu=False, calibrated=False):
        self.layer, self.f = layer, heads * k
        cal = B.GNN_SELECT_CALIBRATED if calibrated else B.GNN_SELECT_PAPER_RULE
        self.plan = B.Plan(layer, g.n, g.nnz, m, k, heads=heads, need_input_grad=dx, has_bias=bias, fuse_relu=relu,
                           fuse_elu=elu, selection=cal)
        self.cache = B.alloc(self.plan.info.cache_bytes)
        self.ws = B.alloc(self.plan.info.workspace_bytes)
        self.act = relu or elu
        self.W = _glorot(gen, m, self.f)
        self.W2 = _glorot(gen, m, self.f) if layer == B.GNN_LAYER_SAGE else None
        self.a = (_glorot(gen, heads, k), _glorot(gen, heads, k)) if layer == B.GNN_LAYER_GAT else None
        self.b = _normal(gen, self.f) if bias else None
        new = lambda *s: torch.empty(*s, device="cuda")  # noqa: E731
        self.Y = new(g.n, self.f)
        if bwd:
            self.dW = new(m, self.f)
            self.dW2 = new(m, self.f) if self.W2 is not None else None
            self.da = (new(heads, k), new(heads, k)) if self.a else None
            self.db = new(self.f) if bias else None
            self.dX = new(g.n, m) if dx else None

    def forward(self, g, X):
        if self.layer == B.GNN_LAYER_GCN:
            B.gcn_layer_fwd(self.plan, g, X, self.W, self.b, self.Y, self.cache, self.ws)
        elif self.layer == B.GNN_LAYER_SAGE:
            B.sage_layer_fwd(self.plan, g, X, self.W, self.W2, self.b, self.Y, self.cache, self.ws)
        else:
            B.gat_layer_fwd(self.plan, g, X, self.W, *self.a, self.b, self.Y, self.cache, self.ws)
        return self.Y

    def backward(self, g, X, dY):
        Y = self.Y if self.act else None
        if self.layer == B.GNN_LAYER_GCN:
            B.gcn_layer_bwd(self.plan, g, X, self.W, Y, dY, self.dW, self.db, self.dX, self.cache, self.ws)
        elif self.layer == B.GNN_LAYER_SAGE:
            B.sage_layer_bwd(self.plan, g, X, self.W, self.W2, Y, dY, self.dW, self.dW2, self.db, self.dX, self.cache,
                             self.ws)
        else:
            B.gat_layer_bwd(self.plan, g, X, self.W, *self.a, dY, self.dW, *self.da, self.db, self.dX, self.cache,
                            self.ws, Y=Y)
        return self.dX

    def gradients(self):
        return [t for t in (self.dW, self.dW2, *(self.da or ()), self.db, self.dX) if t is not None]


class _State:
    pass


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    s = _State()
    s.kind, n, kind = case["kind"], case["n"], case["kind"]
    if kind == "setup":
        s.n, (s.rowptr, s.col) = n, _pattern(case, gen, directed=True)
        return s
    s.g = g = _graph(case, gen, {"sage": "mean", "gat": "gat", "gat2": "gat"}.get(kind, "sym"))
    s.X = _normal(gen, n, case["f_in"])
    if kind == "spmm":
        s.f = case["f_in"]
        s.C = torch.empty_like(s.X)
        s.ws = B.alloc(B.gnn_spmm_workspace_bytes(n, g.nnz, s.f))
        return s
    layer = {"gcn": B.GNN_LAYER_GCN, "gcn2": B.GNN_LAYER_GCN, "sage": B.GNN_LAYER_SAGE}.get(kind, B.GNN_LAYER_GAT)
    heads = case.get("heads", 1)
    if kind == "gcn2":
        dims = [(case["f_in"], case["hidden"], dict(relu=True)), (case["hidden"], case["f_out"], {})]
        s.labels = torch.randint(0, case["f_out"], (n,), generator=gen, device="cuda", dtype=torch.int32)
        s.lws = B.alloc(4 * ((n + 255) // 256))
    elif kind == "gat2":
        k = case["f_out"]
        dims = [(case["f_in"], k, dict(elu=True, bias=True)), (heads * k, k, dict(bias=True))]
        s.target = _normal(gen, n, heads * k)
        s.lws = B.alloc(4096)
    else:
        dims = [(case["f_in"], case["f_out"], dict(bias=case["bias"], relu=case.get("relu", False),
                                                   elu=case.get("elu", False)))]
        s.step = case["step"]
        s.dY = _normal(gen, n, heads * case["f_out"]) if s.step else None
    two = kind in ("gcn2", "gat2")
    s.layers = [_Layer(gen, layer, g, m, k, dx=(i > 0 if two else True), bwd=two or s.step, heads=heads,
                       calibrated=case.get("calibrated", False), **opt) for i, (m, k, opt) in enumerate(dims)]
    if two:
        s.loss = torch.empty(1, device="cuda")
        s.dZ = torch.empty_like(s.layers[1].Y)
    return s


def run(s):
    if s.kind == "setup":
        rp, col, deg = graphs.add_self_loops(s.n, s.rowptr, s.col)
        q = int(col.numel())
        val = torch.empty(q, device="cuda")
        B.gnn_gcn_normalize(s.n, rp, col, deg, val)
        erow = graphs.expand(s.n, rp, q)
        colptr, row, perm = graphs.transpose(s.n, rp, col)
        csc_val = torch.empty_like(val)
        B.gnn_gather_f32(q, val, perm, csc_val)
        ecol = graphs.expand(s.n, colptr, q)
        return [rp, col, deg, val, erow, colptr, row, perm, csc_val, ecol]
    g = s.g
    if s.kind == "spmm":
        B.gnn_spmm_csr(g.n, g.nnz, g.rowptr, g.col, g.val, g.erow, s.X, s.f, s.C, workspace=s.ws)
        return s.C
    if s.kind in ("gcn2", "gat2"):
        first, second = s.layers
        H = first.forward(g, s.X)
        Z = second.forward(g, H)
        if s.kind == "gcn2":
            B.gnn_softmax_xent(g.n, second.f, Z, s.labels, s.dZ, s.loss, s.lws)
        else:
            B.gnn_sum_squared_error(Z.numel(), Z, s.target, s.dZ, s.loss, s.lws)
        dH = second.backward(g, H, s.dZ)
        first.backward(g, s.X, dH)
        return [s.loss, Z, *second.gradients(), *first.gradients()]
    layer = s.layers[0]
    layer.forward(g, s.X)
    if not s.step:
        return layer.Y
    layer.backward(g, s.X, s.dY)
    return [layer.Y, *layer.gradients()]


# ---- the same path in 64 bits, in plain torch ----------------------------------------------------------
SLOPE = 0.2                           # LeakyReLU of the attention logits (the plan's default)


def _entries64(case, seed):
    """(row, col) of A + I in row order, from the same draws as the inputs' graph."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    n = case["n"]
    rowptr, col = _pattern(case, gen, directed=case["kind"] in ("sage", "gat", "gat2", "setup"))
    row = torch.repeat_interleave(torch.arange(n, device="cuda"), (rowptr[1:] - rowptr[:-1]).long())
    loops = torch.arange(n, device="cuda")             # the pattern has no diagonal
    key = torch.cat([row * n + col.long(), loops * (n + 1)]).sort().values
    row = torch.div(key, n, rounding_mode="floor")
    return row, key - row * n


def _propagate64(to, frm, val, X, n):
    """out[to] += val * X[frm], in pieces that fit beside the operands; val [q] or [q, heads], X [n, ...]."""
    out = torch.zeros((n,) + X.shape[1:], dtype=torch.float64, device="cuda")
    piece = max(1 << 16, (1 << 28) // X[0].numel())
    for lo in range(0, to.numel(), piece):
        hi = min(lo + piece, to.numel())
        v = val[lo:hi]
        out.index_add_(0, to[lo:hi], X[frm[lo:hi]] * v.reshape(v.shape + (1,) * (X.dim() - v.dim())))
    return out


def _gat64(layer, row, col, n, X):
    """Forward of one attention layer; returns what backward needs."""
    h, k = layer.a[0].shape
    M = (X @ layer.W.double()).view(n, h, k)
    a_src, a_dst = (t.double() for t in layer.a)
    y = (M * a_src).sum(2)[row] + (M * a_dst).sum(2)[col]
    w = torch.where(y > 0, y, SLOPE * y)
    top = torch.full((n, h), -math.inf, dtype=torch.float64, device="cuda").index_reduce_(0, row, w, "amax")
    alpha = torch.exp(w - top[row])
    alpha = alpha / torch.zeros(n, h, dtype=torch.float64, device="cuda").index_add_(0, row, alpha)[row]
    Y = _propagate64(row, col, alpha, M, n).reshape(n, h * k)
    return M, y, alpha, Y + layer.b.double() if layer.b is not None else Y


def _gat64_backward(layer, row, col, n, X, saved, G):
    M, y, alpha = saved
    h, k = layer.a[0].shape
    a_src, a_dst = (t.double() for t in layer.a)
    Gh = G.view(n, h, k)
    ga = torch.empty_like(alpha)
    piece = max(1 << 16, (1 << 28) // (h * k))
    for lo in range(0, row.numel(), piece):
        ga[lo:lo + piece] = (Gh[row[lo:lo + piece]] * M[col[lo:lo + piece]]).sum(2)
    zero = lambda: torch.zeros(n, h, dtype=torch.float64, device="cuda")  # noqa: E731
    gy = alpha * (ga - zero().index_add_(0, row, alpha * ga)[row]) * torch.where(y > 0, 1.0, SLOPE)
    ds, dd = zero().index_add_(0, row, gy), zero().index_add_(0, col, gy)
    dM = _propagate64(col, row, alpha, Gh, n) + ds[:, :, None] * a_src + dd[:, :, None] * a_dst
    out = [X.t() @ dM.view(n, h * k), (ds[:, :, None] * M).sum(0), (dd[:, :, None] * M).sum(0)]
    return out + ([G.sum(0)] if layer.b is not None else []), dM.view(n, h * k) @ layer.W.double().t()


def _elu(Z):
    return torch.where(Z > 0, Z, torch.expm1(Z))


def exact(case, seed):
    """What `run` returns, in 64 bits; None in the place of whole numbers."""
    kind, n = case["kind"], case["n"]
    row, col = _entries64(case, seed)
    deg = torch.bincount(row, minlength=n).double()
    sym = 1.0 / torch.sqrt(deg[row] * deg[col])
    if kind == "setup":
        order = torch.sort(col, stable=True).indices
        return [None, None, None, sym, None, None, None, None, sym[order], None]
    s = prepare(case, seed)
    X = s.X.double()
    if kind == "spmm":
        return _propagate64(row, col, sym, X, n)
    if kind == "gcn2":
        W1, W2 = (l.W.double() for l in s.layers)
        P = _propagate64(row, col, sym, X, n)
        H = torch.relu(P @ W1)
        Z = _propagate64(row, col, sym, H @ W2, n)
        at = torch.arange(n, device="cuda"), s.labels.long()
        loss = (torch.logsumexp(Z, 1) - Z[at]).sum().reshape(1)
        dZ = torch.softmax(Z, 1)
        dZ[at] -= 1.0
        D = _propagate64(row, col, sym, dZ, n)         # the operator is symmetric
        dH = D @ W2.t()
        return [loss, Z, H.t() @ D, dH, P.t() @ (dH * (H > 0))]
    if kind == "gat2":
        first, second = s.layers
        *saved1, Z1 = _gat64(first, row, col, n, X)
        H = _elu(Z1)
        *saved2, Z = _gat64(second, row, col, n, H)
        dZ = Z - s.target.double()
        g2, dH = _gat64_backward(second, row, col, n, H, saved2, dZ)
        g1, _ = _gat64_backward(first, row, col, n, X, saved1, dH * torch.where(H > 0, 1.0, H + 1.0))
        return [0.5 * (dZ * dZ).sum().reshape(1), Z, *g2, dH, *g1]
    layer = s.layers[0]
    if kind == "gat":
        *saved, Z = _gat64(layer, row, col, n, X)
        Y = _elu(Z) if case["elu"] else Z
        if not s.step:
            return Y
        G = s.dY.double()
        if case["elu"]:
            G = G * torch.where(Y > 0, 1.0, Y + 1.0)
        grads, dX = _gat64_backward(layer, row, col, n, X, saved, G)
        return [Y, *grads, dX]
    val = sym if kind == "gcn" else 1.0 / deg[row]
    W = layer.W.double()
    Wn = W if kind == "gcn" else layer.W2.double()     # the weight behind the operator
    P = _propagate64(row, col, val, X, n)
    Y = P @ Wn
    if kind == "sage":
        Y += X @ W
    if layer.b is not None:
        Y += layer.b.double()
    if case["relu"]:
        Y = torch.relu(Y)
    if not s.step:
        return Y
    G = s.dY.double()
    if case["relu"]:
        G = G * (Y > 0)
    dX = _propagate64(col, row, val, G @ Wn.t(), n)
    grads = [P.t() @ G]
    if kind == "sage":
        grads.insert(0, X.t() @ G)
        dX += G @ W.t()
    return [Y, *grads, *([G.sum(0)] if layer.b is not None else []), dX]
