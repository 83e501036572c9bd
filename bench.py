#!/usr/bin/env python3
"""Benchmark of the GCN / GAT layer hot path on one MI355X.

Default workload: the largest single-GPU configuration, a GCN layer on the R-MAT graph of 2^22 nodes
(degree 32, F_in = 64).  A step = forward + backward of one layer for every F_out of the workload
(64 and 256), each with the plan that gnn_plan_create picks (adaptive ordering + caching, input gradient
required).  Inputs are seeded and synthetic, resident in HBM before the timed region, and all graph
preprocessing (self-loops, degrees, normalisation, row-index expansion, transpose) has run in the
library's kernels.

Prints ONE JSON line:
  value         edge.features per second: sum over the layers of q (F_in + F_out) / time per step
  roofline      the dominant kernel of the workload (the entry-balanced SpMM; for the GAT workloads the
                fused edge kernels): algorithmic HBM bytes per launch / its average duration, timed with
                HIP events on the launch stream around batches of back-to-back launches of that entry point
  cpu_baseline  the fp64 oracle on a bounded sample of the same workload, host cores
  config        names the workload; `all_configs` (default run only) holds, for each of the five
                configurations, the time of the adaptive plan and of the fixed transform-first /
                fused-propagate scheme without cache (GAT: of each caching variant)
Other workloads: --workload cfg1 | cfg2 | cfg3 | cfg4 | gatnet.
"""
from __future__ import annotations

import argparse
import ctypes
import json
import os
import sys
import time

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
HBM_PEAK_GBPS = 8000.0


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--workload", default="cfg5", choices=["cfg1", "cfg2", "cfg3", "cfg4", "cfg5", "gatnet"],
                    help="gatnet: two GAT layers (8 heads, ELU between, squared error) on the cfg4 graph")
    ap.add_argument("--hidden", type=int, default=8, help="gatnet: features per head of both layers (paper: 8..128)")
    ap.add_argument("--selection", default="rule", choices=["rule", "calibrated"],
                    help="GCN AUTO plans: the paper's width rule or the measured SpMM time model")
    ap.add_argument("--aggregator", default="gcn", choices=["gcn", "mean", "gin"],
                    help="GCN workloads: entry values of the propagation matrix (same layer, same schemes)")
    ap.add_argument("--layer", default="gcn", choices=["gcn", "sage"],
                    help="cfg1/cfg2/cfg5: GCN (the headline) or GraphSAGE, which adds a dense self term X W_self")
    ap.add_argument("--constant-input", action="store_true",
                    help="GCN: promise a constant X, so that the cached A'X is computed once")
    ap.add_argument("--scale", type=int, default=None, help="override the R-MAT scale (debug)")
    ap.add_argument("--scheme", default="auto", choices=["auto", "tf_fp", "pf_sp_nocache", "pf_sp_cache"])
    ap.add_argument("--gat-cache", default="auto", choices=["auto", "none", "feat", "nodeatt", "edge"],
                    help="cfg4 / gatnet: GAT caching variant")
    ap.add_argument("--graph", action="store_true",
                    help="GCN workloads: record one step in a HIP graph and time its replays (small graphs are launch-bound)")
    ap.add_argument("--no-input-grad", action="store_true")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-summary", action="store_true", help="default workload: skip the table over all five configurations")
    ap.add_argument("--breakdown", action="store_true", help="also print per-F_out / per-scheme timings to stderr")
    ap.add_argument("--format-study", action="store_true",
                    help="time SpMM on the cfg2 graph and on an even-degree graph of the same size in CSR, coordinate, "
                         "ELLPACK and hybrid storage (App. D / E.1); prints one JSON line")
    ap.add_argument("--row-order-study", action="store_true",
                    help="time SpMM on the chosen GCN workload with the rows of the matrix stored in other orders (by degree, by "
                         "smallest neighbour, by a min-hash of the neighbour set, random): does co-scheduling similar rows cut "
                         "the re-fetch of dense rows?  prints one JSON line")
    ap.add_argument("--copy-reference", action="store_true",
                    help="only run three plain 256 MiB device copies (known bytes, to scale rocprofv3 byte counters)")
    return ap.parse_args()


class HipEvents:
    """Raw HIP events recorded on the stream the binding launches on (torch's events see only torch's
    current stream object; these take the stream handle itself)."""

    def __init__(self, stream):
        self.hip = ctypes.CDLL("libamdhip64.so")
        self.hip.hipEventCreate.argtypes = [ctypes.POINTER(ctypes.c_void_p)]
        self.hip.hipEventElapsedTime.argtypes = [ctypes.POINTER(ctypes.c_float), ctypes.c_void_p, ctypes.c_void_p]
        self.hip.hipEventSynchronize.argtypes = [ctypes.c_void_p]
        self.hip.hipEventRecord.argtypes = [ctypes.c_void_p, ctypes.c_void_p]
        self.stream = stream
        self.e0, self.e1 = self._create(), self._create()

    def _create(self):
        e = ctypes.c_void_p()
        assert self.hip.hipEventCreate(ctypes.byref(e)) == 0
        return e

    def time_ms(self, fn, runs):
        """Average duration of one call of fn over `runs` back-to-back calls between two events."""
        assert self.hip.hipEventRecord(self.e0, ctypes.c_void_p(self.stream)) == 0
        for _ in range(runs):
            fn()
        assert self.hip.hipEventRecord(self.e1, ctypes.c_void_p(self.stream)) == 0
        assert self.hip.hipEventSynchronize(self.e1) == 0
        ms = ctypes.c_float()
        assert self.hip.hipEventElapsedTime(ctypes.byref(ms), self.e0, self.e1) == 0
        return ms.value / runs

    def blocks(self, fn, blocks, runs, warm=2):
        """The paper's protocol (Sec. 4 "Experimental Setup"): blocks of runs, one time per block."""
        for _ in range(warm):
            self.time_ms(fn, max(1, runs // 4))
        return [self.time_ms(fn, runs) for _ in range(blocks)]


def stats(per_run):
    return {"median": round(float(np.median(per_run)), 5), "min": round(float(np.min(per_run)), 5),
            "max": round(float(np.max(per_run)), 5)}


def wall_ms_per_step(torch, step, warmup, steps):
    """W untimed steps, then exactly `steps` steps between two device synchronisations."""
    for _ in range(warmup):
        step()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        step()
    torch.cuda.synchronize()
    return (time.perf_counter() - t0) * 1e3 / steps


# ---- algorithmic bytes (every operand once; re-reads that miss the caches are what a better kernel avoids) ----
def spmm_bytes(n, q, f):
    """One SpMM launch of dense width f: row index, column index and value per entry (12 q), the dense
    operand read once (4 n f), the result written once (4 n f)."""
    return 12 * q + 8 * n * f


def profile_traffic(workload, key):
    """HBM-side bytes per launch of a kernel from the committed rocprofv3 counter summary of this workload
    (FETCH_SIZE and WRITE_SIZE runs, scaled by a plain copy of known size), or None when profiles/ holds none.
    Returns (bytes, file name)."""
    path = os.path.join(HERE, "profiles", f"{workload}_hbm_traffic.txt")
    if not os.path.exists(path):
        return None, None
    for line in open(path):
        if line.startswith("traffic_bytes_per_launch"):
            for item in line.split()[1:]:
                name, value = item.split("=")
                if name == key:
                    return int(value), os.path.relpath(path, HERE)
    return None, None


def spmm_roofline(torch, B, ev, g, launch_widths, workload, step_ms):
    """Times gnn_spmm_csr (main kernel + fix-up) at every dense width a step launches it with."""
    n, q = g.n, g.nnz
    per_width, tot_bytes, tot_ms = {}, 0.0, 0.0
    for f in sorted(set(launch_widths)):
        Bm = torch.randn((n, f), dtype=torch.float32, device="cuda")
        C = torch.empty((n, f), dtype=torch.float32, device="cuda")
        ws = B.alloc(B.gnn_spmm_workspace_bytes(n, q, f))
        runs = 20 if q < 20_000_000 else 5
        times = ev.blocks(lambda: B.gnn_spmm_csr(n, q, g.rowptr, g.col, g.val, g.erow, Bm, f, C, None, False, ws),
                          10 if q < 20_000_000 else 6, runs)
        avg = float(np.mean(times))
        per_width[f] = dict(avg_ms=avg, bytes=spmm_bytes(n, q, f), gather_gbps=(12 * q + 4 * q * f + 4 * n * f) / avg / 1e6)
        cnt = launch_widths.count(f)
        tot_bytes += cnt * spmm_bytes(n, q, f)
        tot_ms += cnt * avg
        del Bm, C, ws
    achieved = tot_bytes / tot_ms / 1e6
    traffic = src = None
    parts = [profile_traffic(workload, f"spmm_f{f}") for f in launch_widths]
    if parts and all(p[0] is not None for p in parts):
        traffic, src = round(sum(p[0] for p in parts) / len(parts)), parts[0][1]
    widths = sorted(per_width)
    return {"bound": "hbm", "kernel": "gnn_spmm_csr (spmm_seg_kernel or hub_gather_kernel, + spmm_fixup_kernel)", "achieved": round(achieved, 1),
            "peak": HBM_PEAK_GBPS, "unit": "GB/s", "frac": round(achieved / HBM_PEAK_GBPS, 4),
            "traffic": traffic, "traffic_source": src,
            # the same launches priced by the bytes the L2s exchanged with the fabric (the profile above)
            "traffic_GBps": None if traffic is None else round(traffic * len(launch_widths) / tot_ms / 1e6, 1),
            "traffic_frac": None if traffic is None else round(traffic * len(launch_widths) / tot_ms / 1e6 / HBM_PEAK_GBPS, 4),
            "launches_per_step": len(launch_widths),
            "bytes_per_launch": {str(f): per_width[f]["bytes"] for f in widths},
            "avg_ms_per_launch": {str(f): round(per_width[f]["avg_ms"], 5) for f in widths},
            "no_reuse_gather_GBps": {str(f): round(per_width[f]["gather_gbps"], 1) for f in widths},
            "time_share_of_step": round(tot_ms / step_ms, 3)}


def spmm_launch_widths(B, info, f_in, k):
    """Dense width of every SpMM that forward + backward of a GCN plan launch."""
    out = [int(info.spmm_width_fwd)] if info.spmm_width_fwd else []
    if info.bwd == B.GNN_BWD_FUSED_PROPAGATE:
        out.append(k)
    else:
        out += [f_in] * int(info.spmm_width_bwd // f_in)
    return out


def summary_record(rec):
    """One line of the adaptive-against-fixed table.  `equal_spmm_work`: both schemes run SpMMs of the same total
    dense width (F_out = F_in with dX, or the same scheme): the method predicts a tie there (Sec. 3.1)."""
    (auto_ms, auto_name, auto_w), (fix_ms, fix_name, fix_w) = rec["auto"], rec["tf_fp"]
    return {"auto_ms": round(auto_ms, 4), "fixed_ms": round(fix_ms, 4), "auto_scheme": auto_name,
            "spmm_width_auto": auto_w, "spmm_width_fixed": fix_w, "equal_spmm_work": auto_w == fix_w,
            "speedup": round(fix_ms / auto_ms, 3)}


SCHEMES = ("auto", "tf_fp", "pf_sp_nocache", "pf_sp_cache")


def scheme_kw(B, name):
    return {"auto": {},
            "tf_fp": dict(order=B.GNN_ORDER_TRANSFORM_FIRST, bwd=B.GNN_BWD_FUSED_PROPAGATE, cache=B.GNN_CACHE_NONE),
            "pf_sp_nocache": dict(order=B.GNN_ORDER_PROPAGATE_FIRST, bwd=B.GNN_BWD_SPLIT_PROPAGATE, cache=B.GNN_CACHE_NONE),
            "pf_sp_cache": dict(order=B.GNN_ORDER_PROPAGATE_FIRST, bwd=B.GNN_BWD_SPLIT_PROPAGATE, cache=B.GNN_CACHE_AX)}[name]


def scheme_name(B, info):
    order = "TF" if info.order == B.GNN_ORDER_TRANSFORM_FIRST else "PF"
    bwd = "FP" if info.bwd == B.GNN_BWD_FUSED_PROPAGATE else "SP"
    return f"{order}+{bwd}" + ("+cache" if info.cache == B.GNN_CACHE_AX else "")


# =================================================================================================
# GCN (and GraphSAGE) single layer: cfg1, cfg2, cfg5
# =================================================================================================
class GcnSingle:
    def __init__(self, args, torch, B, graphs, w, layer="gcn", aggregator="gcn"):
        self.args, self.torch, self.B, self.w, self.layer = args, torch, B, w, layer
        agg = {"gcn": B.GNN_AGG_GCN_SYM, "mean": B.GNN_AGG_MEAN, "gin": B.GNN_AGG_GIN_SUM}[aggregator]
        self.g = graphs.gcn_graph(w.rowptr, w.col, "cuda", symmetric=True, aggregator=agg, eps=0.1)
        self.f_in, self.f_outs = w.dims["f_in"], w.dims["f_outs"]
        self.X = torch.from_numpy(w.tensors["X"]).cuda()

    def make_layer(self, k, scheme, dx, selection="rule", constant_input=False):
        B, torch, w, g = self.B, self.torch, self.w, self.g
        kind = B.GNN_LAYER_SAGE if self.layer == "sage" else B.GNN_LAYER_GCN
        plan = B.Plan(kind, g.n, g.nnz, self.f_in, k, need_input_grad=dx, constant_input=constant_input,
                      selection=B.GNN_SELECT_CALIBRATED if selection == "calibrated" else B.GNN_SELECT_PAPER_RULE,
                      **scheme_kw(B, scheme))
        e = lambda *s: torch.empty(s, dtype=torch.float32, device="cuda")
        L = dict(k=k, plan=plan, W=torch.from_numpy(w.tensors[f"W{k}"]).cuda(),
                 dY=torch.from_numpy(w.tensors[f"dY{k}"]).cuda(), Y=e(g.n, k), dW=e(self.f_in, k),
                 dX=e(g.n, self.f_in) if dx else None, ws=B.alloc(plan.info.workspace_bytes),
                 cache=B.alloc(plan.info.cache_bytes) if plan.info.cache_bytes else None)
        if self.layer == "sage":
            L["Ws"] = torch.from_numpy(np.ascontiguousarray(w.tensors[f"W{k}"][::-1])).cuda()   # SAGE self weight
            L["dWs"] = e(self.f_in, k)
        return L

    def fwd(self, L):
        B, g = self.B, self.g
        if self.layer == "sage":
            B.sage_layer_fwd(L["plan"], g, self.X, L["Ws"], L["W"], None, L["Y"], L["cache"], L["ws"])
        else:
            B.gcn_layer_fwd(L["plan"], g, self.X, L["W"], None, L["Y"], L["cache"], L["ws"])

    def bwd(self, L):
        B, g = self.B, self.g
        if self.layer == "sage":
            B.sage_layer_bwd(L["plan"], g, self.X, L["Ws"], L["W"], None, L["dY"], L["dWs"], L["dW"], None, L["dX"],
                             L["cache"], L["ws"])
        else:
            B.gcn_layer_bwd(L["plan"], g, self.X, L["W"], None, L["dY"], L["dW"], None, L["dX"], L["cache"], L["ws"])

    def step_ms(self, layers, warmup, steps):
        def step():
            for L in layers:
                self.fwd(L)
                self.bwd(L)
        return wall_ms_per_step(self.torch, step, warmup, steps)

    def summary(self, warmup=3, steps=10):
        """Adaptive plan against the fixed transform-first / fused-propagate scheme without cache, for every
        F_out of the workload, with and without the input gradient (the design of Sec. 4.1)."""
        out = {}
        for dx in (True, False):
            for k in self.f_outs:
                rec = {}
                for scheme in ("auto", "tf_fp"):
                    L = self.make_layer(k, scheme, dx)
                    info = L["plan"].info
                    rec[scheme] = (self.step_ms([L], warmup, steps), scheme_name(self.B, info),
                                   int(info.spmm_width_fwd + info.spmm_width_bwd))
                    del L
                out[f"F_out={k},{'dX' if dx else 'no dX'}"] = summary_record(rec)
        return out


def bench_gcn_single(args, torch, B, graphs, synth, oracle_mod):
    if args.workload == "cfg1":
        w = synth.config1()
    elif args.workload == "cfg2":
        w = synth.config2(scale=args.scale or 17)
    else:
        w = synth.config5(scale=args.scale or 22)
    run = GcnSingle(args, torch, B, graphs, w, args.layer, args.aggregator)
    g, f_in, f_outs = run.g, run.f_in, run.f_outs
    n, q = g.n, g.nnz
    need_dx = not args.no_input_grad
    layers = [run.make_layer(k, args.scheme, need_dx, args.selection, args.constant_input) for k in f_outs]
    def step():
        for L in layers:
            run.fwd(L)
            run.bwd(L)

    if args.graph:
        for _ in range(args.warmup):
            step()
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            step()
        torch.cuda.current_stream().wait_stream(side)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            step()
        ms_per_step = wall_ms_per_step(torch, graph.replay, 2, args.steps)
    else:
        ms_per_step = wall_ms_per_step(torch, step, args.warmup, args.steps)
    edge_feat = sum(q * (f_in + k) for k in f_outs)

    ev = HipEvents(torch.cuda.current_stream().cuda_stream)
    launch_widths = []
    for L in layers:
        launch_widths += spmm_launch_widths(B, L["plan"].info, f_in, L["k"])
    wl = args.workload
    roofline = spmm_roofline(torch, B, ev, g, launch_widths, wl, ms_per_step)

    # per-layer forward / backward times, the paper's protocol with shorter blocks
    big = q > 20_000_000
    layer_times = {}
    for L in layers:
        layer_times[str(L["k"])] = {
            "scheme": scheme_name(B, L["plan"].info),
            "fwd_ms": stats(ev.blocks(lambda: run.fwd(L), 5 if big else 10, 4 if big else 20)),
            "bwd_ms": stats(ev.blocks(lambda: run.bwd(L), 5, 4 if big else 20))}
    if args.breakdown:
        print(json.dumps(layer_times, indent=1), file=sys.stderr)

    cpu = None
    if oracle_mod is not None:
        cpu = cpu_baseline_gcn(oracle_mod, w, args, f_in, f_outs, need_dx, q)

    config = {"workload": f"{w.name}: R-MAT/ER graph n={n}, nnz={q} (self-loops incl.), F_in={f_in}, "
                          f"F_out={list(f_outs)}, {args.layer.upper()} single layer fwd+bwd, scheme={args.scheme}, "
                          f"input_grad={need_dx}, selection={args.selection}, constant_input={args.constant_input}, "
                          f"aggregator={args.aggregator}, hip_graph={args.graph}",
              "layer_times_ms": layer_times}
    del layers
    return w, run, {"metric": "GCN layer fwd+bwd edge-feat/s (adaptive ordering + caching)",
                    "value": edge_feat / (ms_per_step * 1e-3), "ms_per_step": ms_per_step, "config": config,
                    "roofline": roofline, "cpu_baseline": cpu}


def cpu_baseline_gcn(oracle, w, args, f_in, f_outs, need_dx, q):
    """The fp64 oracle on whole layers (forward + backward) of the same workload, about 10-30 s of CPU work:
    as many whole steps as fit, or on the large graphs the first layer of the step only."""
    rp, c, deg = oracle.add_self_loops_degree(w.rowptr, w.col)
    val = oracle.gcn_normalize(rp, c, deg) if args.aggregator == "gcn" else \
        oracle.aggregator_weights(rp, c, deg, args.aggregator, 0.1)
    sym = args.aggregator != "mean"                       # undirected graph, symmetric weights: A'^T G = A' G
    ks = list(f_outs) if q < 20_000_000 else list(f_outs)[:1]
    Xh = w.tensors["X"]

    def one_pass():
        for k in ks:
            Wh, dYh = w.tensors[f"W{k}"], w.tensors[f"dY{k}"]
            if args.layer == "sage":
                oracle.sage_forward(rp, c, val, Xh, Wh[::-1], Wh)
                oracle.sage_backward(rp, c, val, Xh, Wh[::-1], Wh, dYh, None, need_dx)
            else:
                oracle.gcn_forward(rp, c, val, Xh, Wh)
                oracle.gcn_backward(rp, c, val, Xh, Wh, dYh, None, need_dx, symmetric=sym)

    t0 = time.perf_counter()
    passes = 0
    while passes < 8 and time.perf_counter() - t0 < 10.0:
        one_pass()
        passes += 1
    dt = (time.perf_counter() - t0) / passes
    return {"value": sum(q * (f_in + k) for k in ks) / dt, "unit": "edge*feat/s", "cores": oracle.num_threads(),
            "kind": "oracle",
            "sample": f"{passes} x (forward + backward of the layer(s) F_out = {ks} of the step's {list(f_outs)}), "
                      f"{dt * passes:.1f} s in total, scaled by q (F_in + F_out) of those layers",
            "ms_per_sample": round(dt * 1e3, 2)}


# =================================================================================================
# two-layer GCN network: cfg3
# =================================================================================================
class GcnNetwork:
    """R-MAT 2^20, degree 50, 100 -> 256 -> 47, ReLU between the layers, sum-reduced softmax cross-entropy:
    one training step without the optimiser."""

    def __init__(self, torch, B, graphs, w):
        self.torch, self.B, self.w = torch, B, w
        self.g = graphs.gcn_graph(w.rowptr, w.col, "cuda")
        self.d = {key: torch.from_numpy(v).cuda() for key, v in w.tensors.items()}

    def make(self, scheme, selection="rule", constant_input=False):
        B, torch, g = self.B, self.torch, self.g
        f0, f1, f2 = self.w.dims["dims"]
        n, q = g.n, g.nnz
        kw = scheme_kw(B, scheme)
        sel = B.GNN_SELECT_CALIBRATED if selection == "calibrated" else B.GNN_SELECT_PAPER_RULE
        p1 = B.Plan(B.GNN_LAYER_GCN, n, q, f0, f1, need_input_grad=False, fuse_relu=True, selection=sel,
                    constant_input=constant_input, **kw)
        p2 = B.Plan(B.GNN_LAYER_GCN, n, q, f1, f2, need_input_grad=True, selection=sel, **kw)
        e = lambda *s: torch.empty(s, dtype=torch.float32, device="cuda")
        net = dict(p1=p1, p2=p2, ws=B.alloc(max(p1.info.workspace_bytes, p2.info.workspace_bytes, 4 * ((n + 255) // 256))),
                   c1=B.alloc(p1.info.cache_bytes) if p1.info.cache_bytes else None,
                   c2=B.alloc(p2.info.cache_bytes) if p2.info.cache_bytes else None,
                   H1=e(n, f1), Z=e(n, f2), dZ=e(n, f2), dH1=e(n, f1), dW1=e(f0, f1), dW2=e(f1, f2), loss=e(1))
        return net

    def step(self, N):
        B, g, d = self.B, self.g, self.d
        f2 = self.w.dims["dims"][2]
        B.gcn_layer_fwd(N["p1"], g, d["X"], d["W1"], None, N["H1"], N["c1"], N["ws"])
        B.gcn_layer_fwd(N["p2"], g, N["H1"], d["W2"], None, N["Z"], N["c2"], N["ws"])
        B.gnn_softmax_xent(g.n, f2, N["Z"], d["labels"], N["dZ"], N["loss"], N["ws"])
        B.gcn_layer_bwd(N["p2"], g, N["H1"], d["W2"], None, N["dZ"], N["dW2"], None, N["dH1"], N["c2"], N["ws"])
        B.gcn_layer_bwd(N["p1"], g, None if N["p1"].info.cache == B.GNN_CACHE_AX else d["X"], d["W1"], N["H1"],
                        N["dH1"], N["dW1"], None, None, N["c1"], N["ws"])

    def summary(self, warmup=2, steps=5):
        rec = {}
        for scheme in ("auto", "tf_fp"):
            N = self.make(scheme)
            rec[scheme] = (wall_ms_per_step(self.torch, lambda: self.step(N), warmup, steps),
                           [scheme_name(self.B, N[p].info) for p in ("p1", "p2")],
                           sum(int(N[p].info.spmm_width_fwd + N[p].info.spmm_width_bwd) for p in ("p1", "p2")))
            del N
        return {"100->256->47": summary_record(rec)}


def bench_gcn_network(args, torch, B, graphs, synth, oracle):
    if args.scheme not in ("auto", "tf_fp"):
        sys.exit("bench.py: cfg3 takes --scheme auto or tf_fp")
    w = synth.config3(scale=args.scale or 20)
    run = GcnNetwork(torch, B, graphs, w)
    g, (f0, f1, f2) = run.g, w.dims["dims"]
    n, q = g.n, g.nnz
    N = run.make(args.scheme, args.selection, args.constant_input)
    ms = wall_ms_per_step(torch, lambda: run.step(N), args.warmup, args.steps)
    edge_feat = q * (f0 + f1) + q * (f1 + f2)
    ev = HipEvents(torch.cuda.current_stream().cuda_stream)
    launch_widths = spmm_launch_widths(B, N["p1"].info, f0, f1) + spmm_launch_widths(B, N["p2"].info, f1, f2)
    if args.constant_input and N["p1"].info.cache == B.GNN_CACHE_AX:
        launch_widths.remove(f0)                          # the cached A'X is not recomputed
    roofline = spmm_roofline(torch, B, ev, g, launch_widths, "cfg3", ms)
    cpu = None
    if oracle is not None:
        # sample: forward + backward of the second layer (256 -> 47, with dX) on the oracle's own first-layer output
        rp, c, deg = oracle.add_self_loops_degree(w.rowptr, w.col)
        val = oracle.gcn_normalize(rp, c, deg)
        H1 = np.maximum(w.tensors["X"].astype(np.float64) @ w.tensors["W1"].astype(np.float64), 0.0)   # any input of that shape
        dZ = np.random.default_rng(0).standard_normal((n, f2))
        t0 = time.perf_counter()
        oracle.gcn_forward(rp, c, val, H1, w.tensors["W2"])
        oracle.gcn_backward(rp, c, val, H1, w.tensors["W2"], dZ, None, True, symmetric=True)
        dt = time.perf_counter() - t0
        cpu = {"value": q * (f1 + f2) / dt, "unit": "edge*feat/s", "cores": oracle.num_threads(), "kind": "oracle",
               "sample": f"forward + backward of the second layer only ({f1} -> {f2}, with dX), {dt:.1f} s, scaled by "
                         f"q (F_in + F_out) of that layer", "ms_per_sample": round(dt * 1e3, 2)}
    config = {"workload": f"{w.name}: R-MAT n={n}, nnz={q} (self-loops incl.), {f0}->{f1}->{f2}, ReLU, "
                          f"softmax cross-entropy, fwd+bwd, scheme={args.scheme}, selection={args.selection}, "
                          f"constant_input={args.constant_input}",
              "schemes": [scheme_name(B, N[p].info) for p in ("p1", "p2")],
              "spmm_widths": launch_widths, "loss": float(N["loss"].item())}
    return {"metric": "two-layer GCN training step edge-feat/s", "value": edge_feat / (ms * 1e-3), "ms_per_step": ms,
            "config": config, "roofline": roofline, "cpu_baseline": cpu}


# =================================================================================================
# GAT layer: cfg4, and the two-layer GAT network
# =================================================================================================
GAT_VARIANTS = ("none", "feat", "nodeatt", "edge")


def gat_variant(B, name):
    return {"auto": B.GNN_CACHE_AUTO, "none": B.GNN_CACHE_NONE, "feat": B.GNN_CACHE_GAT_FEAT,
            "nodeatt": B.GNN_CACHE_GAT_FEAT_NODEATT, "edge": B.GNN_CACHE_GAT_FEAT_EDGE}[name]


class GatSingle:
    """R-MAT 2^17 directed, F_in = 256, 8 heads x 8 features, LeakyReLU slope 0.2, bias."""

    def __init__(self, torch, B, graphs, w):
        self.torch, self.B, self.w = torch, B, w
        self.g = graphs.gat_graph(w.rowptr, w.col, "cuda")
        self.d = {key: torch.from_numpy(v).cuda() for key, v in w.tensors.items()}
        self.h, self.k, self.m = w.dims["heads"], w.dims["f_out"], w.dims["f_in"]

    def make(self, variant, need_dx=True, selection="rule"):
        B, torch, g = self.B, self.torch, self.g
        h, k, m = self.h, self.k, self.m
        sel = B.GNN_SELECT_CALIBRATED if selection == "calibrated" else B.GNN_SELECT_PAPER_RULE
        plan = B.Plan(B.GNN_LAYER_GAT, g.n, g.nnz, m, k, heads=h, need_input_grad=need_dx, has_bias=True,
                      leaky_slope=0.2, cache=gat_variant(B, variant), selection=sel)
        e = lambda *s: torch.empty(s, dtype=torch.float32, device="cuda")
        return dict(plan=plan, Y=e(g.n, h * k), dW=e(m, h * k), das=e(h, k), dad=e(h, k), db=e(h * k),
                    dX=e(g.n, m) if need_dx else None, ws=B.alloc(plan.info.workspace_bytes),
                    cache=B.alloc(plan.info.cache_bytes) if plan.info.cache_bytes else None)

    def fwd(self, L):
        d = self.d
        self.B.gat_layer_fwd(L["plan"], self.g, d["X"], d["W"], d["a_src"], d["a_dst"], d["b"], L["Y"], L["cache"], L["ws"])

    def bwd(self, L):
        d = self.d
        self.B.gat_layer_bwd(L["plan"], self.g, d["X"], d["W"], d["a_src"], d["a_dst"], d["dY"], L["dW"], L["das"],
                             L["dad"], L["db"], L["dX"], L["cache"], L["ws"])

    def summary(self, warmup=3, steps=10):
        out = {}
        for variant in GAT_VARIANTS:
            L = self.make(variant)
            ms = wall_ms_per_step(self.torch, lambda: (self.fwd(L), self.bwd(L)), warmup, steps)
            out[variant] = {"fwd_bwd_ms": round(ms, 4), "cache_MiB": round(L["plan"].info.cache_bytes / 2**20, 1)}
            del L
        return out


def gat_edge_bytes(n, q, h, k, variant):
    """Algorithmic bytes of the edge phase of one GAT forward + backward (everything between the dense
    products), every array once per pass that needs it: the index arrays of the three passes (erow, col twice;
    ecol, row, perm: 28 q), forward M read and Y written (8 n h k), backward G and M read by both passes and dM
    written (20 n h k), the per-node vectors s, d, row statistics, node values, ds, dd (about 60 n h), and, for
    the variant that keeps them, alpha and the mask written once and read by both backward passes (15 q h)."""
    per_edge = 15 * q * h if variant == "edge" else 0
    return 28 * q + 28 * n * h * k + 60 * n * h + per_edge


def bench_gat(args, torch, B, graphs, synth, oracle):
    w = synth.config4(scale=args.scale or 17)
    run = GatSingle(torch, B, graphs, w)
    g, h, k, m = run.g, run.h, run.k, run.m
    n, q, f = g.n, g.nnz, h * k
    need_dx = not args.no_input_grad
    L = run.make(args.gat_cache, need_dx, args.selection)
    ms = wall_ms_per_step(torch, lambda: (run.fwd(L), run.bwd(L)), args.warmup, args.steps)
    ev = HipEvents(torch.cuda.current_stream().cuda_stream)
    fwd_ms = stats(ev.blocks(lambda: run.fwd(L), 10, 20))
    bwd_ms = stats(ev.blocks(lambda: run.bwd(L), 5, 20))
    edge_feat = q * (m + f)

    # the two sparse operators on their own: the fused edge softmax + aggregation (the forward edge phase, one
    # launch of the entry-balanced walker and its fix-up) and the SDDMM (App. E.2)
    variant_name = {int(gat_variant(B, v)): v for v in GAT_VARIANTS}[int(L["plan"].info.cache)]
    roofline = gat_operator_roofline(torch, B, ev, g, h, k, run.d["dY"], "cfg4")
    roofline["edge_phase"] = gat_edge_phase(args, torch, B, ev, run, L, variant_name)
    cpu = None
    if oracle is not None:
        t = w.tensors
        rp, c, _ = oracle.add_self_loops_degree(w.rowptr, w.col)
        t0 = time.perf_counter()
        passes = 0
        while passes < 4 and time.perf_counter() - t0 < 10.0:
            oracle.gat_forward(rp, c, t["X"], t["W"], t["a_src"], t["a_dst"], t["b"], h, 0.2)
            oracle.gat_backward(rp, c, t["X"], t["W"], t["a_src"], t["a_dst"], t["dY"], h, 0.2, need_dx)
            passes += 1
        dt = (time.perf_counter() - t0) / passes
        cpu = {"value": edge_feat / dt, "unit": "edge*feat/s", "cores": oracle.num_threads(), "kind": "oracle",
               "sample": f"{passes} whole steps (forward + backward, recomputing variant) of the same workload, "
                         f"{dt * passes:.1f} s in total", "ms_per_sample": round(dt * 1e3, 2)}
    config = {"workload": f"{w.name}: R-MAT directed n={n}, nnz={q} (self-loops incl.), F_in={m}, heads={h}, "
                          f"F_out={k}, GAT single layer fwd+bwd, cache variant={variant_name}, input_grad={need_dx}, "
                          f"selection={args.selection}",
              "fwd_ms": fwd_ms, "bwd_ms": bwd_ms, "cache_bytes": int(L["plan"].info.cache_bytes)}
    return {"metric": "GAT layer fwd+bwd edge-feat/s", "value": edge_feat / (ms * 1e-3), "ms_per_step": ms,
            "config": config, "roofline": roofline, "cpu_baseline": cpu}


def gat_operator_roofline(torch, B, ev, g, h, k, feat, workload):
    """gnn_gat_aggregate_csr and gnn_sddmm_csr timed on their own, priced by their algorithmic bytes: index
    arrays once, every dense operand once, outputs once."""
    n, q, f = g.n, g.nnz, h * k
    e = lambda *s: torch.empty(s, dtype=torch.float32, device="cuda")
    sv, dv = torch.randn((n, h), device="cuda"), torch.randn((n, h), device="cuda")
    Y, stat, D = e(n, f), e(n, h, 2), e(q, h)
    ws = B.alloc(B.gnn_gat_aggregate_workspace_bytes(q, h, k))
    agg_ms = float(np.mean(ev.blocks(lambda: B.gnn_gat_aggregate_csr(n, q, g.rowptr, g.erow, g.col, feat, sv, dv, h, k, 0.2,
                                                                      None, False, Y, stat, ws), 10, 20)))
    agg_bytes = 8 * q + 8 * n * f + 16 * n * h              # erow, col; M read, Y written; s, d read, (max, sum) written
    sddmm_ms = float(np.mean(ev.blocks(lambda: B.gnn_sddmm_csr(n, q, g.erow, g.col, None, feat, Y, h, k, D), 10, 20)))
    sddmm_bytes = 8 * q + 8 * n * f + 4 * q * h             # erow, col; both dense operands once; D written
    traffic, src = profile_traffic(workload, "gat_aggregate")
    return {"bound": "hbm", "kernel": f"seg_walk_kernel<FwdOp> + seg_fixup_kernel (gnn_gat_aggregate_csr: edge softmax + "
                                      f"aggregation in one pass, {h} heads x {k} features)",
            "achieved": round(agg_bytes / agg_ms / 1e6, 1), "peak": HBM_PEAK_GBPS, "unit": "GB/s",
            "frac": round(agg_bytes / agg_ms / 1e6 / HBM_PEAK_GBPS, 4), "traffic": traffic, "traffic_source": src,
            "traffic_frac": None if traffic is None else round(traffic / agg_ms / 1e6 / HBM_PEAK_GBPS, 4),
            "bytes_per_launch": agg_bytes, "avg_ms_per_launch": round(agg_ms, 5),
            "no_reuse_gather_GBps": round((8 * q + 4 * q * f + 4 * n * f + 16 * n * h) / agg_ms / 1e6, 1),
            "sddmm": {"kernel": "sddmm_edge_kernel (gnn_sddmm_csr)", "bytes_per_launch": sddmm_bytes,
                      "avg_ms_per_launch": round(sddmm_ms, 5), "achieved": round(sddmm_bytes / sddmm_ms / 1e6, 1),
                      "frac": round(sddmm_bytes / sddmm_ms / 1e6 / HBM_PEAK_GBPS, 4),
                      "traffic": profile_traffic(workload, "sddmm")[0]}}


def gat_edge_phase(args, torch, B, ev, run, L, variant_name):
    """Time of the layer's sparse (edge) phase: the whole layer minus its dense products, which are timed on
    their own through gnn_gemm with the same shapes; priced by gat_edge_bytes."""
    g, h, k, m = run.g, run.h, run.k, run.m
    n, q, f = g.n, g.nnz, h * k
    X, W = run.d["X"], run.d["W"]
    e = lambda *s: torch.empty(s, dtype=torch.float32, device="cuda")
    Mb, dWb, dXb = e(n, f), e(m, f), e(n, m)
    ws = B.alloc(max(B.gnn_gemm_workspace_bytes(0, 0, n, f, m), B.gnn_gemm_workspace_bytes(1, 0, m, f, n)))
    t_nn = float(np.mean(ev.blocks(lambda: B.gnn_gemm(0, 0, n, f, m, X, W, Mb, None, False, ws), 5, 20)))
    t_tn = float(np.mean(ev.blocks(lambda: B.gnn_gemm(1, 0, m, f, n, X, Mb, dWb, None, False, ws), 5, 20)))
    t_nt = float(np.mean(ev.blocks(lambda: B.gnn_gemm(0, 1, n, m, f, Mb, W, dXb, None, False, ws), 5, 20)))
    layer = float(np.mean(ev.blocks(lambda: (run.fwd(L), run.bwd(L)), 5, 20)))
    dense = t_nn * (2 if variant_name == "none" else 1) + t_tn + (t_nt if L["dX"] is not None else 0.0)
    edge = max(layer - dense, 1e-6)
    by = gat_edge_bytes(n, q, h, k, variant_name)
    return {"ms": round(edge, 5), "dense_products_ms": round(dense, 5), "algorithmic_bytes": by,
            "achieved_GBps": round(by / edge / 1e6, 1), "frac_of_hbm_peak": round(by / edge / 1e6 / HBM_PEAK_GBPS, 4)}


def bench_gat_network(args, torch, B, graphs, synth, oracle):
    """Two-layer GAT network of Sec. 4 on the cfg4 graph: GAT(256 -> 8 x hidden) -> ELU -> GAT(-> 8 x hidden),
    squared-error loss; one step = forward + loss + backward of both layers."""
    w = synth.config4(scale=args.scale or 17)
    h, m, k = w.dims["heads"], w.dims["f_in"], args.hidden
    g = graphs.gat_graph(w.rowptr, w.col, "cuda")
    n, q, f = g.n, g.nnz, h * k
    variant = gat_variant(B, args.gat_cache)
    sel = B.GNN_SELECT_CALIBRATED if args.selection == "calibrated" else B.GNN_SELECT_PAPER_RULE
    p1 = B.Plan(B.GNN_LAYER_GAT, n, q, m, k, heads=h, need_input_grad=False, has_bias=True, cache=variant, fuse_elu=True,
                selection=sel)
    p2 = B.Plan(B.GNN_LAYER_GAT, n, q, f, k, heads=h, need_input_grad=True, has_bias=True, cache=variant, selection=sel)
    gen = torch.Generator(device="cuda").manual_seed(0)
    rnd = lambda *s, scale=1.0: torch.randn(s, device="cuda", generator=gen) * scale
    X = torch.from_numpy(w.tensors["X"]).cuda()
    W1, W2 = rnd(m, f, scale=(2.0 / (m + f)) ** 0.5), rnd(f, f, scale=(1.0 / f) ** 0.5)
    a = [rnd(h, k, scale=(2.0 / (h + k)) ** 0.5) for _ in range(4)]
    b1, b2, T = rnd(f, scale=0.1), rnd(f, scale=0.1), rnd(n, f)
    e = lambda *s: torch.empty(s, dtype=torch.float32, device="cuda")
    H1, Z, dZ, dH1, loss = e(n, f), e(n, f), e(n, f), e(n, f), e(1)
    g1 = (e(m, f), e(h, k), e(h, k), e(f))
    g2 = (e(f, f), e(h, k), e(h, k), e(f))
    ws = B.alloc(max(p1.info.workspace_bytes, p2.info.workspace_bytes, 4096))
    c1 = B.alloc(p1.info.cache_bytes) if p1.info.cache_bytes else None
    c2 = B.alloc(p2.info.cache_bytes) if p2.info.cache_bytes else None

    def step():
        B.gat_layer_fwd(p1, g, X, W1, a[0], a[1], b1, H1, c1, ws)
        B.gat_layer_fwd(p2, g, H1, W2, a[2], a[3], b2, Z, c2, ws)
        B.gnn_sum_squared_error(Z.numel(), Z, T, dZ, loss, ws)
        B.gat_layer_bwd(p2, g, H1, W2, a[2], a[3], dZ, g2[0], g2[1], g2[2], g2[3], dH1, c2, ws)
        B.gat_layer_bwd(p1, g, X, W1, a[0], a[1], dH1, g1[0], g1[1], g1[2], g1[3], None, c1, ws, Y=H1)

    ms = wall_ms_per_step(torch, step, args.warmup, args.steps)
    edge_feat = q * (m + f) + q * (f + f)
    ev = HipEvents(torch.cuda.current_stream().cuda_stream)
    roofline = gat_operator_roofline(torch, B, ev, g, h, k, dZ, "gatnet") if k % 4 == 0 and k <= 256 and (k // 4) & (k // 4 - 1) == 0 \
        else None
    cpu = None
    if oracle is not None:
        # sample: forward + backward of the first layer alone (256 -> 8 x hidden), on the host copies of its inputs
        rp, c, _ = oracle.add_self_loops_degree(w.rowptr, w.col)
        Xh, W1h, a0, a1, b1h = (x.cpu().numpy() for x in (X, W1, a[0], a[1], b1))
        Gh = np.random.default_rng(0).standard_normal((n, f))
        t0 = time.perf_counter()
        oracle.gat_forward(rp, c, Xh, W1h, a0, a1, b1h, h, 0.2)
        oracle.gat_backward(rp, c, Xh, W1h, a0, a1, Gh, h, 0.2, False)
        dt = time.perf_counter() - t0
        cpu = {"value": q * (m + f) / dt, "unit": "edge*feat/s", "cores": oracle.num_threads(), "kind": "oracle",
               "sample": f"forward + backward of the first layer only ({m} -> {h} x {k}, no dX, without the ELU), {dt:.1f} s, "
                         f"scaled by q (F_in + heads F_out) of that layer", "ms_per_sample": round(dt * 1e3, 2)}
    config = {"workload": f"gatnet on {w.name}: n={n}, nnz={q}, GAT({m} -> {h} x {k}) -> ELU -> GAT({f} -> {h} x {k}), "
                          f"squared error, cache variant={int(p1.info.cache)}",
              "cache_bytes": int(p1.info.cache_bytes + p2.info.cache_bytes)}
    return {"metric": "two-layer GAT network fwd+bwd edge-feat/s", "value": edge_feat / (ms * 1e-3), "ms_per_step": ms,
            "config": config, "roofline": roofline, "cpu_baseline": cpu}


# =================================================================================================
def all_configs_summary(args, torch, B, graphs, synth, have):
    """Adaptive against fixed scheme on every configuration (GAT: every caching variant).  `have` holds the
    runner of the workload that was just benchmarked, so that its graph is not built twice."""
    out = {}
    makers = {"cfg1": lambda: GcnSingle(args, torch, B, graphs, synth.config1()),
              "cfg2": lambda: GcnSingle(args, torch, B, graphs, synth.config2()),
              "cfg3": lambda: GcnNetwork(torch, B, graphs, synth.config3()),
              "cfg4": lambda: GatSingle(torch, B, graphs, synth.config4()),
              "cfg5": lambda: GcnSingle(args, torch, B, graphs, synth.config5())}
    for name in ("cfg5", "cfg1", "cfg2", "cfg3", "cfg4"):
        run = have.pop(name, None) or makers[name]()
        out[name] = run.summary()
        del run
        torch.cuda.empty_cache()
    gcn = [rec for name in ("cfg1", "cfg2", "cfg3", "cfg5") for rec in out[name].values()]
    out["adaptive_within_3_percent_of_fixed_where_work_is_equal"] = all(
        r["auto_ms"] <= 1.03 * r["fixed_ms"] for r in gcn if r["equal_spmm_work"])
    out["adaptive_faster_where_work_differs"] = all(r["auto_ms"] < r["fixed_ms"] for r in gcn if not r["equal_spmm_work"])
    return out


def format_study(args, torch, B, graphs, synth):
    """SpMM time by storage format.  Two graphs of the same size: the R-MAT graph of cfg2 (hubs) and a
    uniform random graph with the same number of nodes and edges (even rows, where ELLPACK is at home)."""
    dev = "cuda"
    ev = HipEvents(torch.cuda.current_stream().cuda_stream)
    w = synth.config2(scale=args.scale or 17)
    rng = synth.substream(0, "graph", 99)
    pairs = (w.rowptr[-1] // 2)
    er_rowptr, er_col = synth.erdos_renyi_gnm(w.n, int(pairs), rng)
    out = {}

    def timed(fn):
        return float(np.mean(ev.blocks(fn, 5, 5, warm=3)))

    for gname, (rowptr, col) in (("rmat", (w.rowptr, w.col)), ("uniform", (er_rowptr, er_col))):
        g = graphs.gcn_graph(rowptr, col, dev, symmetric=True)
        n, q = g.n, g.nnz
        rest_ptr = torch.empty(n + 1, dtype=torch.int32, device=dev)
        ws = B.alloc(B.gnn_hyb_workspace_bytes(n))
        _, longest = B.gnn_csr_hyb_count(n, g.rowptr, 0, rest_ptr, ws)
        res = {"n": n, "nnz": q, "longest_row": longest, "ell_padding": round(1 - q / (n * longest), 4), "ms": {}}
        forms = {}
        for t in sorted({16, 32, longest}):
            rest, _ = B.gnn_csr_hyb_count(n, g.rowptr, t, rest_ptr, ws)
            h = dict(t=t, rest=rest,
                     ell_col=torch.empty((t, n), dtype=torch.int32, device=dev),
                     ell_val=torch.empty((t, n), dtype=torch.float32, device=dev),
                     row=torch.empty(max(rest, 1), dtype=torch.int32, device=dev),
                     col=torch.empty(max(rest, 1), dtype=torch.int32, device=dev),
                     val=torch.empty(max(rest, 1), dtype=torch.float32, device=dev))
            B.gnn_csr_to_hyb(n, t, g.rowptr, g.col, g.val, rest_ptr, h["ell_col"], h["ell_val"], h["row"], h["col"],
                             h["val"])
            forms["ellpack" if t == longest else f"hybrid_t{t}"] = h
        for f in (16, 64, 128):
            Bm = torch.randn((n, f), dtype=torch.float32, device=dev)
            C = torch.empty((n, f), dtype=torch.float32, device=dev)
            sws = B.alloc(B.gnn_spmm_workspace_bytes(n, q, f))
            ms = {"csr": timed(lambda: B.gnn_spmm_csr(n, q, g.rowptr, g.col, g.val, g.erow, Bm, f, C, None, False, sws)),
                  "coo": timed(lambda: B.gnn_spmm_coo(n, q, g.erow, g.col, g.val, Bm, f, C))}
            ref = C.clone()
            B.gnn_spmm_csr(n, q, g.rowptr, g.col, g.val, g.erow, Bm, f, ref, None, False, sws)
            for name, h in forms.items():
                ms[name] = timed(lambda: B.gnn_spmm_hyb(n, h["t"], h["ell_col"], h["ell_val"], h["rest"], h["row"],
                                                        h["col"], h["val"], Bm, f, C))
                err = float((C - ref).abs().max())
                assert err < 1e-3, (name, f, err)
            res["ms"][str(f)] = {k: round(v, 4) for k, v in ms.items()}
            print(f"{gname} f={f}: {res['ms'][str(f)]}", file=sys.stderr)
        res["rest_entries"] = {k: int(h["rest"]) for k, h in forms.items()}
        out[gname] = res
        del forms
    print(json.dumps({"format_study": out}))


def row_order_study(args, torch, B, graphs, synth):
    """SpMM on P A' for row permutations P: the kernel walks an explicit entry list, so the storage order of
    the rows decides which rows share a block, an XCD and a moment in time, while B and the column indices stay
    as they are.  Every order launches gnn_spmm_csr 3 + 5 times (the counters of a rocprofv3 --pmc run of this
    command can be matched to the orders by dispatch sequence)."""
    w = synth.config2() if args.workload == "cfg2" else synth.config5()
    f = 128 if args.workload == "cfg2" else 64
    g = graphs.gcn_graph(w.rowptr, w.col, "cuda")
    n, q = g.n, g.nnz
    rp, col, val = g.rowptr.cpu().numpy().astype(np.int64), g.col.cpu().numpy(), g.val.cpu().numpy()
    deg = np.diff(rp)
    ev = HipEvents(torch.cuda.current_stream().cuda_stream)
    Bm = torch.randn((n, f), device="cuda")
    C = torch.empty((n, f), device="cuda")
    ws = B.alloc(B.gnn_spmm_workspace_bytes(n, q, f))

    def order_of(name):
        if name == "as given":
            return None
        if name == "by degree, hubs first":
            return np.argsort(-deg, kind="stable")
        if name == "by smallest neighbour":
            return np.argsort(col[rp[:-1]], kind="stable")
        if name == "by min-hash of the neighbour set":
            hsh = (col.astype(np.uint64) * np.uint64(2654435761)) % np.uint64(1 << 32)
            return np.argsort(np.minimum.reduceat(hsh, rp[:-1]), kind="stable")
        return np.random.default_rng(1).permutation(n)

    out = {}
    for name in ("as given", "by degree, hubs first", "by smallest neighbour", "by min-hash of the neighbour set", "random"):
        perm = order_of(name)
        if perm is None:
            d_rp, d_col, d_val, d_erow = g.rowptr, g.col, g.val, g.erow
        else:
            lens = deg[perm]
            nrp = np.zeros(n + 1, np.int64)
            np.cumsum(lens, out=nrp[1:])
            idx = np.repeat(rp[perm] - nrp[:-1], lens) + np.arange(q)
            d_rp = torch.from_numpy(nrp.astype(np.int32)).cuda()
            d_col, d_val = torch.from_numpy(col[idx]).cuda(), torch.from_numpy(val[idx]).cuda()
            d_erow = torch.from_numpy(np.repeat(np.arange(n, dtype=np.int32), lens)).cuda()
            del idx
        call = lambda: B.gnn_spmm_csr(n, q, d_rp, d_col, d_val, d_erow, Bm, f, C, None, False, ws)
        for _ in range(3):
            call()
        out[name] = round(ev.time_ms(call, 5), 5)
        print(f"{name}: {out[name]} ms", file=sys.stderr)
    print(json.dumps({"row_order_study": {"workload": w.name, "n": n, "nnz": q, "f": f, "launches_per_order": 8, "ms": out}}))


def main():
    args = parse()
    if args.gpus != 1:
        sys.exit("bench.py: this build runs on ONE GPU; there is no multi-GPU path (--gpus must be 1)")

    import torch
    if not torch.cuda.is_available():
        sys.exit("bench.py: no GPU visible")
    if args.copy_reference:
        x = torch.empty(64 << 20, dtype=torch.float32, device="cuda").normal_()
        y = torch.empty_like(x)
        for _ in range(3):
            y.copy_(x)
        torch.cuda.synchronize()
        print(json.dumps({"copy_reference": {"bytes_read": x.numel() * 4, "bytes_written": x.numel() * 4, "copies": 3}}))
        return
    from paper_2308_12093_amd import binding as B, graphs, synth

    if args.format_study:
        return format_study(args, torch, B, graphs, synth)
    if args.row_order_study:
        return row_order_study(args, torch, B, graphs, synth)
    oracle = None
    if not args.no_cpu_baseline:
        import oracle
    have = {}
    if args.workload == "cfg4":
        res = bench_gat(args, torch, B, graphs, synth, oracle)
    elif args.workload == "cfg3":
        res = bench_gcn_network(args, torch, B, graphs, synth, oracle)
    elif args.workload == "gatnet":
        res = bench_gat_network(args, torch, B, graphs, synth, oracle)
    else:
        w, run, res = bench_gcn_single(args, torch, B, graphs, synth, oracle)
        have[args.workload] = run
    default_run = (args.workload == "cfg5" and args.scheme == "auto" and args.layer == "gcn" and args.aggregator == "gcn"
                   and args.scale is None and not args.no_input_grad and not args.constant_input)
    if default_run and not args.no_summary:
        res["config"]["all_configs"] = all_configs_summary(args, torch, B, graphs, synth, have)

    out = {"metric": res["metric"], "value": res["value"], "unit": "edge*feat/s", "n_gpus": 1, "steps": args.steps,
           "warmup": args.warmup, "ms_per_step": res["ms_per_step"], "higher_is_better": True, "scaling": "weak",
           "vs_baseline": None, "dtype": "f32", "data": "synthetic", "config": res["config"],
           "roofline": res["roofline"], "cpu_baseline": res["cpu_baseline"]}
    print(json.dumps(out))


if __name__ == "__main__":
    main()
