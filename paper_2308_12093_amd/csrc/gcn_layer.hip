// GCN layer forward / backward as sequences of SpMM and GEMM launches, in the order
// the plan chose (Sec. 3.1; Fig. "Two schemes of computing the forward pass", Fig.
// "Alternative schemes of computing the backward pass", Fig. "GCN computation scheme
// using caching").  Host code: it only carves the workspace and enqueues kernels.
// The GraphSAGE layer (Sec. 3.1 "Generalizability") is the same chain plus a dense
// self term, added by the GEMM that follows or precedes the SpMM.
#include "plan.h"

namespace gnn {

namespace {

struct SparseView {            // a CSR view of A' or of A'^T
    const int32_t *ptr, *idx, *eidx;
    EdgeWeights w;
};

SparseView forward_view(const gnn_graph_t &g, int f) {
    return SparseView{g.csr_rowptr, g.csr_col, g.csr_erow, EdgeWeights{g.csr_val, nullptr, 1, f}};
}

// A'^T as a CSR matrix is the CSC arrays of A'; a symmetric A' is its own transpose.
SparseView transposed_view(const gnn_graph_t &g, int f) {
    if (g.symmetric) return forward_view(g, f);
    if (g.csc_val) return SparseView{g.csc_colptr, g.csc_row, g.csc_ecol, EdgeWeights{g.csc_val, nullptr, 1, f}};
    return SparseView{g.csc_colptr, g.csc_row, g.csc_ecol, EdgeWeights{g.csr_val, g.csc_perm, 1, f}};
}

gnn_status_t spmm(const gnn_graph_t &g, const SparseView &v, const float *B, int f, float *C, const float *bias,
                  int relu, void *ws, hipStream_t st, bool pieces = true) {
    return spmm_launch(g.n, g.nnz, v.ptr, v.idx, v.eidx, v.w, B, g.n, f, C, bias, relu, ws, st, pieces);
}

// Layers whose sums before a ReLU keep the order they have had: those with dX, where a pre-activation that falls on the other
// side of zero changes a row of dX by its full size.  That is a choice, not a bound: the other sums are the more exact ones
// (see relu_flags).  Outputs of few elements take the other sums as well: one pre-activation in 10^7 changes sides.
constexpr int64_t kFewSigns = 1 << 17;
bool sums_decide_signs(const gnn_plan_desc_t &d) {
    return d.fuse_relu && d.need_input_grad && (int64_t)d.n * d.f_out > kFewSigns;
}

// Flags of the product before a fused ReLU.  Without dX it may run on split parts, whose sums lie closer to 64 bits than those
// of the fp32 instruction, so that fewer pre-activations fall on the wrong side of zero.  fp32 instruction / split parts, a
// forward pass in us, relative error of Y, wrong signs in three runs:
//   2^17 nodes, 128 -> 512 240 / 195, 1.5e-7 / 5.9e-8, 4 / 2; 512 -> 128 289 / 254, 3.0e-7 / 1.1e-7, 3 / 2;
//   2^19, 100 -> 256 508 / 419, 1.4e-7 / 5.9e-8, 15 / 5; 65536, 128 -> 512 121 / 95, 1.5e-7 / 5.9e-8, 4 / 1;
//   50021, 100 -> 256 76 / 54, 1.3e-7 / 5.7e-8.
// A wrong sign puts one term too many or too few into the sums of dW and db, 1e-4 of them at these sizes (else 2.5e-8).
// Few outputs, four wavefronts to a tile: 3001 nodes, 203 -> 7, forward, 23.7 / 19.2 us, 1.4e-7 / 8.6e-8.
int relu_flags(const gnn_plan_desc_t &d, int with_relu) {
    return !d.fuse_relu ? 0 : sums_decide_signs(d) ? with_relu : with_relu | kActAnySign;
}

bool overlap(const float *a, size_t count_a, const float *b, size_t count_b) {
    const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
    return a && b && x < y + count_b * sizeof(float) && y < x + count_a * sizeof(float);
}

// Gradient through the fused ReLU, G = dY .* [Y > 0], and through the bias, db = G^T 1.
// Split-propagate scheme: G is read by the weight-gradient products, which mask dY as they load it and add up db on the
// side, and with dX by the products with the weights, which take the mask as bits from the first of those: G is never
// written, nothing but products reads dY or Y (2^17 nodes, 128 -> 512, a step: 930 -> 828 us; GraphSAGE 128 -> 128:
// 588 -> 573).  One pass makes G and db where those products run on a kernel that takes no bits, where dY is read again after
// dX was written and shares memory with it, in the fused-propagate scheme, whose gather would fetch Y beside dY, and with dX
// where the weight gradients would read Y too often (`pass_us`): products / pass, us of a backward pass without aggregation,
// GraphSAGE 58450 x 403 -> 293 without bias 1207 / 1030, 131072 x 512 -> 256 with bias 1866 / 1725, GCN 58450 x 403 -> 293
// without 649 / 549, 124552 x 480 -> 16 without 259 / 235; the other way round GCN 307451 x 43 -> 45 with bias 145 / 206,
// 131072 x 64 -> 16 48 / 63.
struct BiasAndMask {
    const float *G = nullptr, *mask_y = nullptr;       // G, or dY and what the products mask it by
    GemmExtras side{}, plain{}, masked{};              // for the first weight-gradient product, others, those with the weights

    // W, W2: the weights behind G; dX: where the input gradient goes if dY is read once more behind it, or NULL
    gnn_status_t start(const Plan &p, const float *W, const float *W2, const float *Y, const float *dY, const float *dX,
                       float *db, Carver &ws, hipStream_t st) {
        const gnn_plan_desc_t &d = p.desc;
        const int n = d.n, m = d.f_in, k = d.f_out;
        const bool dx = d.need_input_grad != 0, split = p.info.bwd == GNN_BWD_SPLIT_PROPAGATE;
        // carved either way: the layout is the plan's
        float *Gm = d.fuse_relu ? ws.take<float>((size_t)n * k) : nullptr;
        void *red = d.has_bias ? ws.take<char>(bias_gradient_bytes(p)) : nullptr;
        // what the pass takes, about: with the bias gradient two launches, and the sums in double
        const double pass_us = d.has_bias ? 5 + 2.5e-6 * n * k : 1.6e-6 * n * k;
        const double products_us = (d.layer == GNN_LAYER_SAGE ? 2 : 1) * gemm_side_us(p.tn, m, k, n);
        const bool in_products = split && (!d.fuse_relu || !dx ||
                                           (products_us < pass_us && !overlap(dX, (size_t)n * m, dY, (size_t)n * k) &&
                                            gemm_takes_bits(1, n, m, k, dY, W) && gemm_takes_bits(1, n, m, k, dY, W2)));
        G = dY;
        side.tn = plain.tn = &p.tn;
        if (in_products) {
            if (d.has_bias) {
                side.sums = db;
                side.workspace = red;
            }
            if (d.fuse_relu) {
                mask_y = Y;
                // a word holds 16 columns in the place of 16 floats
                if (dx) side.bits = reinterpret_cast<uint16_t *>(Gm);
                masked.a_bits = side.bits;
            }
            return GNN_OK;
        }
        if (d.has_bias) {
            GNN_TRY(colsum_launch(n, k, dY, db, red, st, d.fuse_relu ? Y : nullptr, kActRelu, Gm));
        } else if (d.fuse_relu) {
            GNN_TRY(activation_grad_launch((int64_t)n * k, dY, Y, Gm, kActRelu, st));
        }
        if (d.fuse_relu) G = Gm;
        return GNN_OK;
    }
};

// A weight gradient X^T G.
gnn_status_t weight_gradient(int m, int k, int n, const float *X, const float *G, float *dW, void *ws, hipStream_t st,
                             const float *mask_y, const GemmExtras &extras) {
    return gemm_launch(1, 0, m, k, n, X, G, dW, nullptr, 0, ws, st, mask_y, kActRelu, 0, nullptr, nullptr, &extras);
}

}  // namespace

size_t bias_gradient_bytes(const Plan &p) {
    const size_t pass = colsum_workspace_bytes(p.desc.n, p.desc.f_out), side = gemm_sums_bytes(p.tn, p.desc.f_out);
    return pass > side ? pass : side;
}

gnn_status_t gcn_forward(Plan &p, const gnn_graph_t &g, const float *X, const float *W, const float *b, float *Y,
                         void *cache, void *workspace, hipStream_t st) {
    const gnn_plan_desc_t &d = p.desc;
    const int n = d.n, m = d.f_in, k = d.f_out;
    const float *bias = d.has_bias ? b : nullptr;
    const bool signs = sums_decide_signs(d);
    Carver ws(workspace);
    if (p.info.order == GNN_ORDER_TRANSFORM_FIRST) {
        // T = X W, then Y = A' T (+ b, ReLU) fused into the SpMM write
        float *T = ws.take<float>((size_t)n * k);
        void *sp = ws.take<char>(spmm_workspace_bytes(n, d.nnz, k));
        void *wt = ws.take<char>(gemm_workspace_bytes(0, 0, n, k, m));
        // a width that the SpMM runs on a padded operand: the GEMM writes T in that layout, where the SpMM looks for it
        int ldt = k;
        if (float *Tp = spmm_padded_operand(sp, g.csr_erow, n, d.nnz, k, &ldt)) T = Tp;
        GNN_TRY(gemm_launch(0, 0, n, k, m, X, W, T, nullptr, relu_flags(d, kActSigns), wt, st, nullptr, 0, ldt));
        GNN_TRY(spmm(g, forward_view(g, k), T, k, Y, bias, d.fuse_relu, sp, st, !signs));
    } else {
        // P = A' X (kept in the cache slot when the plan caches it), then Y = P W (+ b, ReLU)
        const bool cached = p.info.cache == GNN_CACHE_AX;
        float *P = cached ? static_cast<float *>(cache) : ws.take<float>((size_t)n * m);
        void *sp = ws.take<char>(spmm_workspace_bytes(n, d.nnz, m));
        void *wt = ws.take<char>(gemm_workspace_bytes(0, 0, n, k, m));
        // a constant input (promised by the caller) needs its A'X only once
        if (!(cached && d.constant_input && p.cache_filled))
            GNN_TRY(spmm(g, forward_view(g, m), X, m, P, nullptr, 0, sp, st, !signs));
        GNN_TRY(gemm_launch(0, 0, n, k, m, P, W, Y, bias, relu_flags(d, kActRelu), wt, st));
        if (cached) p.cache_filled = true;
    }
    return GNN_OK;
}

gnn_status_t gcn_backward(Plan &p, const gnn_graph_t &g, const float *X, const float *W, const float *Y,
                          const float *dY, float *dW, float *db, float *dX, void *cache, void *workspace,
                          hipStream_t st) {
    const gnn_plan_desc_t &d = p.desc;
    const int n = d.n, m = d.f_in, k = d.f_out;
    const bool dx = d.need_input_grad != 0;
    Carver ws(workspace);

    BiasAndMask bm;
    GNN_TRY(bm.start(p, W, W, Y, dY, nullptr, db, ws, st));
    const float *G = bm.G;
    void *gemm_ws = ws.take<char>(backward_gemm_bytes(p, 1));   // one product at a time

    if (p.info.bwd == GNN_BWD_FUSED_PROPAGATE) {
        // H = A'^T G once; dW = X^T H; dX = H W^T
        float *H = ws.take<float>((size_t)n * k);
        void *sp = ws.take<char>(spmm_workspace_bytes(n, d.nnz, k));
        GNN_TRY(spmm(g, transposed_view(g, k), G, k, H, nullptr, 0, sp, st));
        GNN_TRY(weight_gradient(m, k, n, X, H, dW, gemm_ws, st, nullptr, bm.plain));
        if (dx) GNN_TRY(gemm_launch(0, 1, n, m, k, H, W, dX, nullptr, 0, gemm_ws, st));
    } else {
        // dW = (A'X)^T G with A'X from the cache or recomputed; dX = A'^T (G W^T)
        const bool cached = p.info.cache == GNN_CACHE_AX;
        const float *P = static_cast<const float *>(cache);
        float *Pw = cached ? nullptr : ws.take<float>((size_t)n * m);
        float *U = dx ? ws.take<float>((size_t)n * m) : nullptr;
        void *sp = ws.take<char>(spmm_workspace_bytes(n, d.nnz, m));
        if (!cached) {
            GNN_TRY(spmm(g, forward_view(g, m), X, m, Pw, nullptr, 0, sp, st));
            P = Pw;
        }
        GNN_TRY(weight_gradient(m, k, n, P, G, dW, gemm_ws, st, bm.mask_y, bm.side));
        if (dx) {
            const SparseView tv = transposed_view(g, m);
            int ldu = m;                                    // as in the forward pass: U written where the SpMM pads
            if (float *Up = spmm_padded_operand(sp, tv.eidx, n, d.nnz, m, &ldu)) U = Up;
            GNN_TRY(gemm_launch(0, 1, n, m, k, G, W, U, nullptr, 0, gemm_ws, st, nullptr, 0, ldu, nullptr, nullptr,
                                &bm.masked));
            GNN_TRY(spmm(g, tv, U, m, dX, nullptr, 0, sp, st));
        }
    }
    return GNN_OK;
}

// Y = X Ws + A' X Wn + b.  Aggregate first: one product over both operand pairs, [X | A'X] [Ws; Wn], writes Y
// once with bias and ReLU.  Transform first: the self term is a GEMM that adds to what the SpMM wrote.
gnn_status_t sage_forward(Plan &p, const gnn_graph_t &g, const float *X, const float *Ws, const float *Wn,
                          const float *b, float *Y, void *cache, void *workspace, hipStream_t st) {
    const gnn_plan_desc_t &d = p.desc;
    const int n = d.n, m = d.f_in, k = d.f_out;
    const float *bias = d.has_bias ? b : nullptr;
    const bool signs = sums_decide_signs(d);
    const int last = kActAccumulate | relu_flags(d, kActRelu);
    Carver ws(workspace);
    if (p.info.order == GNN_ORDER_TRANSFORM_FIRST) {
        float *T = ws.take<float>((size_t)n * k);
        void *sp = ws.take<char>(spmm_workspace_bytes(n, d.nnz, k));
        void *wt = ws.take<char>(2 * gemm_workspace_bytes(0, 0, n, k, m));
        int ldt = k;
        if (float *Tp = spmm_padded_operand(sp, g.csr_erow, n, d.nnz, k, &ldt)) T = Tp;
        GNN_TRY(gemm_launch(0, 0, n, k, m, X, Wn, T, nullptr, relu_flags(d, kActSigns), wt, st, nullptr, 0, ldt));
        GNN_TRY(spmm(g, forward_view(g, k), T, k, Y, nullptr, 0, sp, st, !signs));
        GNN_TRY(gemm_launch(0, 0, n, k, m, X, Ws, Y, bias, last, wt, st));
    } else {
        const bool cached = p.info.cache == GNN_CACHE_AX;
        float *P = cached ? static_cast<float *>(cache) : ws.take<float>((size_t)n * m);
        void *sp = ws.take<char>(spmm_workspace_bytes(n, d.nnz, m));
        void *wt = ws.take<char>(2 * gemm_workspace_bytes(0, 0, n, k, m));
        if (!(cached && d.constant_input && p.cache_filled))
            GNN_TRY(spmm(g, forward_view(g, m), X, m, P, nullptr, 0, sp, st, !signs));
        GNN_TRY(gemm_launch(0, 0, n, k, m, X, Ws, Y, bias, relu_flags(d, kActRelu), wt, st, nullptr, 0, 0, P, Wn));
        if (cached) p.cache_filled = true;
    }
    return GNN_OK;
}

gnn_status_t sage_backward(Plan &p, const gnn_graph_t &g, const float *X, const float *Ws, const float *Wn,
                           const float *Y, const float *dY, float *dWs, float *dWn, float *db, float *dX,
                           void *cache, void *workspace, hipStream_t st) {
    const gnn_plan_desc_t &d = p.desc;
    const int n = d.n, m = d.f_in, k = d.f_out;
    const bool dx = d.need_input_grad != 0;
    Carver ws(workspace);

    BiasAndMask bm;
    GNN_TRY(bm.start(p, Ws, Wn, Y, dY, dX, db, ws, st));
    const float *G = bm.G;
    void *gemm_ws = ws.take<char>(backward_gemm_bytes(p, 2));
    GNN_TRY(weight_gradient(m, k, n, X, G, dWs, gemm_ws, st, bm.mask_y, bm.side));

    if (p.info.bwd == GNN_BWD_FUSED_PROPAGATE) {
        // H = A'^T G once; dWn = X^T H; dX = G Ws^T + H Wn^T
        float *H = ws.take<float>((size_t)n * k);
        void *sp = ws.take<char>(spmm_workspace_bytes(n, d.nnz, k));
        GNN_TRY(spmm(g, transposed_view(g, k), G, k, H, nullptr, 0, sp, st));
        GNN_TRY(weight_gradient(m, k, n, X, H, dWn, gemm_ws, st, nullptr, bm.plain));
        if (dx) {
            GNN_TRY(gemm_launch(0, 1, n, m, k, G, Ws, dX, nullptr, 0, gemm_ws, st, nullptr, 0, 0, H, Wn));
        }
    } else {
        // dWn = (A'X)^T G with A'X from the cache or recomputed; dX = A'^T (G Wn^T) + G Ws^T
        const bool cached = p.info.cache == GNN_CACHE_AX;
        const float *P = static_cast<const float *>(cache);
        float *Pw = cached ? nullptr : ws.take<float>((size_t)n * m);
        float *U = dx ? ws.take<float>((size_t)n * m) : nullptr;
        void *sp = ws.take<char>(spmm_workspace_bytes(n, d.nnz, m));
        if (!cached) {
            GNN_TRY(spmm(g, forward_view(g, m), X, m, Pw, nullptr, 0, sp, st));
            P = Pw;
        }
        GNN_TRY(weight_gradient(m, k, n, P, G, dWn, gemm_ws, st, bm.mask_y, bm.plain));
        if (dx) {
            const SparseView tv = transposed_view(g, m);
            int ldu = m;
            if (float *Up = spmm_padded_operand(sp, tv.eidx, n, d.nnz, m, &ldu)) U = Up;
            GNN_TRY(gemm_launch(0, 1, n, m, k, G, Wn, U, nullptr, 0, gemm_ws, st, nullptr, 0, ldu, nullptr, nullptr,
                                &bm.masked));
            GNN_TRY(spmm(g, tv, U, m, dX, nullptr, 0, sp, st));
            GNN_TRY(gemm_launch(0, 1, n, m, k, G, Ws, dX, nullptr, kActAccumulate, gemm_ws, st, nullptr, 0, 0, nullptr,
                                nullptr, &bm.masked));
        }
    }
    return GNN_OK;
}

}  // namespace gnn
