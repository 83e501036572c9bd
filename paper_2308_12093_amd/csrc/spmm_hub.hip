// Sparse-dense product of a large graph with hubs: long rows in pieces, ordered by where their columns lie.
//
// What bounds the SpMM on a large graph are the lines that miss the L2s: a compute unit has at most 64 lines under way
// (TCP_TCC_READ_REQ_LATENCY over cycles and CUs is 64 in this kernel), so its rate is 64 lines over their mean latency, and
// a line from beyond the L2 takes three to four times as long as one in it.  Each of the eight L2s (4 MB) meets the columns
// of its share of the rows in no order and fetches nearly every gathered row anew (2^20 nodes, f = 100: 19.6 GB of 25 GB
// requested).  But the columns of a row ascend, and where a graph has hubs most entries lie in long rows (in rows of 128
// and more: 78 % of the entries there, 70 % at 2^22 nodes).  So long rows are cut into pieces, and the pieces of all rows
// are processed in the order of their position inside the row, XCD x the x-th eighth of that order: it gathers from about
// an eighth of the dense operand, walked once from beginning to end in step with all other long rows.  Lines fetched at
// f = 100: 19.6 -> 12.7 GB; 2960 -> 2330 us.  f = 64 at 2^22 nodes: 4300 -> 3630 us.
// Nothing but the time depends on the order of the columns.
//
//   hub_count_kernel    looks at kSamples rows: is a third of the entries in long ones?  If not, all that follow return
//                       at once and spmm_seg_kernel runs (a uniform random graph gains nothing here and pays these
//                       launches, 20 us).  Else, per block of rows: pieces by position, short rows by length
//   (scan)              counts -> places
//   hub_scatter_kernel  writes the ordered list of pieces and short rows, and the list of long rows
//   hub_gather_kernel   one group of lanes per item: a partial row for a piece, a row of C for a short row
//   hub_reduce          (in spmm_fixup_kernel) one wavefront per long row: its partials in a fixed order, bias,
//                       activation
//
// Shorter pieces, or pieces cut at columns instead of positions, miss less often (11.4 instead of 12.7 GB) and are no
// faster, within 2 %; with the gathers of the next sixteen entries under way while sixteen are folded it is 4 % slower: the
// lines under way are what is short.
#include "spmm_hub.h"

#include <type_traits>

namespace gnn {
namespace {

constexpr int kRowsPerBlock = 1024;
constexpr int kShortClasses = 6;
// per block of rows: pieces by position, short rows by length, then the number of long rows and of all their pieces
constexpr int kHubLists = kHubBuckets + kShortClasses + 2;
constexpr int kGrab = 4;                   // items a group takes at a time: 2 and 8 are 1 - 4 % slower
constexpr int kQueueStride = 64;           // counters in lines of their own: in one line each of them waits for all others
constexpr int kBlocksPerCu = 5;            // by registers
constexpr int kSamples = 1024;

// Pieces of a row of d >= kHubRow entries.
__device__ __forceinline__ int hub_pieces(int d) { return min(d / kHubPiece, kHubMaxPieces); }

// First entry of piece p of np: equal shares, moved to the next multiple of sixteen entries so that the sixteen
// columns and weights read at a time lie in one line each.
__device__ __forceinline__ int hub_begin(int a, int d, int p, int np) {
    if (p <= 0) return a;
    if (p >= np) return a + d;
    return min((a + (int)((int64_t)d * p / np) + 15) & -16, a + d);
}

// Rows with fewer than kHubRow entries in classes of similar length, the longest first: the groups of a wavefront then
// have about as much to do as each other, and what is left for the end is short.
__device__ __forceinline__ int short_class(int d) {
    return d > 64 ? 0 : d > 32 ? 1 : d > 16 ? 2 : d > 8 ? 3 : d > 1 ? 4 : 5;
}

// Are a third of the entries in long rows?  Every block looks at the same kSamples rows and comes to the same answer.
__device__ __forceinline__ bool many_in_long_rows(int n, const int32_t *__restrict__ rowptr, unsigned long long *s_sum) {
    if (threadIdx.x < 2) s_sum[threadIdx.x] = 0;
    __syncthreads();
    unsigned long long all = 0, in_long = 0;
#pragma unroll
    for (int i = 0; i < kSamples / 256; ++i) {
        const int r = (int)((int64_t)n * (i * 256 + threadIdx.x) / kSamples);
        const int d = rowptr[r + 1] - rowptr[r];
        all += d;
        in_long += d >= kHubRow ? d : 0;
    }
    for (int m = 1; m < kWave; m <<= 1) {
        all += __shfl_xor(all, m, kWave);
        in_long += __shfl_xor(in_long, m, kWave);
    }
    if (threadIdx.x % kWave == 0) {
        atomicAdd(&s_sum[0], all);
        atomicAdd(&s_sum[1], in_long);
    }
    __syncthreads();
    return 3 * s_sum[1] >= s_sum[0];
}

// Per block of rows: the long ones go to s_hub (first entry, length, row, pieces before it; in no order), their number
// and that of their pieces to *s_n; `short_row(class, row, start, length)` sees the others.  Ends with a barrier.
constexpr int kCountBits = 11;                             // kRowsPerBlock long rows at most, of kHubMaxPieces pieces
static_assert(kRowsPerBlock < 1 << kCountBits && (int64_t)kRowsPerBlock * kHubMaxPieces < (int64_t)1 << (32 - kCountBits),
              "both counts in one word");
template <typename F>
__device__ __forceinline__ void block_rows(int n, int nnz, const int32_t *__restrict__ rowptr, int4 *s_hub, uint32_t *s_n,
                                           F short_row) {
    if (threadIdx.x == 0) *s_n = 0;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kRowsPerBlock / 256; ++i) {
        const long r = (long)blockIdx.x * kRowsPerBlock + i * 256 + threadIdx.x;
        const int a = r < n ? rowptr[r] : 0, d = r < n ? min(rowptr[r + 1], nnz) - a : 0;
        if (d >= kHubRow) {
            const uint32_t at = atomicAdd(s_n, (uint32_t)hub_pieces(d) << kCountBits | 1u);
            s_hub[at & ((1 << kCountBits) - 1)] = make_int4(a, d, (int)r, (int)(at >> kCountBits));
        }
        short_row(r >= n || d >= kHubRow ? -1 : short_class(d), (int)r, a, d);
    }
    __syncthreads();
}

__device__ __forceinline__ int hub_bucket(int p, int np) { return (int)((2u * p + 1) * (unsigned)kHubBuckets / (2u * np)); }

// The last of s_hub[0 .. hubs) with no more than t pieces before it.
__device__ __forceinline__ int hub_of_piece(const int4 *s_hub, int hubs, int t) {
    int lo = 0, hi = hubs - 1;
    while (lo < hi) {
        const int m = (lo + hi + 1) / 2;
        if (s_hub[m].w <= t) lo = m;
        else hi = m - 1;
    }
    return lo;
}

__global__ void __launch_bounds__(256)
hub_count_kernel(int n, int nnz, const int32_t *__restrict__ rowptr, int32_t *__restrict__ use, int32_t *__restrict__ counts,
                 int32_t *__restrict__ queues, int nqueues) {
    __shared__ int4 s_hub[kRowsPerBlock];
    __shared__ int32_t s_hist[kHubLists];
    __shared__ unsigned long long s_sum[2];
    __shared__ uint32_t s_n;
    const bool go = many_in_long_rows(n, rowptr, s_sum);
    if (blockIdx.x == 0 && threadIdx.x == 0) *use = go;
    if (!go) return;
    if (blockIdx.x == 0)
        for (int i = threadIdx.x; i < nqueues; i += 256) queues[i] = 0;
    if (threadIdx.x < kHubLists) s_hist[threadIdx.x] = 0;
    const int lane = threadIdx.x % kWave;
    block_rows(n, nnz, rowptr, s_hub, &s_n, [&](int cls, int, int, int) {
#pragma unroll
        for (int c = 0; c < kShortClasses; ++c) {
            const unsigned long long m = __ballot(cls == c);
            if (lane == 0 && m) atomicAdd(&s_hist[kHubBuckets + c], __popcll(m));
        }
    });
    const int hubs = s_n & ((1 << kCountBits) - 1), total = s_n >> kCountBits;
    for (int t = threadIdx.x; t < total; t += 256) {
        const int4 h = s_hub[hub_of_piece(s_hub, hubs, t)];
        atomicAdd(&s_hist[hub_bucket(t - h.w, hub_pieces(h.y))], 1);
    }
    if (threadIdx.x == 0) {
        s_hist[kHubLists - 2] = hubs;
        s_hist[kHubLists - 1] = total;
    }
    __syncthreads();
    if (threadIdx.x < kHubLists) counts[(size_t)threadIdx.x * gridDim.x + blockIdx.x] = s_hist[threadIdx.x];
}

__global__ void __launch_bounds__(256)
hub_scatter_kernel(int n, int nnz, const int32_t *__restrict__ rowptr, const int32_t *__restrict__ use,
                   const int32_t *__restrict__ place, int4 *__restrict__ items, int4 *__restrict__ rows) {
    __shared__ int4 s_hub[kRowsPerBlock];
    __shared__ int32_t s_place[kHubLists];
    __shared__ uint32_t s_n;
    if (!*use) return;
    if (threadIdx.x < kHubLists) {
        const int32_t *p = place + (size_t)threadIdx.x * gridDim.x;
        // the last two lists are numbered from zero
        s_place[threadIdx.x] = p[blockIdx.x] - (threadIdx.x >= kHubLists - 2 ? p[0] : 0);
    }
    const int lane = threadIdx.x % kWave;
    block_rows(n, nnz, rowptr, s_hub, &s_n, [&](int cls, int row, int a, int d) {
#pragma unroll
        for (int c = 0; c < kShortClasses; ++c) {
            const unsigned long long m = __ballot(cls == c);
            if (!m) continue;
            int at = 0;
            if (lane == 0) at = atomicAdd(&s_place[kHubBuckets + c], __popcll(m));
            at = __builtin_amdgcn_readfirstlane(at) + __popcll(m & ((1ull << lane) - 1));
            if (cls == c) items[at] = make_int4(a, d, row, 0);
        }
    });
    const int hubs = s_n & ((1 << kCountBits) - 1), total = s_n >> kCountBits;
    const int row0 = s_place[kHubLists - 2], base = s_place[kHubLists - 1];
    for (int i = threadIdx.x; i < hubs; i += 256)
        rows[row0 + i] = make_int4(s_hub[i].z, base + s_hub[i].w, hub_pieces(s_hub[i].y), 0);
    for (int t = threadIdx.x; t < total; t += 256) {
        const int4 h = s_hub[hub_of_piece(s_hub, hubs, t)];
        const int np = hub_pieces(h.y), p = t - h.w;
        const int x = hub_begin(h.x, h.y, p, np), end = hub_begin(h.x, h.y, p + 1, np);
        items[atomicAdd(&s_place[hub_bucket(p, np)], 1)] = make_int4(x, end - x, base + t, 0);
    }
}

// Lane l of every four holds entries 4 l ... 4 l + 3 of the batch of sixteen in x, y, z, w; every lane gets entry u.
template <int Q> __device__ __forceinline__ int quad_lane(int v) { return __builtin_amdgcn_mov_dpp(v, Q * 0x55, 0xf, 0xf, true); }
struct Entries {
    int32_t c[4], v[4];    // columns, and weights as bits
};

// Entries x ... x + 3, those past the end of the list read as any other.  The list has at least four.
__device__ __forceinline__ void load_four(const int32_t *__restrict__ p, unsigned x, unsigned nnz, int32_t (&out)[4]) {
    const unsigned at = min(x, nnz - 4);
    const int4u q = *reinterpret_cast<const int4u *>(p + at);
    int32_t a = q.x, b = q.y, c = q.z;
    const int32_t d = q.w;
    if (at != x) {                                         // the last few of the list
        a = x == at + 1 ? b : x == at + 2 ? c : d;
        b = x == at + 1 ? c : d;
        c = d;
    }
    out[0] = a; out[1] = b; out[2] = c; out[3] = d;
}

__device__ __forceinline__ void load_batch(Entries &e, const int32_t *__restrict__ col, const EdgeWeights &w, unsigned x,
                                           unsigned nnz) {
    load_four(col, x, nnz, e.c);
    if (w.val && w.perm) {
        int32_t p[4];
        load_four(w.perm, x, nnz, p);
#pragma unroll
        for (int j = 0; j < 4; ++j) e.v[j] = __float_as_int(w.val[p[j]]);
    } else if (w.val) {
        load_four(reinterpret_cast<const int32_t *>(w.val), x, nnz, e.v);
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) e.v[j] = __float_as_int(1.f);
    }
}

// One group of LPE lanes per item, four features a lane (wider rows take blockIdx.y).  The wavefronts of an XCD take the
// pieces of its eighth in order, kGrab per group at a time, from a counter: wavefronts do not advance evenly, and with a
// fixed share each they drift apart until the L2 serves a much wider range of columns than the list asks for at any one
// place.  Counter 2 x is the x-th eighth of the pieces, 2 x + 1 every eighth share of the short rows.
template <int LPE, bool WIDE, bool RAGGED>
__global__ void __launch_bounds__(256, kBlocksPerCu)
hub_gather_kernel(int nnz, int nblk, int f, int ld, const int32_t *__restrict__ use,
                  const int32_t *__restrict__ place, int32_t *__restrict__ queues,
                  const int4 *__restrict__ items, const int32_t *__restrict__ col, EdgeWeights w,
                  const float *__restrict__ B, float *__restrict__ part, float *__restrict__ C,
                  const float *__restrict__ bias, int act) {
    constexpr int GW = kWave / LPE, U = 8;
    __shared__ float4 s_bias[LPE];
    if (!*use) return;
    const int lane = threadIdx.x % kWave, l = lane % LPE, grp = lane / LPE;
    const int foff = (blockIdx.y * LPE + l) * 4;
    if (threadIdx.x < LPE) {                               // x + -0 is x
        float b[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) b[j] = bias && foff + j < f ? bias[foff + j] : -0.f;
        s_bias[l] = make_float4(b[0], b[1], b[2], b[3]);
    }
    __syncthreads();
    const unsigned pieces = place[(size_t)kHubBuckets * nblk], all = place[(size_t)(kHubBuckets + kShortClasses) * nblk];
    const unsigned xcd = blockIdx.x % 8;
    const bool ok = foff < ld;
    const float *src = B + (ok ? foff : 0);
    for (int turn = 0; turn < 2; ++turn) {
        int32_t *queue = queues + (16 * blockIdx.y + 2 * xcd + turn) * kQueueStride;
        const unsigned lo = turn ? pieces + xcd * (GW * kGrab) : (unsigned)((uint64_t)pieces * xcd / 8);
        const unsigned hi = turn ? all : (unsigned)((uint64_t)pieces * (xcd + 1) / 8);
        const unsigned stride = turn ? 8 * GW * kGrab : GW * kGrab;
        if (lo >= hi) continue;
        auto grab = [&]() {
            int c = 0;
            if (lane == 0) c = atomicAdd(queue, 1);
            return c;
        };
        unsigned base = lo + __builtin_amdgcn_readfirstlane(grab()) * stride;
        if (base >= hi) continue;
        int ahead = grab(), k = 0;
        int4 p = items[min(base + grp, hi - 1)];
        if (base + grp >= hi) p.y = -1;
        Entries e;
        load_batch(e, col, w, p.x + 4 * (l % 4), nnz);
        while (base < hi) {
            if (++k == kGrab) {
                k = 0;
                base = lo + __builtin_amdgcn_readfirstlane(ahead) * stride;
                ahead = grab();
            }
            const unsigned i = base + k * GW + grp;
            int4 pnext = items[min(i, hi - 1)];
            if (i >= hi) pnext.y = -1;
            float acc[4] = {0.f, 0.f, 0.f, 0.f};
            int x = 0;
            do {
                const int32_t nc[4] = {e.c[0], e.c[1], e.c[2], e.c[3]}, nv[4] = {e.v[0], e.v[1], e.v[2], e.v[3]};
                // the next sixteen of this item, or the first of the next one
                load_batch(e, col, w, (x + 16 < p.y ? p.x + x + 16 : pnext.x) + 4 * (l % 4), nnz);
                auto batch = [&](auto lower, auto whole, int rem) {
                    constexpr int Q = lower.value / 4;
                    float4 b[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int c = u < 4 ? quad_lane<Q>(nc[u % 4]) : quad_lane<Q + 1>(nc[u % 4]);
                        b[u] = make_float4(0.f, 0.f, 0.f, 0.f);
                        if (ok && (whole.value || u < rem)) {
                            if constexpr (WIDE) b[u] = *reinterpret_cast<const float4 *>(src + (size_t)c * ld);
                            else b[u] = *reinterpret_cast<const float4 *>(reinterpret_cast<const char *>(src) +
                                                                          __umul24(c, ld * 4));
                        }
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const float v = __int_as_float(u < 4 ? quad_lane<Q>(nv[u % 4]) : quad_lane<Q + 1>(nv[u % 4]));
                        if (whole.value || u < rem) {
                            acc[0] = fmaf(v, b[u].x, acc[0]);
                            acc[1] = fmaf(v, b[u].y, acc[1]);
                            acc[2] = fmaf(v, b[u].z, acc[2]);
                            acc[3] = fmaf(v, b[u].w, acc[3]);
                        }
                    }
                };
                constexpr std::integral_constant<int, 0> lower{};
                constexpr std::integral_constant<int, U> upper{};
                const int rem = p.y - x;
                if (rem >= U) batch(lower, std::true_type{}, U);
                else batch(lower, std::false_type{}, rem);
                if (rem >= 2 * U) batch(upper, std::true_type{}, U);
                else if (rem > U) batch(upper, std::false_type{}, rem - U);
                x += 16;
            } while (x < p.y);
            if (ok && p.y >= 0) {
                if (turn) {                                // a whole row
                    const float4 bv = s_bias[l];
                    const float o[4] = {activate(acc[0] + bv.x, act), activate(acc[1] + bv.y, act),
                                        activate(acc[2] + bv.z, act), activate(acc[3] + bv.w, act)};
                    float *to = C + (size_t)p.z * f + foff;
                    if (RAGGED && foff + 4 > f) {
#pragma unroll
                        for (int j = 0; j < 3; ++j)
                            if (foff + j < f) to[j] = o[j];
                    } else {
                        const float4u q = {o[0], o[1], o[2], o[3]};
                        if constexpr (RAGGED) *reinterpret_cast<float4u *>(to) = q;
                        else *reinterpret_cast<float4 *>(to) = make_float4(o[0], o[1], o[2], o[3]);
                    }
                } else {
                    *reinterpret_cast<float4 *>(part + (size_t)p.z * ld + foff) = make_float4(acc[0], acc[1], acc[2], acc[3]);
                }
            }
            p = pnext;
        }
    }
}

long hub_blocks(int64_t n) { return ceil_div(n, kRowsPerBlock); }

struct HubBuffers {
    int32_t *use, *place, *queues, *scan;
    int4 *items, *rows;
    float *part;
    int nqueues;
    size_t bytes;
};

HubBuffers carve(void *base, int64_t n, int64_t nnz, int ld) {
    Carver c(base);
    HubBuffers b;
    b.nqueues = 16 * kQueueStride * (int)ceil_div(ld, 4 * kWave);
    b.use = c.take<int32_t>(1);
    b.place = c.take<int32_t>(kHubLists * hub_blocks(n));
    b.queues = c.take<int32_t>(b.nqueues);
    b.scan = reinterpret_cast<int32_t *>(c.take<char>(scan_workspace_bytes(kHubLists * hub_blocks(n))));
    b.items = c.take<int4>(nnz / kHubPiece + n);           // a row of d entries has at most d / kHubPiece pieces
    b.rows = c.take<int4>(nnz / kHubRow);
    b.part = c.take<float>((size_t)(nnz / kHubPiece) * ld);
    b.bytes = c.off;
    return b;
}

int pow2_at_least(int x) {
    int p = 1;
    while (p < x) p <<= 1;
    return p;
}

}  // namespace

size_t hub_workspace_bytes(int64_t n, int64_t nnz, int ld) { return carve(nullptr, n, nnz, ld).bytes; }

gnn_status_t hub_spmm_launch(int n, int nnz, const int32_t *rowptr, const int32_t *col, EdgeWeights w, const float *B,
                             int f, int ld, float *C, const float *bias, int act, void *workspace, hipStream_t st,
                             HubReduce *rest) {
    const HubBuffers b = carve(workspace, n, nnz, ld);
    const int nblk = (int)hub_blocks(n);
    hipLaunchKernelGGL(hub_count_kernel, dim3(nblk), dim3(256), 0, st, n, nnz, rowptr, b.use, b.place, b.queues, b.nqueues);
    GNN_TRY(launch_status());
    GNN_TRY(exclusive_scan_launch(b.place, (long)kHubLists * nblk, b.scan, st));
    hipLaunchKernelGGL(hub_scatter_kernel, dim3(nblk), dim3(256), 0, st, n, nnz, rowptr, b.use, b.place, b.items, b.rows);
    GNN_TRY(launch_status());
    int lpe = pow2_at_least(ld / 4);
    if (lpe < 4) lpe = 4;
    if (lpe > kWave) lpe = kWave;
    const dim3 grid(kBlocksPerCu * 256, (unsigned)ceil_div(ld, 4 * lpe));
    // offsets of 32 bits from a 24-bit multiplication, where they reach
    const bool wide = n >= (1 << 24) || ld >= (1 << 22) || (int64_t)n * ld * 4 >= ((int64_t)1 << 32), ragged = f != ld;
#define HUB_LAUNCH(LPE_, WIDE_, RAGGED_)                                                                                   \
    if (lpe == LPE_ && wide == WIDE_ && ragged == RAGGED_)                                                                 \
        hipLaunchKernelGGL((hub_gather_kernel<LPE_, WIDE_, RAGGED_>), grid, dim3(256), 0, st, nnz, nblk, f, ld, b.use,     \
                           b.place, b.queues, b.items, col, w, B, b.part, C, bias, act);
#define HUB_CASE(LPE_)                                                                                                     \
    HUB_LAUNCH(LPE_, false, false) HUB_LAUNCH(LPE_, false, true) HUB_LAUNCH(LPE_, true, false) HUB_LAUNCH(LPE_, true, true)
    HUB_CASE(4) HUB_CASE(8) HUB_CASE(16) HUB_CASE(32) HUB_CASE(64)
    GNN_TRY(launch_status());
    *rest = HubReduce{b.use, b.place + (size_t)(kHubLists - 2) * nblk, b.rows, b.part, nblk, ld, lpe};
    return GNN_OK;
}

}  // namespace gnn
