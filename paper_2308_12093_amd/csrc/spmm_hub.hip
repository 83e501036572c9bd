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
// f = 100: 19.6 -> 12.7 GB; 2774 -> 2149 us.  f = 64 at 2^22 nodes: 4839 -> 3553 us.
// Nothing but the time depends on the order of the columns.
//
//   hub_count_kernel    looks at kSamples rows: is a third of the entries in long ones?  If not, all that follow return
//                       at once and spmm_seg_kernel runs (a uniform random graph gains nothing here and pays these
//                       launches).  Else, per block: pieces by position, short rows by length
//   hub_scatter_kernel  counts -> places; writes the ordered list of pieces and short rows, and the shares of long rows
//   hub_gather_kernel   one group of lanes per item: a partial row for a piece, a row of C for a short row
//   hub_reduce          (in spmm_fixup_kernel) one wavefront per 512 partial rows of a long row, in a fixed order, bias,
//                       activation
//
// A row has as many pieces as whole 64s of entries, and their partial rows have places of their own among the 64s of the
// whole list: so one thread per 64 entries finds its row and has its piece, wherever the long rows are.  Walked by rows, the
// blocks that hold the long ones were all there was to wait for (R-MAT as generated, 2^20 nodes, 53 M entries, most of the
// long rows side by side: both kernels 386 us, now 41; rows sorted by length 1300, now 50).  With at most 1024 pieces a row,
// as it once was, pieces of longer rows were long chains of sums, and few: 300 000 nodes, 36 M entries, 16 M of them in one
// row, f = 100: 8050 -> 1050 us, the segments 2210; a chain of 15 625 equal products is off by up to 2e-4 of its sum.
// Shorter pieces, or pieces cut at columns instead of positions, miss less often (11.4 instead of 12.7 GB) and are no
// faster, within 2 %; with the gathers of the next sixteen entries under way while sixteen are folded it is 4 % slower: the
// lines under way are what is short.
#include "spmm_hub.h"

#include <type_traits>

namespace gnn {
namespace {

constexpr int kHubBuckets = 64;            // positions inside a row that the order of the pieces tells apart
constexpr int kShortClasses = 6;
// per block: pieces by position, short rows by length, then the shares of long rows; padded to whole int4
constexpr int kShares = kHubBuckets + kShortClasses, kHubLists = (kShares + 1 + 3) / 4 * 4;
constexpr int kListBlocks = 512;           // blocks that make the lists: each reads the counts of all
constexpr int kListThreads = 1024;         // in each: chains of loads for every item, so as many wavefronts as there is room for
constexpr int kGrab = 4;                   // items a group takes at a time: 2 and 8 are 1 - 4 % slower
constexpr int kQueueStride = 64;           // counters in lines of their own: in one line each of them waits for all others
constexpr int kBlocksPerCu = 5;            // by registers
constexpr int kSamples = 1024;

// Pieces of a row of d >= kHubRow entries that begins at entry a: their partial rows lie at place `first` and behind.  The
// next row's begin no earlier than ceil((a + d) / 64), and entry 64 x belongs to the row whose piece has place x.
struct HubPieces {
    int first, count;
};
__device__ __forceinline__ HubPieces hub_pieces(int a, int d) {
    return HubPieces{(int)(((int64_t)a + kHubPiece - 1) / kHubPiece), d / kHubPiece};
}

// First entry of piece p of np: equal shares, moved to the next multiple of sixteen entries so that the sixteen columns and
// weights read at a time lie in one line each.
__device__ __forceinline__ int hub_begin(int a, int d, int p, int np) {
    if (p <= 0) return a;
    if (p >= np) return a + d;
    return min((a + (int)((int64_t)d * p / np) + 15) & -16, a + d);
}

// Rows with fewer than kHubRow entries in classes of similar length, the longest first: the groups of a wavefront then have
// about as much to do as each other, and what is left for the end is short.
__device__ __forceinline__ int short_class(int d) {
    return d > 64 ? 0 : d > 32 ? 1 : d > 16 ? 2 : d > 8 ? 3 : d > 1 ? 4 : 5;
}

// Are a third of the entries in long rows?  Every block looks at the same kSamples rows and comes to the same answer.
__device__ __forceinline__ bool many_in_long_rows(int n, const int32_t *__restrict__ rowptr, unsigned long long *s_sum) {
    if (threadIdx.x < 2) s_sum[threadIdx.x] = 0;
    __syncthreads();
    unsigned long long all = 0, in_long = 0;
    static_assert(kSamples == kListThreads, "one each");
    const int r = (int)((int64_t)n * threadIdx.x / kSamples), d = rowptr[r + 1] - rowptr[r];
    all += d;
    in_long += d >= kHubRow ? d : 0;
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

__device__ __forceinline__ int hub_bucket(int p, int np) { return (int)((2u * p + 1) * (unsigned)kHubBuckets / (2u * np)); }

// The last row that begins at or before entry e; 64 probes at a time by one wavefront.
__device__ __forceinline__ int row_of(const int32_t *__restrict__ rowptr, int n, int e) {
    const int lane = threadIdx.x % kWave;
    int64_t lo = 0, hi = n;                                // rowptr[lo] <= e < rowptr[hi] or hi = n
    while (hi - lo > 1) {
        const int64_t step = (hi - lo + kWave - 1) / kWave, at = lo + lane * step;
        const int before = __popcll(__ballot(at < hi && rowptr[at < hi ? at : lo] <= e));
        lo += (before > 1 ? before - 1 : 0) * step;
        hi = lo + step < hi ? lo + step : hi;
    }
    return (int)lo;
}

// Every item of this block's part of the entries and rows: piece(list, start, length, place) for the pieces, share(row,
// first, count, which) for the shares of their sums, row(list, row, start, length) for the short rows; the list is -1 if a
// lane has none.  All lanes of a wavefront call piece and row together.  s_rows: two words of LDS.
template <typename P, typename S, typename R>
__device__ __forceinline__ void block_items(int n, int nnz, const int32_t *__restrict__ rowptr, int32_t *s_rows, P piece,
                                            S share, R row) {
    const int places = (int)(((int64_t)nnz + kHubPiece - 1) / kHubPiece), per = (places + (int)gridDim.x - 1) / (int)gridDim.x;
    const int x0 = (int)min((int64_t)blockIdx.x * per, (int64_t)places), x1 = (int)min((int64_t)x0 + per, (int64_t)places);
    const int wave = threadIdx.x / kWave;
    if (wave < 2 && x0 < x1) s_rows[wave] = row_of(rowptr, n, (wave ? x1 - 1 : x0) * kHubPiece);
    __syncthreads();
    for (int xb = x0; xb < x1; xb += kListThreads) {
        const int x = xb + threadIdx.x;
        int a = 0, d = 0, r = s_rows[0];
        if (x < x1) {
            // the expanded row index has the answer in every other of its lines: 280 MB at 2^22 nodes and 138 M entries,
            // where these probes stay within a few thousand row pointers (both kernels 147 -> 92 us)
            for (int hi = s_rows[1]; r < hi;) {
                const int m = r + (hi - r + 1) / 2;
                if (rowptr[m] <= x * kHubPiece) r = m;
                else hi = m - 1;
            }
            a = rowptr[r];
            d = min(rowptr[r + 1], nnz) - a;
        }
        const HubPieces h = hub_pieces(a, d);
        const int p = x - h.first;
        const bool mine = d >= kHubRow && p >= 0 && p < h.count;
        const int begin = mine ? hub_begin(a, d, p, h.count) : 0;
        piece(mine ? hub_bucket(p, h.count) : -1, begin, mine ? hub_begin(a, d, p + 1, h.count) - begin : 0, x);
        if (mine && p % kHubShare == 0) share(r, h.first, h.count, p / kHubShare);
    }
    const int64_t rows = ((int64_t)n + gridDim.x - 1) / gridDim.x;
    const int64_t r0 = min(blockIdx.x * rows, (int64_t)n), r1 = min(r0 + rows, (int64_t)n);
    for (int64_t rb = r0; rb < r1; rb += kListThreads) {
        const int64_t r = rb + threadIdx.x;
        const int a = r < r1 ? rowptr[r] : 0, d = r < r1 ? min(rowptr[r + 1], nnz) - a : kHubRow;
        row(d >= kHubRow ? -1 : short_class(d), (int)r, a, d);
    }
}

// Adds the lanes' items to the lists they name (-1: none) and returns their places in them.  Mostly one list for all.
__device__ __forceinline__ int take_places(int32_t *lists, int list) {
    const unsigned long long any = __ballot(list >= 0);
    if (!any) return 0;
    const int one = __shfl(list, __ffsll(any) - 1, kWave);
    const unsigned long long same = __ballot(list == one);
    const int lane = threadIdx.x % kWave;
    int at = 0;
    if (same == any) {
        if (lane == 0) at = atomicAdd(&lists[one], __popcll(any));
        at = __builtin_amdgcn_readfirstlane(at) + __popcll(any & ((1ull << lane) - 1));
    } else if (list >= 0) {
        at = atomicAdd(&lists[list], 1);
    }
    return at;
}

__global__ void __launch_bounds__(kListThreads)
hub_count_kernel(int n, int nnz, const int32_t *__restrict__ rowptr, int32_t *__restrict__ use,
                 int32_t *__restrict__ counts, int32_t *__restrict__ queues, int nqueues,
                 int32_t *__restrict__ arrived, int narrived) {
    __shared__ int32_t s_hist[kHubLists], s_rows[2];
    __shared__ unsigned long long s_sum[2];
    const bool go = many_in_long_rows(n, rowptr, s_sum);
    if (blockIdx.x == 0 && threadIdx.x == 0) *use = go;
    if (!go) return;
    const int all = gridDim.x * kListThreads, me = blockIdx.x * kListThreads + threadIdx.x;
    for (int i = me; i < nqueues; i += all) queues[i] = 0;
    for (int i = me; i < narrived; i += all) arrived[i] = 0;
    if (threadIdx.x < kHubLists) s_hist[threadIdx.x] = 0;
    __syncthreads();
    block_items(
        n, nnz, rowptr, s_rows, [&](int list, int, int, int) { take_places(s_hist, list); },
        [&](int, int, int, int) { atomicAdd(&s_hist[kShares], 1); },
        [&](int cls, int, int, int) { take_places(s_hist, cls < 0 ? -1 : kHubBuckets + cls); });
    __syncthreads();
    if (threadIdx.x < kHubLists) counts[(size_t)blockIdx.x * kHubLists + threadIdx.x] = s_hist[threadIdx.x];
}

// place: the number of pieces, of pieces and short rows, and of shares
__global__ void __launch_bounds__(kListThreads)
hub_scatter_kernel(int n, int nnz, const int32_t *__restrict__ rowptr,
                   const int32_t *__restrict__ use, const int32_t *__restrict__ counts, int32_t *__restrict__ place,
                   int4 *__restrict__ items, int4 *__restrict__ tasks) {
    constexpr int QUADS = kHubLists / 4, GROUPS = kListThreads / QUADS;
    __shared__ __align__(16) int32_t s_all[GROUPS][kHubLists], s_before[GROUPS][kHubLists];
    __shared__ int32_t s_place[kHubLists], s_rows[2];
    if (!*use) return;
    const int quad = threadIdx.x % QUADS, group = threadIdx.x / QUADS;
    if (group < GROUPS) {                                  // the lists of all blocks, and of those before this one
        int4 all = make_int4(0, 0, 0, 0), before = all;
#pragma unroll 5
        for (int b = group; b < (int)gridDim.x; b += GROUPS) {
            const int4 c = reinterpret_cast<const int4 *>(counts)[(size_t)b * QUADS + quad];
            const bool earlier = b < (int)blockIdx.x;
            all.x += c.x; all.y += c.y; all.z += c.z; all.w += c.w;
            before.x += earlier ? c.x : 0; before.y += earlier ? c.y : 0;
            before.z += earlier ? c.z : 0; before.w += earlier ? c.w : 0;
        }
        *reinterpret_cast<int4 *>(&s_all[group][4 * quad]) = all;
        *reinterpret_cast<int4 *>(&s_before[group][4 * quad]) = before;
    }
    __syncthreads();
    int before = 0;
    if (threadIdx.x < kHubLists) {
        int all = 0;
        for (int g = 0; g < GROUPS; ++g) {
            all += s_all[g][threadIdx.x];
            before += s_before[g][threadIdx.x];
        }
        s_place[threadIdx.x] = all;
    }
    __syncthreads();
    int lists = 0;
    if (threadIdx.x < kHubLists && threadIdx.x != kShares)  // shares are numbered from zero
        for (int k = 0; k < (int)threadIdx.x; ++k) lists += s_place[k];
    if (blockIdx.x == 0 && threadIdx.x == kHubBuckets) place[0] = lists;
    if (blockIdx.x == 0 && threadIdx.x == kShares) {
        int items_all = 0;
        for (int k = 0; k < kShares; ++k) items_all += s_place[k];
        place[1] = items_all;
        place[2] = s_place[kShares];
    }
    __syncthreads();
    if (threadIdx.x < kHubLists) s_place[threadIdx.x] = lists + before;
    __syncthreads();
    block_items(
        n, nnz, rowptr, s_rows,
        [&](int list, int start, int length, int to) {
            const int at = take_places(s_place, list);
            if (list >= 0) items[at] = make_int4(start, length, to, 0);
        },
        [&](int row, int first, int count, int which) {
            tasks[atomicAdd(&s_place[kShares], 1)] = make_int4(row, first, count, which);
        },
        [&](int cls, int row, int start, int length) {
            const int at = take_places(s_place, cls < 0 ? -1 : kHubBuckets + cls);
            if (cls >= 0) items[at] = make_int4(start, length, row, 0);
        });
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
hub_gather_kernel(int nnz, int f, int ld, const int32_t *__restrict__ use,
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
    const unsigned pieces = place[0], all = place[1];
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

struct HubBuffers {
    int32_t *use, *place, *queues, *counts, *arrived;
    int4 *items, *tasks;
    float *part;
    int nqueues, narrived;
    size_t bytes;
};

HubBuffers carve(void *base, int64_t n, int64_t nnz, int ld) {
    Carver c(base);
    HubBuffers b;
    const int64_t pieces = ceil_div(nnz, kHubPiece);       // places for partial rows
    b.nqueues = 16 * kQueueStride * (int)ceil_div(ld, 4 * kWave);
    b.narrived = (int)(pieces / kHubShare + 1);
    b.use = c.take<int32_t>(1);
    b.place = c.take<int32_t>(3);
    b.queues = c.take<int32_t>(b.nqueues);
    b.counts = c.take<int32_t>(kHubLists * kListBlocks);
    b.arrived = c.take<int32_t>(b.narrived);
    b.items = c.take<int4>(pieces + n);
    b.tasks = c.take<int4>(nnz / kHubRow + pieces / kHubShare);             // long rows, and shares beyond their first
    b.part = c.take<float>((size_t)pieces * ld);
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
    const int64_t want = ceil_div(nnz / kHubPiece + n, 2 * kListThreads);
    const int blocks = (int)(want < kListBlocks ? want : kListBlocks);
    hipLaunchKernelGGL(hub_count_kernel, dim3(blocks), dim3(kListThreads), 0, st, n, nnz, rowptr, b.use, b.counts, b.queues,
                       b.nqueues, b.arrived, b.narrived);
    GNN_TRY(launch_status());
    hipLaunchKernelGGL(hub_scatter_kernel, dim3(blocks), dim3(kListThreads), 0, st, n, nnz, rowptr, b.use, b.counts, b.place,
                       b.items, b.tasks);
    GNN_TRY(launch_status());
    int lpe = pow2_at_least(ld / 4);
    if (lpe < 4) lpe = 4;
    if (lpe > kWave) lpe = kWave;
    const dim3 grid(kBlocksPerCu * 256, (unsigned)ceil_div(ld, 4 * lpe));
    // offsets of 32 bits from a 24-bit multiplication, where they reach
    const bool wide = n >= (1 << 24) || ld >= (1 << 22) || (int64_t)n * ld * 4 >= ((int64_t)1 << 32), ragged = f != ld;
#define HUB_LAUNCH(LPE_, WIDE_, RAGGED_)                                                                                   \
    if (lpe == LPE_ && wide == WIDE_ && ragged == RAGGED_)                                                                 \
        hipLaunchKernelGGL((hub_gather_kernel<LPE_, WIDE_, RAGGED_>), grid, dim3(256), 0, st, nnz, f, ld, b.use,           \
                           b.place, b.queues, b.items, col, w, B, b.part, C, bias, act);
#define HUB_CASE(LPE_)                                                                                                     \
    HUB_LAUNCH(LPE_, false, false) HUB_LAUNCH(LPE_, false, true) HUB_LAUNCH(LPE_, true, false) HUB_LAUNCH(LPE_, true, true)
    HUB_CASE(4) HUB_CASE(8) HUB_CASE(16) HUB_CASE(32) HUB_CASE(64)
    GNN_TRY(launch_status());
    *rest = HubReduce{b.use, b.place + 2, b.tasks, b.part, b.arrived, ld, lpe};
    return GNN_OK;
}

}  // namespace gnn
