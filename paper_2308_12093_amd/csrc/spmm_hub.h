// Sparse-dense product of a graph with hubs, rows in pieces: see spmm_hub.hip.
#pragma once

#include "common.h"

namespace gnn {

constexpr int kHubRow = 128;          // entries from which on a row is cut into pieces
constexpr int kHubPiece = 64;         // entries of a piece, about: 49 to 111, whatever the length of its row
// Partial rows that one wavefront adds up.  Rows beyond 512 pieces are shared by several: the longest one alone was half of
// the kernel.  256 / 512 / 1024, us, 2^20 nodes, 53 M entries, f = 100 122 / 103 / 131, f = 47 93 / 59 / 70: small shares
// pay for the fences between them.
constexpr int kHubShare = 512;

__device__ __forceinline__ float activate(float x, int act) {
    if (act == kActRelu) x = fmaxf(x, 0.f);
    else if (act == kActElu) x = x > 0.f ? x : expm1f(x);
    return x;
}

// four floats at a 4-byte aligned address: global dwordx4 accesses need no more than that
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));

// What is left for the last kernel of the product: *use says whether there is anything, *ntasks how much: sums of up to
// kHubShare partial rows of one row (row, its first partial, its partials, which of its shares), partials of ld floats for
// groups of lpf lanes.  arrived counts the shares of a row that are done, at the row's first partial over kHubShare: rows
// with more than one share are more than kHubShare partials apart.
struct HubReduce {
    const int32_t *use, *ntasks;
    const int4 *tasks;
    float *part;
    int32_t *arrived;
    int ld, lpf;
};

// Rows x, x + by, ... (n of them) of `part` added up, column c ... c + 3 of each: 64 / lpf slots of lpf lanes take them in
// turn, four rotating sums a slot, then a fixed shuffle tree over the slots.
__device__ __forceinline__ void hub_add(const float *part, int ld, int lpf, size_t x, size_t by, int n, int c, float (&t)[4]) {
    const int slots = kWave / lpf, slot = threadIdx.x % kWave / lpf;
    const float *src = part + x * ld + c;
    float a[4][4];
#pragma unroll
    for (int j = 0; j < 16; ++j) a[j / 4][j % 4] = -0.f;   // x + -0 is x: sums that underflow to -0 stay that
    if (c < ld) {
        int i = slot;
        for (; i + 3 * slots < n; i += 4 * slots)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float4 q = *reinterpret_cast<const float4 *>(src + (size_t)(i + j * slots) * by * ld);
                a[j][0] += q.x; a[j][1] += q.y; a[j][2] += q.z; a[j][3] += q.w;
            }
        for (; i < n; i += slots) {
            const float4 q = *reinterpret_cast<const float4 *>(src + (size_t)i * by * ld);
            a[0][0] += q.x; a[0][1] += q.y; a[0][2] += q.z; a[0][3] += q.w;
        }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) t[j] = (a[0][j] + a[1][j]) + (a[2][j] + a[3][j]);
    for (int d = lpf; d < kWave; d <<= 1)
#pragma unroll
        for (int j = 0; j < 4; ++j) t[j] += __shfl_xor(t[j], d, kWave);
}

// One wavefront per share.  The sum of a row's only share is the row; else it takes the place of the share's first partial,
// and the wavefront that finds all others of the row done adds those sums, in their order, whichever wavefront that is.
__device__ __forceinline__ void hub_reduce(const HubReduce &h, int f, float *__restrict__ C, const float *__restrict__ bias,
                                           int act) {
    const int tasks = *h.ntasks, ld = h.ld, lpf = h.lpf;
    const int lane = threadIdx.x % kWave, l = lane % lpf;
    auto finish = [&](int row, size_t x, size_t by, int n) __attribute__((always_inline)) {
        for (int c = 4 * l; c - 4 * l < ld; c += 4 * lpf) {
            float t[4];
            hub_add(h.part, ld, lpf, x, by, n, c, t);
            if (lane < lpf && c < ld) {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (c + j < f) t[j] = activate(bias ? t[j] + bias[c + j] : t[j], act);
                float *dst = C + (size_t)row * f + c;
                if (f == ld) *reinterpret_cast<float4 *>(dst) = make_float4(t[0], t[1], t[2], t[3]);
                else
                    for (int j = 0; j < 4; ++j)
                        if (c + j < f) dst[j] = t[j];
            }
        }
    };
    for (int i = blockIdx.x * 4 + threadIdx.x / kWave; i < tasks; i += gridDim.x * 4) {
        const int4 p = h.tasks[i];
        if (p.z <= kHubShare) {
            finish(p.x, p.y, 1, p.z);
            continue;
        }
        const size_t x = (size_t)p.y + (size_t)p.w * kHubShare;
        for (int c = 4 * l; c - 4 * l < ld; c += 4 * lpf) {
            float t[4];
            hub_add(h.part, ld, lpf, x, 1, min(p.z - p.w * kHubShare, kHubShare), c, t);
            if (lane < lpf && c < ld) *reinterpret_cast<float4 *>(h.part + x * ld + c) = make_float4(t[0], t[1], t[2], t[3]);
        }
        __threadfence();
        const int shares = (p.z + kHubShare - 1) / kHubShare;
        int before = 0;
        if (lane == 0) before = atomicAdd(&h.arrived[p.y / kHubShare], 1);
        if (__builtin_amdgcn_readfirstlane(before) != shares - 1) continue;
        __threadfence();
        finish(p.x, p.y, kHubShare, shares);
    }
}

// C = act(A B + bias) but for hub_reduce, unless few entries lie in long rows: then nothing is written and *rest->use is
// zero once the launches have run.  n rows, columns < n.  B has rows of ld floats (a multiple of four, 16-byte
// aligned), C rows of f <= ld.  workspace: hub_workspace_bytes
size_t hub_workspace_bytes(int64_t n, int64_t nnz, int ld);
gnn_status_t hub_spmm_launch(int n, int nnz, const int32_t *rowptr, const int32_t *col, EdgeWeights w, const float *B,
                             int f, int ld, float *C, const float *bias, int act, void *workspace, hipStream_t st,
                             HubReduce *rest);

}  // namespace gnn
