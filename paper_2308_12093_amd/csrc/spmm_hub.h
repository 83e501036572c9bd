// Sparse-dense product of a graph with hubs, rows in pieces: see spmm_hub.hip.
#pragma once

#include "common.h"

namespace gnn {

constexpr int kHubRow = 128;          // entries from which on a row is cut into pieces
constexpr int kHubPiece = 64;         // entries of a piece, about
constexpr int kHubMaxPieces = 1024;   // pieces a row has at most
constexpr int kHubBuckets = 64;       // positions inside a row that the order of the pieces tells apart

__device__ __forceinline__ float activate(float x, int act) {
    if (act == kActRelu) x = fmaxf(x, 0.f);
    else if (act == kActElu) x = x > 0.f ? x : expm1f(x);
    return x;
}

// four floats at a 4-byte aligned address: global dwordx4 accesses need no more than that
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));

// What is left for the last kernel of the product: *use says whether there is anything, place[0] and place[nblk] how
// many long rows, rows their (row, first partial, partials), partials of ld floats for groups of lpf lanes.
struct HubReduce {
    const int32_t *use, *place;
    const int4 *rows;
    const float *part;
    int nblk, ld, lpf;
};

// One wavefront per long row: 64 / lpf slots of lpf lanes (four features each) take the row's partials in turn, four
// rotating sums a slot, then a fixed shuffle tree over the slots.
__device__ __forceinline__ void hub_reduce(const HubReduce &h, int f, float *__restrict__ C, const float *__restrict__ bias,
                                           int act) {
    const int hubs = h.place[h.nblk] - h.place[0], ld = h.ld, lpf = h.lpf;
    const int4 *__restrict__ rows = h.rows;
    const float *__restrict__ part = h.part;
    const int lane = threadIdx.x % kWave, slots = kWave / lpf, slot = lane / lpf, l = lane % lpf;
    for (int i = blockIdx.x * 4 + threadIdx.x / kWave; i < hubs; i += gridDim.x * 4) {
        const int4 r = rows[i];
        for (int cb = 0; cb < ld; cb += 4 * lpf) {
            const int c = cb + 4 * l;
            const bool ok = c < ld;
            const float *src = part + (size_t)r.y * ld + c;
            float a[4][4] = {};
            if (ok) {
                int x = slot;
                for (; x + 3 * slots < r.z; x += 4 * slots)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float4 q = *reinterpret_cast<const float4 *>(src + (size_t)(x + j * slots) * ld);
                        a[j][0] += q.x; a[j][1] += q.y; a[j][2] += q.z; a[j][3] += q.w;
                    }
                for (; x < r.z; x += slots) {
                    const float4 q = *reinterpret_cast<const float4 *>(src + (size_t)x * ld);
                    a[0][0] += q.x; a[0][1] += q.y; a[0][2] += q.z; a[0][3] += q.w;
                }
            }
            float t[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) t[j] = (a[0][j] + a[1][j]) + (a[2][j] + a[3][j]);
            for (int d = lpf; d < kWave; d <<= 1)
#pragma unroll
                for (int j = 0; j < 4; ++j) t[j] += __shfl_xor(t[j], d, kWave);
            if (ok && slot == 0) {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (c + j < f) t[j] = activate(bias ? t[j] + bias[c + j] : t[j], act);
                float *dst = C + (size_t)r.x * f + c;
                if (f == ld) *reinterpret_cast<float4 *>(dst) = make_float4(t[0], t[1], t[2], t[3]);
                else
                    for (int j = 0; j < 4; ++j)
                        if (c + j < f) dst[j] = t[j];
            }
        }
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
