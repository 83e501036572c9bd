// Graph preprocessing: integer kernels (self-loops + degrees, CSR -> CSC, expansion of
// row pointers) and the symmetric normalisation  A' = D^-1/2 (A + I) D^-1/2
// (Sec. "GCN Forward Pass").  Every output is deterministic: integer atomics are
// only used for counts and maxima, and the CSC order comes from a stable radix sort.
#include "common.h"

namespace gnn {
namespace {

constexpr int SCAN_ITEMS = 16;                   // per thread
constexpr int SCAN_TILE = 256 * SCAN_ITEMS;

// Sum of one value per thread over a block of 256; every thread gets it.
__device__ __forceinline__ int32_t block_sum(int32_t v, int32_t *wave_tot) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    if (threadIdx.x % 64 == 0) wave_tot[threadIdx.x / 64] = v;
    __syncthreads();
    return wave_tot[0] + wave_tot[1] + wave_tot[2] + wave_tot[3];
}

// Exclusive scan of one tile per block; block totals go to `sums` (if not NULL).
__global__ void __launch_bounds__(256)
scan_tile_kernel(long count, int32_t *__restrict__ data, int32_t *__restrict__ sums) {
    __shared__ int32_t wave_tot[4];
    const long base = (long)blockIdx.x * SCAN_TILE + (long)threadIdx.x * SCAN_ITEMS;
    int32_t v[SCAN_ITEMS];
    int32_t tsum = 0;
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        v[i] = base + i < count ? data[base + i] : 0;
        tsum += v[i];
    }
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    int32_t incl = tsum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int32_t o = __shfl_up(incl, d, 64);
        if (lane >= d) incl += o;
    }
    if (lane == 63) wave_tot[wave] = incl;
    __syncthreads();
    int32_t off = 0;
    for (int w = 0; w < wave; ++w) off += wave_tot[w];
    int32_t run = off + incl - tsum;
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        if (base + i < count) data[base + i] = run;
        run += v[i];
    }
    if (sums && threadIdx.x == 255) sums[blockIdx.x] = off + incl;
}

// Adds to every element of a tile what stands before the tile: the sum of the preceding tiles' totals, which each
// block forms by itself (RAW: `sums` holds totals), or the scanned totals as they are.
template <bool RAW>
__global__ void __launch_bounds__(256)
scan_add_kernel(long count, int32_t *__restrict__ data, const int32_t *__restrict__ sums) {
    __shared__ int32_t wave_tot[4];
    const long i = (long)blockIdx.x * SCAN_TILE + threadIdx.x;
    int32_t add;
    if constexpr (RAW) {
        int32_t t = 0;
        for (int b = threadIdx.x; b < (int)blockIdx.x; b += 256) t += sums[b];
        add = block_sum(t, wave_tot);
    } else {
        add = sums[blockIdx.x];
    }
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; ++k) {
        const long j = i + (long)k * 256;
        if (j < count) data[j] += add;
    }
}

// A scan of a few elements is bound by its launches (4 - 5 us each): up to kScanFlat tiles the second kernel sums the
// tile totals itself, at most 16 per thread, and two launches do; only longer arrays scan the totals in between.
constexpr long kScanFlat = 4096;

gnn_status_t exclusive_scan_inplace(int32_t *data, long count, int32_t *ws, hipStream_t st) {
    if (count <= 0) return GNN_OK;
    const long blocks = ceil_div(count, SCAN_TILE);
    int32_t *sums = blocks > 1 ? ws : nullptr;
    hipLaunchKernelGGL(scan_tile_kernel, dim3((unsigned)blocks), dim3(256), 0, st, count, data, sums);
    GNN_TRY(launch_status());
    if (blocks > kScanFlat) {
        GNN_TRY(exclusive_scan_inplace(sums, blocks, ws + align_up(blocks * sizeof(int32_t)) / sizeof(int32_t), st));
        hipLaunchKernelGGL(scan_add_kernel<false>, dim3((unsigned)blocks), dim3(256), 0, st, count, data, sums);
        GNN_TRY(launch_status());
    } else if (blocks > 1) {
        hipLaunchKernelGGL(scan_add_kernel<true>, dim3((unsigned)blocks), dim3(256), 0, st, count, data, sums);
        GNN_TRY(launch_status());
    }
    return GNN_OK;
}

// ---- the rows of a tile of entries ----------------------------------------------------
// Kernels that need the row of every stored entry walk tiles of consecutive entries, not rows: rows of an R-MAT graph
// have from 0 to 10^5 entries and 15 - 30 on average, so a wavefront per row leaves most lanes idle and still waits
// for the hubs.  A tile finds the rows that start inside it by a search over the row pointers, marks their first
// entries in LDS and spreads the marks with a running maximum.
// Tiles of 4096 entries amortise the search; lists of less than 2^20 entries are cut into tiles of 1024, four times as
// many blocks and a quarter of the rounds per thread (30 000 entries, insertion of the diagonal: 15 -> 7.5 us).
constexpr int ROW_THREADS = 256;
constexpr int ROW_TILE = 4096, ROW_TILE_SMALL = 1024;
constexpr long ROW_SMALL = 1 << 20;

// First index in [0, len) with ptr[index] >= x (len if there is none); ptr ascending.  All 64 lanes of a wavefront
// probe at once: four dependent loads for a million rows.
__device__ __forceinline__ int wave_lower_bound(const int32_t *__restrict__ ptr, int len, long x) {
    const int lane = threadIdx.x % 64;
    long lo = 0, hi = len;
    while (lo < hi) {
        const long step = (hi - lo + 63) / 64;
        const long p = lo + lane * step;
        const int c = __popcll(__ballot(p < hi && (long)ptr[p < hi ? p : hi - 1] < x));
        if (c == 0) { hi = lo; break; }
        const long top = lo + (long)c * step;
        lo += (long)(c - 1) * step + 1;
        hi = top < hi ? top : hi;
    }
    return (int)lo;
}

// A tile in which more rows start than this times its entries holds a long run of empty ones (isolated nodes at the end of
// the numbering, say) and searches the row of every entry: some 28 us for 4096 entries in half a million rows, where one
// block that visits the rows takes 1.1 ns for each (2^20 rows, the last half empty, 4.2 M entries: 584 and 39 us).
constexpr int kRowsPerEntry = 4;

// s_row[j] = row of entry base + j for the j < T whose entry exists.  Ends with a barrier.
template <int THREADS, int T>
__device__ __forceinline__ void tile_rows(int n, const int32_t *__restrict__ ptr, long base, int32_t *s_row,
                                          int32_t *s_misc /* [2 + THREADS / 64] */) {
    constexpr int PER = T / THREADS;
    static_assert(PER % 4 == 0, "marks are read four at a time");
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    if (wave < 2) {
        const int r = wave_lower_bound(ptr, n, base + (wave == 0 ? 0 : T));
        if (lane == 0) s_misc[wave] = r;
    }
    for (int j = threadIdx.x; j < T; j += THREADS) s_row[j] = -1;
    __syncthreads();
    const int first = s_misc[0], last = s_misc[1];           // rows [first, last) start in the tile
    if (last - first > kRowsPerEntry * T) {                  // uniform
        const long q = ptr[n];
        for (int j = threadIdx.x; j < T && base + j < q; j += THREADS) {
            int lo = max(first - 1, 0), hi = last;           // the last row of [lo, hi) that starts at the entry or before
            while (hi - lo > 1) {
                const int mid = lo + (hi - lo) / 2;
                if ((long)ptr[mid] <= base + j) lo = mid; else hi = mid;
            }
            s_row[j] = lo;
        }
        __syncthreads();
        return;
    }
    for (int r = first + (int)threadIdx.x; r < last; r += THREADS)
        atomicMax(&s_row[ptr[r] - base], r);                 // of rows that share a slot only the last has entries
    __syncthreads();
    int32_t v[PER];
    int32_t run = -1;
#pragma unroll
    for (int k = 0; k < PER; k += 4) {
        const int4 q = *reinterpret_cast<const int4 *>(s_row + (int)threadIdx.x * PER + k);
        v[k] = run = max(run, q.x);
        v[k + 1] = run = max(run, q.y);
        v[k + 2] = run = max(run, q.z);
        v[k + 3] = run = max(run, q.w);
    }
    int32_t incl = run;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int32_t o = __shfl_up(incl, d, 64);
        if (lane >= d) incl = max(incl, o);
    }
    if (lane == 63) s_misc[2 + wave] = incl;
    int32_t before = __shfl_up(incl, 1, 64);
    if (lane == 0) before = -1;
    __syncthreads();
    before = max(before, first - 1);                         // the row that began before the tile
    for (int w = 0; w < wave; ++w) before = max(before, s_misc[2 + w]);
#pragma unroll
    for (int k = 0; k < PER; k += 4)
        *reinterpret_cast<int4 *>(s_row + (int)threadIdx.x * PER + k) =
            make_int4(max(v[k], before), max(v[k + 1], before), max(v[k + 2], before), max(v[k + 3], before));
    __syncthreads();
}

// blocks for a list whose length is only known on the device, and for the rows: they share them among themselves
constexpr int kRowBlocks = 2048;                             // eight blocks of 256 threads per CU

// ---- self-loops ---------------------------------------------------------------------
// new length of row i: one more unless the diagonal is already stored
__global__ void __launch_bounds__(256)
selfloop_count_kernel(int n, const int32_t *__restrict__ rowptr, const int32_t *__restrict__ col,
                      int32_t *__restrict__ newlen, int32_t *__restrict__ deg) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i > n) return;
    if (i == n) { newlen[n] = 0; return; }
    int lo = rowptr[i], hi = rowptr[i + 1];
    const int len = hi - lo;
    while (lo < hi) {                               // first slot with col >= i
        const int mid = (lo + hi) >> 1;
        if (col[mid] < i) lo = mid + 1; else hi = mid;
    }
    const int has = lo < rowptr[i + 1] && col[lo] == i;
    newlen[i] = len + 1 - has;
    deg[i] = len + 1 - has;
}

// Copies the entry list, inserting the diagonal of every row that lacks it at its sorted position: in front of the
// first entry above it, behind the last entry below it, or alone in an empty row.  Bound by the list's bytes (read
// once, written once): 2^20 nodes, 16.8 M entries 351 -> 68 us against a wavefront per row.
template <int T>
__global__ void __launch_bounds__(ROW_THREADS)
selfloop_fill_kernel(int n, const int32_t *__restrict__ rowptr, const int32_t *__restrict__ col,
                     const int32_t *__restrict__ rowptr_out, int32_t *__restrict__ col_out) {
    __shared__ __align__(16) int32_t s_row[T];
    __shared__ int32_t s_misc[2 + ROW_THREADS / 64];
    const long q = rowptr[n];
    // empty rows have no entry in any tile: dealt to the blocks on their own
    for (long r = (long)blockIdx.x * ROW_THREADS + threadIdx.x; r < n; r += (long)gridDim.x * ROW_THREADS)
        if (rowptr[r] == rowptr[r + 1]) col_out[rowptr_out[r]] = (int32_t)r;
    for (long base = (long)blockIdx.x * T; base < q; base += (long)gridDim.x * T) {
        tile_rows<ROW_THREADS, T>(n, rowptr, base, s_row, s_misc);
        for (int j = threadIdx.x; j < T && base + j < q; j += ROW_THREADS) {
            const long x = base + j;
            const int i = s_row[j], c = col[x];
            const long s = rowptr[i], e = rowptr[i + 1], o = rowptr_out[i];
            const long grow = (rowptr_out[i + 1] - o) - (e - s);     // 1 if the diagonal has to be inserted
            const long at = o + (x - s) + (c > i ? grow : 0);
            col_out[at] = c;
            if (grow) {
                if (c > i && (x == s || col[x - 1] < i)) col_out[at - 1] = i;
                else if (c < i && x + 1 == e) col_out[at + 1] = i;
            }
        }
        __syncthreads();                                     // the next tile overwrites s_row
    }
}

// One weight per entry.  Bound by the 4-byte gathers of the column's degree: 2^20 nodes, 17.8 M entries 494 -> 110 us
// against a wavefront per row.
template <int T>
__global__ void __launch_bounds__(ROW_THREADS)
normalize_kernel(int n, const int32_t *__restrict__ rowptr, const int32_t *__restrict__ col,
                 const int32_t *__restrict__ deg, float *__restrict__ val, int kind, float eps) {
    __shared__ __align__(16) int32_t s_row[T];
    __shared__ int32_t s_misc[2 + ROW_THREADS / 64];
    const long q = rowptr[n];
    for (long base = (long)blockIdx.x * T; base < q; base += (long)gridDim.x * T) {
        tile_rows<ROW_THREADS, T>(n, rowptr, base, s_row, s_misc);
#pragma unroll 4
        for (int j = threadIdx.x; j < T && base + j < q; j += ROW_THREADS) {
            const long x = base + j;
            const int i = s_row[j], c = col[x];
            float v;
            if (kind == GNN_AGG_GCN_SYM) v = 1.0f / sqrtf((float)deg[i] * (float)deg[c]);
            else if (kind == GNN_AGG_MEAN) v = 1.0f / (float)deg[i];
            else v = c == i ? 1.0f + eps : 1.0f;
            val[x] = v;
        }
        __syncthreads();
    }
}

// out[x] = row of entry x: a write of the list and little else (17.8 M entries 118 -> 29 us).
template <int T>
__global__ void __launch_bounds__(ROW_THREADS)
expand_ptr_kernel(int n, const int32_t *__restrict__ ptr, int32_t *__restrict__ out) {
    __shared__ __align__(16) int32_t s_row[T];
    __shared__ int32_t s_misc[2 + ROW_THREADS / 64];
    const long q = ptr[n];
    for (long base = (long)blockIdx.x * T; base < q; base += (long)gridDim.x * T) {
        tile_rows<ROW_THREADS, T>(n, ptr, base, s_row, s_misc);
        for (int j = threadIdx.x; j < T && base + j < q; j += ROW_THREADS) out[base + j] = s_row[j];
        __syncthreads();
    }
}

__global__ void __launch_bounds__(256)
gather_f32_kernel(long count, const float *__restrict__ in, const int32_t *__restrict__ perm, float *__restrict__ out) {
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i < count) out[i] = in[perm[i]];
}

// ---- CSR -> CSC ---------------------------------------------------------------------
constexpr int RADIX_THREADS = 512;
constexpr int RADIX_ITEMS = 16;                             // entries per thread
constexpr int RADIX_TILE = RADIX_THREADS * RADIX_ITEMS;     // entries per block
constexpr int RADIX_WAVES = RADIX_THREADS / 64;             // wavefront w owns entries [w * 1024, (w + 1) * 1024) of it
constexpr int RADIX_DIGITS = 256;                           // digits of at most eight bits

__global__ void __launch_bounds__(RADIX_THREADS)
radix_hist_kernel(long count, const int32_t *__restrict__ keys, int shift, int mask, int nblocks,
                  int32_t *__restrict__ hist) {
    __shared__ int32_t h[RADIX_DIGITS];
    if (threadIdx.x < RADIX_DIGITS) h[threadIdx.x] = 0;
    __syncthreads();
    const long base = (long)blockIdx.x * RADIX_TILE;
#pragma unroll
    for (int r = 0; r < RADIX_ITEMS; ++r) {
        const long idx = base + r * RADIX_THREADS + threadIdx.x;
        if (idx < count) atomicAdd(&h[(keys[idx] >> shift) & mask], 1);
    }
    __syncthreads();
    if ((int)threadIdx.x <= mask) hist[(size_t)threadIdx.x * nblocks + blockIdx.x] = h[threadIdx.x];
}

// Stable scatter of one tile by one digit of the column.  `offs` holds, digit-major, the exclusive scan of the
// per-block digit counts.  Order inside a tile: wavefront, then round, then lane.  An entry travels as (column, row,
// CSR slot); FIRST: the row and the slot are those of the entry's place in the CSR arrays.
//
// Bound by memory: 24 bytes per entry and pass.  The tile is ordered in LDS first, one array after the other through
// the same 32 KB, so that the entries of a digit leave as one run (64 of them on average at 7-bit digits): written
// straight from registers, the 4-byte stores of 256 open runs per block filled lines piecemeal and a pass over 17.8 M
// entries took 357 us for two arrays; 115 us now for three.  Carrying the row costs 8 bytes per pass and saves
// the gather of every row through the sorted slots (188 us, one line per entry).
template <bool FIRST>
__global__ void __launch_bounds__(RADIX_THREADS)
radix_scatter_kernel(long count, int n, const int32_t *__restrict__ rowptr, const int32_t *__restrict__ keys,
                     const int32_t *__restrict__ rows, const int32_t *__restrict__ slots, int shift, int mask,
                     int nblocks, const int32_t *__restrict__ offs, int32_t *__restrict__ keys_out,
                     int32_t *__restrict__ rows_out, int32_t *__restrict__ slots_out) {
    __shared__ __align__(16) int32_t s_tile[RADIX_TILE];
    __shared__ int32_t wbase[RADIX_WAVES][RADIX_DIGITS];
    __shared__ int32_t shift_of[RADIX_DIGITS];              // global position of a digit's run minus its place in the tile
    __shared__ int32_t s_misc[2 + RADIX_WAVES];
    const int t = threadIdx.x, wave = t / 64, lane = t % 64;
    const long tile0 = (long)blockIdx.x * RADIX_TILE;
    const int here = (int)min((long)RADIX_TILE, count - tile0);
    const int mine = wave * (64 * RADIX_ITEMS) + lane;      // item r of this thread: entry mine + 64 r of the tile
    for (int i = t; i < RADIX_WAVES * RADIX_DIGITS; i += RADIX_THREADS) (&wbase[0][0])[i] = 0;
    int32_t k[RADIX_ITEMS], row[RADIX_ITEMS], slot[RADIX_ITEMS];
#pragma unroll
    for (int r = 0; r < RADIX_ITEMS; ++r) {
        const int j = mine + 64 * r;
        k[r] = j < here ? keys[tile0 + j] : 0;
        if constexpr (!FIRST) {
            row[r] = j < here ? rows[tile0 + j] : 0;
            slot[r] = j < here ? slots[tile0 + j] : 0;
        } else {
            slot[r] = (int32_t)(tile0 + j);
        }
    }
    if constexpr (FIRST) {
        tile_rows<RADIX_THREADS, RADIX_TILE>(n, rowptr, tile0, s_tile, s_misc);
#pragma unroll
        for (int r = 0; r < RADIX_ITEMS; ++r) row[r] = s_tile[mine + 64 * r];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RADIX_ITEMS; ++r)
        if (mine + 64 * r < here) atomicAdd(&wbase[wave][(k[r] >> shift) & mask], 1);
    __syncthreads();
    // start of every digit inside the tile (exclusive scan over the digits), then per wavefront inside the digit
    int32_t total = 0, incl = 0;
    if (t < RADIX_DIGITS) {
#pragma unroll
        for (int w = 0; w < RADIX_WAVES; ++w) total += wbase[w][t];
        incl = total;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int32_t o = __shfl_up(incl, d, 64);
            if (lane >= d) incl += o;
        }
        if (lane == 63) s_misc[wave] = incl;
    }
    __syncthreads();
    if (t < RADIX_DIGITS) {
        int32_t run = incl - total;
        for (int w = 0; w < wave; ++w) run += s_misc[w];
        shift_of[t] = (t <= mask ? offs[(size_t)t * nblocks + blockIdx.x] : 0) - run;
#pragma unroll
        for (int w = 0; w < RADIX_WAVES; ++w) {
            const int32_t c = wbase[w][t];
            wbase[w][t] = run;
            run += c;
        }
    }
    __syncthreads();
    int32_t pos[RADIX_ITEMS];
    volatile int32_t *cnt = wbase[wave];
    const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
    for (int r = 0; r < RADIX_ITEMS; ++r) {
        const bool valid = mine + 64 * r < here;
        const int digit = (k[r] >> shift) & mask;
        unsigned long long same = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const bool bit = (digit >> b) & 1;
            const unsigned long long bal = __ballot(valid && bit);
            same &= bit ? bal : ~bal;
        }
        const int rank = __popcll(same & below);
        const int in_digit = __popcll(same);
        pos[r] = 0;
        if (valid) pos[r] = cnt[digit] + rank;
        __builtin_amdgcn_wave_barrier();
        if (valid && rank == in_digit - 1) cnt[digit] = pos[r] + 1;
        __builtin_amdgcn_wave_barrier();
    }
    // through LDS in tile order, out in runs
    auto place = [&](const int32_t (&v)[RADIX_ITEMS]) __attribute__((always_inline)) {
        __syncthreads();
#pragma unroll
        for (int r = 0; r < RADIX_ITEMS; ++r)
            if (mine + 64 * r < here) s_tile[pos[r]] = v[r];
        __syncthreads();
    };
    int32_t to[RADIX_ITEMS];                                // where entry t + RADIX_THREADS r of the ordered tile goes
    place(k);
#pragma unroll
    for (int r = 0; r < RADIX_ITEMS; ++r) {
        const int j = t + RADIX_THREADS * r;
        if (j < here) {
            const int32_t key = s_tile[j];
            to[r] = shift_of[(key >> shift) & mask] + j;
            keys_out[to[r]] = key;
        }
    }
    place(row);
#pragma unroll
    for (int r = 0; r < RADIX_ITEMS; ++r)
        if (t + RADIX_THREADS * r < here) rows_out[to[r]] = s_tile[t + RADIX_THREADS * r];
    place(slot);
#pragma unroll
    for (int r = 0; r < RADIX_ITEMS; ++r)
        if (t + RADIX_THREADS * r < here) slots_out[to[r]] = s_tile[t + RADIX_THREADS * r];
}

// colptr[j] = first place of the sorted column list that holds a column >= j.  (Counting the columns with atomics, the
// other way to it, serialises on the hubs: 910 us at 17.8 M entries, 32 us for the search.)
__global__ void __launch_bounds__(256)
column_start_kernel(int n, long nnz, const int32_t *__restrict__ sorted, int32_t *__restrict__ colptr) {
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j > n) return;
    long lo = 0, hi = nnz;
    while (lo < hi) {
        const long mid = (lo + hi) >> 1;
        if (sorted[mid] < j) lo = mid + 1; else hi = mid;
    }
    colptr[j] = (int32_t)lo;
}

// Digits of the column number: as few passes as eight bits each allow, and then digits as short as that many passes
// allow (20 bits: 7 each), which makes the runs longer.
int radix_bits(int n) {
    int bits = 0;
    while ((1ll << bits) < (long long)n) ++bits;
    return bits < 1 ? 1 : bits;
}

size_t scan_ws_ints(long count) {
    size_t total = 0;
    long c = count;
    while (c > SCAN_TILE) {
        c = ceil_div(c, SCAN_TILE);
        total += align_up(c * sizeof(int32_t)) / sizeof(int32_t);
    }
    return total + kAlign / sizeof(int32_t);
}

}  // namespace

size_t scan_workspace_bytes(int64_t n) { return align_up(scan_ws_ints(n + 1) * sizeof(int32_t)); }

gnn_status_t exclusive_scan_launch(int32_t *data, long count, void *workspace, hipStream_t st) {
    return exclusive_scan_inplace(data, count, static_cast<int32_t *>(workspace), st);
}

gnn_status_t add_self_loops_launch(int n, int nnz, const int32_t *rowptr, const int32_t *col, int32_t *rowptr_out,
                                   int32_t *col_out, int32_t *deg_out, void *workspace, hipStream_t st) {
    hipLaunchKernelGGL(selfloop_count_kernel, dim3((unsigned)ceil_div(n + 1, 256)), dim3(256), 0, st, n, rowptr, col,
                       rowptr_out, deg_out);
    GNN_TRY(launch_status());
    GNN_TRY(exclusive_scan_inplace(rowptr_out, (long)n + 1, static_cast<int32_t *>(workspace), st));
    if (n > 0) {
        const bool small = nnz < ROW_SMALL;
        const long tiles = ceil_div(nnz, small ? ROW_TILE_SMALL : ROW_TILE);
        const long rows = ceil_div(n, ROW_THREADS), blocks = rows < kRowBlocks ? rows : kRowBlocks;   // for the empty rows
        hipLaunchKernelGGL(small ? selfloop_fill_kernel<ROW_TILE_SMALL> : selfloop_fill_kernel<ROW_TILE>,
                           dim3((unsigned)(tiles > blocks ? tiles : blocks)), dim3(ROW_THREADS), 0, st, n, rowptr, col,
                           rowptr_out, col_out);
        GNN_TRY(launch_status());
    }
    return GNN_OK;
}

gnn_status_t normalize_launch(int n, const int32_t *rowptr, const int32_t *col, const int32_t *deg, float *val,
                              int kind, float eps, hipStream_t st) {
    if (n <= 0) return GNN_OK;
    // the number of entries stands in rowptr[n]: taken as some 16 per row here
    const bool small = n < ROW_SMALL / 16;
    hipLaunchKernelGGL(small ? normalize_kernel<ROW_TILE_SMALL> : normalize_kernel<ROW_TILE>, dim3(kRowBlocks),
                       dim3(ROW_THREADS), 0, st, n, rowptr, col, deg, val, kind, eps);
    return launch_status();
}

gnn_status_t expand_ptr_launch(int n, int nnz, const int32_t *ptr, int32_t *out, hipStream_t st) {
    if (n <= 0) return GNN_OK;
    // nnz sets the number of blocks alone: what is written is what ptr says
    const bool small = nnz < ROW_SMALL;
    const long tiles = ceil_div(nnz > 0 ? nnz : 1, small ? ROW_TILE_SMALL : ROW_TILE);
    hipLaunchKernelGGL(small ? expand_ptr_kernel<ROW_TILE_SMALL> : expand_ptr_kernel<ROW_TILE>, dim3((unsigned)tiles),
                       dim3(ROW_THREADS), 0, st, n, ptr, out);
    return launch_status();
}

gnn_status_t gather_f32_launch(int64_t count, const float *in, const int32_t *perm, float *out, hipStream_t st) {
    if (count <= 0) return GNN_OK;
    hipLaunchKernelGGL(gather_f32_kernel, dim3((unsigned)ceil_div(count, 256)), dim3(256), 0, st, (long)count, in,
                       perm, out);
    return launch_status();
}

// workspace layout: keys_a[nnz] | keys_b[nnz] | rows_b[nnz] | slots_b[nnz] | hist[256 * nblocks] | scan scratch
size_t transpose_workspace_bytes(int n, int nnz) {
    const long nblocks = ceil_div(nnz > 0 ? nnz : 1, RADIX_TILE);
    const long hist = RADIX_DIGITS * nblocks;
    const long biggest_scan = hist > (long)n + 1 ? hist : (long)n + 1;
    return 4 * align_up((size_t)(nnz > 0 ? nnz : 1) * sizeof(int32_t)) + align_up(hist * sizeof(int32_t)) +
           align_up(scan_ws_ints(biggest_scan) * sizeof(int32_t));
}

gnn_status_t transpose_launch(int n, int nnz, const int32_t *rowptr, const int32_t *col, int32_t *colptr,
                              int32_t *row, int32_t *perm, void *workspace, hipStream_t st) {
    Carver ws(workspace);
    const long q = nnz;
    const long nblocks = ceil_div(q > 0 ? q : 1, RADIX_TILE);
    int32_t *keys_a = ws.take<int32_t>(q > 0 ? q : 1);
    int32_t *keys_b = ws.take<int32_t>(q > 0 ? q : 1);
    int32_t *rows_b = ws.take<int32_t>(q > 0 ? q : 1);
    int32_t *slots_b = ws.take<int32_t>(q > 0 ? q : 1);
    int32_t *hist = ws.take<int32_t>(RADIX_DIGITS * nblocks);
    int32_t *scan_ws = reinterpret_cast<int32_t *>(ws.base + ws.off);

    // Stable LSD radix sort of the entry list by column; with an entry go its row and its CSR slot.
    // Buffers alternate so that the last pass lands in (row, perm).
    if (q > 0) {
        const int bits = radix_bits(n), passes = (bits + 7) / 8, width = (bits + passes - 1) / passes;
        const int mask = (1 << width) - 1;
        const int32_t *kin = col, *rin = nullptr, *sin = nullptr;
        for (int p = 0; p < passes; ++p) {
            const bool to_out = ((passes - 1 - p) % 2) == 0;
            int32_t *kout = to_out ? keys_a : keys_b, *rout = to_out ? row : rows_b, *sout = to_out ? perm : slots_b;
            hipLaunchKernelGGL(radix_hist_kernel, dim3((unsigned)nblocks), dim3(RADIX_THREADS), 0, st, q, kin, width * p,
                               mask, (int)nblocks, hist);
            GNN_TRY(launch_status());
            GNN_TRY(exclusive_scan_inplace(hist, (mask + 1) * nblocks, scan_ws, st));
            if (p == 0)
                hipLaunchKernelGGL(radix_scatter_kernel<true>, dim3((unsigned)nblocks), dim3(RADIX_THREADS), 0, st, q, n,
                                   rowptr, kin, rin, sin, width * p, mask, (int)nblocks, hist, kout, rout, sout);
            else
                hipLaunchKernelGGL(radix_scatter_kernel<false>, dim3((unsigned)nblocks), dim3(RADIX_THREADS), 0, st, q, n,
                                   rowptr, kin, rin, sin, width * p, mask, (int)nblocks, hist, kout, rout, sout);
            GNN_TRY(launch_status());
            kin = kout; rin = rout; sin = sout;
        }
    }
    hipLaunchKernelGGL(column_start_kernel, dim3((unsigned)ceil_div((long)n + 1, 256)), dim3(256), 0, st, n, q, keys_a, colptr);
    return launch_status();
}

}  // namespace gnn
