// P[split][M][N] (double) = partial sums of X^T H over chunks of the rows, on the int8 matrix instruction.
//
// The gradient of a weight sums over every node, so its sums are kept in 64 bits (gemm.hip says why).  The fp64 matrix
// instruction does that at 50 - 57 of its 78.6 TFLOP/s; the int8 instruction is 60 times as fast, and integers are exact:
// every column of an operand is written in fixed point relative to a power of two above its largest magnitude, as five
// digits of eight bits (balanced, -128 .. 127),
//     x = 2^(e - 30) (d1 2^24 + d2 2^16 + d3 2^8 + d4 + d5 2^-8),        |x| <= 2^e,
// and the product of two operands is the sum of fifteen digit products d_i d'_j with i + j <= 6, collected by i + j in five
// int32 accumulators.  What is left out is below 2^-46 of the columns' largest magnitudes per product, the rounding of
// the fifth digit below 2^-39: on normal, positive and one-sided operands the float result is as far from the 64-bit
// one as the rounding to float makes it (relative 2-norm 2.5e-8 on normal operands of 2^13 .. 2^22 rows, both ways).
//
// The exponent of a column starts three bits above the largest magnitude of its first non-zero step of 32 rows.  When a
// larger value arrives, the block folds its integers into the double partials, in memory, and goes on with the new
// exponent; a column that has been zero so far changes its exponent for free.  The same fold runs every 512 steps,
// before the sum of five products (2^14 each) could pass 2^31, and at the end.  Columns that hold infinities or NaN, or
// are nowhere above 2^-105, are not representable: the block then forms its partial again in double arithmetic.
#include "common.h"

namespace gnn {
namespace {

typedef int intx4 __attribute__((ext_vector_type(4)));
typedef int intx16 __attribute__((ext_vector_type(16)));

constexpr int BT = 128;                                     // rows and columns of a block's tile
constexpr int STEP = 32;                                    // reduction rows of a step
constexpr int DIGITS = 5;
constexpr int FOLD_STEPS = 512;                             // 5 * 2^14 * 32 * 512 = 1.34e9 < 2^31
constexpr int HEADROOM = 3;
constexpr int E_MIN = -90;                                  // 2^(30 - e) stays a float
constexpr float kSmallest = 0x1p-105f, kTopScale = 0x1p120f;          // 2^(30 - E_MIN)
constexpr int BUF_WORDS = DIGITS * 8 * 64 * 4;              // [digit][column tile: four of X, four of H][lane][4]

__device__ __forceinline__ unsigned perm(unsigned hi, unsigned lo, unsigned sel) { return __builtin_amdgcn_perm(hi, lo, sel); }

// digits of four floats (scaled: |y| <= 2^30): word d holds digit d of all four, one byte each
__device__ __forceinline__ void digits4(float x0, float x1, float x2, float x3, float scale, unsigned (&out)[DIGITS]) {
    const float x[4] = {x0, x1, x2, x3};
    unsigned u[4], v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float y = x[i] * scale, t = rintf(y);
        u[i] = (unsigned)(int)t + 0x80808080u;             // balanced digits are the bytes of this, less 128
        // the remainder in 1/256: in the low byte of 1.5 * 2^23 + it; 0.498 keeps it below 128
        v[i] = __float_as_uint(fmaf(fminf(y - t, 0.498f), 256.f, 12582912.f));
    }
    const unsigned a = perm(u[1], u[0], 0x05010400), b = perm(u[3], u[2], 0x05010400);
    const unsigned c = perm(u[1], u[0], 0x07030602), d = perm(u[3], u[2], 0x07030602);
    out[3] = perm(b, a, 0x05040100) ^ 0x80808080u;
    out[2] = perm(b, a, 0x07060302) ^ 0x80808080u;
    out[1] = perm(d, c, 0x05040100) ^ 0x80808080u;
    out[0] = perm(d, c, 0x07060302) ^ 0x80808080u;
    out[4] = perm(perm(v[3], v[2], 0x0c0c0400), perm(v[1], v[0], 0x0c0c0400), 0x05040100);
}

// Eight wavefronts as 2 x 4, each 64 x 32 of the tile: 2 x 5 accumulators of 16 registers.  For the staging, wavefront w
// owns column tile w of eight (four of X, four of H): lane (half, l) takes 16 consecutive rows of column l, read as lines
// of 128 bytes, makes their digits and writes them where the instruction's lane (half, l) reads them.  One block per CU,
// 147 KB of LDS, one barrier per step.  Half of the wavefronts stage step s + 1 before they multiply step s, the others
// after.  A step takes some 4900 cycles, of which a wavefront multiplies 1200 (its 30 instructions take no less than
// 960) and stages 3000 - 3400: 1100 for the digits, 500 for the exponent, up to 1200 behind its loads.  Loads into
// registers a step ahead, __shfl, matrix and vector instructions interleaved by hand or by the compiler: all within 3 %.
template <bool MASK>
__global__ void __launch_bounds__(512, 2)
gemm_tn_digits_kernel(int M, int N, long K, const float *__restrict__ A, const float *__restrict__ B,
                      const uint32_t *__restrict__ keep, double *__restrict__ P, long k_chunk, int tiles_m, int tiles_n,
                      int splits, int wide_a, int wide_b) {
    extern __shared__ __align__(16) int lds[];              // two buffers of digits
    __shared__ double s_scale[2 * BT];                      // 2^(e - 30) of every column, as of the accumulators
    __shared__ float s_small[2 * BT];                       // largest magnitude of a column at the smallest exponent, else 1
    __shared__ int s_flag[2], s_bad;
    const long tiles = (long)tiles_m * tiles_n, total = tiles * splits, per_xcd = (total + 7) / 8;
    const long logical = (long)(blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
    if (blockIdx.x / 8 >= per_xcd || logical >= total) return;
    const int split = (int)(logical / tiles), tile = (int)(logical % tiles);
    const int m0 = (tile / tiles_n) * BT, n0 = (tile % tiles_n) * BT;
    const long kend = K - (splits - 1 - split) * k_chunk, kbeg = max(0L, kend - k_chunk);
    const int steps = (int)((kend - kbeg + STEP - 1) / STEP);

    const int t = threadIdx.x, lane = t % 64, wave = __builtin_amdgcn_readfirstlane(t / 64);
    const int l = lane % 32, half = lane / 32;
    const int wm = wave / 4, wn = wave % 4;
    double *out = P + (size_t)split * M * N;

    // ---- staging: this thread's column
    const bool side_b = wave >= 4;
    const int width = side_b ? N : M, colg = (side_b ? n0 : m0) + (wave % 4) * 32 + l;
    const bool colok = colg < width;
    // a uniform row base and the lane's offset inside a step of 32 rows
    const char *src = reinterpret_cast<const char *>(side_b ? B : A);
    const unsigned row_bytes = (unsigned)width * 4u, col_bytes = (unsigned)(colok ? colg : width - 1) * 4u;
    const unsigned pair_off = (unsigned)half * row_bytes + col_bytes;
    float raw[16];
    uint32_t bits = 0;                                                     // MASK: which of the 16 rows count
    // Step 0 is the ragged one; the steps after it are whole.  The loop below reads three steps past the last as well
    // (never used): kept inside the operand.
    const int ragged = (int)(kend - kbeg) - STEP * (steps - 1);            // rows of step 0, 1 .. 32
    auto first_row = [&](int step) __attribute__((always_inline)) { return min(kbeg + ragged + (long)(step - 1) * STEP, K - STEP); };
    // global -> LDS, two steps ahead and without registers: each wavefront fills and reads its own 4 KB of a slot
    int *s_raw = lds + 2 * BUF_WORDS + wave * 1024;
    // sixteen bytes a lane where the operand's rows allow it: 8 rows of 128 bytes per instruction, else 2
    const unsigned wide_off = (unsigned)(lane / 8) * row_bytes +
                              (unsigned)min((side_b ? n0 : m0) + (wave % 4) * 32 + (lane % 8) * 4, width - 4) * 4u;
    const bool wide = side_b ? wide_b : wide_a;
    auto fetch = [&](int step) __attribute__((always_inline)) {
        const char *from = src + (size_t)first_row(step) * row_bytes;
        int *to = s_raw + (step & 1) * 8192;
        if (wide) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(from + (size_t)(8 * r) * row_bytes + wide_off),
                                                 (__attribute__((address_space(3))) void *)(to + r * 256), 16, 0, 0);
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r)
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(from + (size_t)(2 * r) * row_bytes + pair_off),
                                                 (__attribute__((address_space(3))) void *)(to + r * 64), 4, 0, 0);
        }
    };
    auto read_raw = [&](int step) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 16; ++r) raw[r] = __int_as_float(s_raw[(step & 1) * 8192 + (16 * half + r) * 32 + l]);
    };
    auto load_bits = [&](int step) __attribute__((always_inline)) {
        if (MASK && side_b) {                              // past the last column: the next words, never used
            int c = threadIdx.x;
            asm volatile("" : "+v"(c));
            bits = keep[(size_t)((K - first_row(step)) / STEP - 1) * N + n0 + (wave % 4) * 32 + c % 32] >> (c & 32 ? 16 : 0);
        }
    };
    auto mask = [&]() __attribute__((always_inline)) {
        if (MASK && side_b) {
#pragma unroll
            for (int r = 0; r < 16; ++r)
                raw[r] = __uint_as_float(__float_as_uint(raw[r]) & (uint32_t)__builtin_amdgcn_sbfe((int)bits, r, 1));
        }
    };
    auto load_first = [&]() __attribute__((always_inline)) {
        const size_t base = (size_t)kbeg * row_bytes;
        uint32_t w = 0;
        if (MASK && side_b) w = keep[(size_t)((K - kbeg + STEP - 1) / STEP - 1) * N + col_bytes / 4] >> (STEP - ragged);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int q = 16 * half + r;                                   // past the end: the last row again, as zeros
            const unsigned off = (unsigned)min(q, ragged - 1) * row_bytes + col_bytes;
            const float x = *reinterpret_cast<const float *>(src + base + off);
            raw[r] = q < ragged && (!(MASK && side_b) || ((w >> q) & 1)) ? x : 0.f;
        }
    };
    float scale = 0.f;                                      // 2^(30 - e), 0 in a column of zeros
    bool pending = false;                                   // the exponent grew: s_scale is behind until the fold
    bool bad = false;
    // the exponent for the rows in `raw`; both halves of a column see the same magnitudes and hold the same scale
    auto fit = [&](int step, int buf) __attribute__((always_inline)) {
        unsigned mb = 0;                                    // magnitudes order like their bits, NaN last
#pragma unroll
        for (int i = 0; i < 16; ++i) mb = max(mb, __float_as_uint(raw[i]) & 0x7fffffffu);
        const auto halves = __builtin_amdgcn_permlane32_swap(mb, mb, false, false);
        mb = max((unsigned)halves[0], (unsigned)halves[1]);
        const float m = __uint_as_float(mb);
        if (colok && !(m * scale <= 0x1p30f && (mb == 0 || (scale != 0.f && scale != kTopScale)))) {
            int c = threadIdx.x;
            asm volatile("" : "+v"(c));                     // rare: its addresses stay out of the step loop's registers
            c = c / 64 * 32 + c % 32;                       // the column
            if (mb >= 0x7f800000u) bad = true;
            else if (m > 0.f) {
                if (scale == kTopScale) s_small[c] = fmaxf(s_small[c], m);
                if (m * scale > 0x1p30f || scale == 0.f) {
                    const bool grows = scale != 0.f;
                    const int e = max(ilogbf(m) + 1 + HEADROOM, E_MIN);
                    scale = ldexpf(1.f, 30 - e);
                    if (!grows) {
                        s_scale[c] = ldexp(1.0, e - 30);
                        s_small[c] = e == E_MIN ? m : 1.f;
                    } else {
                        pending = true;
                        s_small[c] = 1.f;
                        s_flag[buf] = step + 1;
                    }
                }
            }
        }
    };
    auto convert4 = [&](int buf, int g) __attribute__((always_inline)) {
        unsigned d[DIGITS];
        digits4(raw[4 * g], raw[4 * g + 1], raw[4 * g + 2], raw[4 * g + 3], scale, d);
#pragma unroll
        for (int i = 0; i < DIGITS; ++i) lds[buf * BUF_WORDS + ((i * 8 + wave) * 64 + lane) * 4 + g] = (int)d[i];
    };

    intx16 acc[2][DIGITS];
    auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int s = 0; s < DIGITS; ++s)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[x][s][v] = 0;
    };
    bool folded = false;
    // accumulator register v of lane (half, l): row 8 (v / 4) + 4 half + v % 4, column l of its 32 x 32 tile
    auto fold = [&]() __attribute__((always_inline)) {
        int zero = 0;
        asm volatile("" : "+v"(zero));                      // keeps the addresses below out of the step loop's registers
        const int nl = wn * 32 + l + zero, n = n0 + nl;
        const double sn = s_scale[BT + nl] * 65536.0;
        // eight outputs at a time: what memory holds of them is on its way while their digits are put together
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int v0 = 0; v0 < 16; v0 += 8) {
                const int mr = wm * 64 + x * 32 + v0 * 2 + 4 * half + zero;         // rows 8 (v / 4) + v % 4 from here
                double held[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int m = m0 + mr + 8 * (u / 4) + u % 4;
                    held[u] = folded && m < M && n < N ? out[(size_t)m * N + n] : 0.0;
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int ml = mr + 8 * (u / 4) + u % 4, m = m0 + ml, v = v0 + u;
                    double s = (double)acc[x][0][v];
#pragma unroll
                    for (int c = 1; c < DIGITS; ++c) s = s * 256.0 + (double)acc[x][c][v];
                    s = s * (s_scale[ml] * sn) + held[u];
                    if (m < M && n < N) out[(size_t)m * N + n] = s;
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        folded = true;
        clear();
    };
    clear();
    if (t < 2 * BT) { s_scale[t] = 0.0; s_small[t] = 1.f; }
    if (t < 2) s_flag[t] = 0;
    if (t == 2) s_bad = 0;
    __syncthreads();

    if (steps > 0) {
        load_first();
        fit(-1, 0);                                         // never grows: the columns are new
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            convert4(0, g);
        }
        load_bits(1);
        fetch(1);
        fetch(2);
    }
    int since = 0;
    for (int step = 0;; ++step) {
        const int buf = step & 1;
        // a barrier for the LDS writes alone: __syncthreads would wait for the loads of the steps ahead as well
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (step == steps || (step > 0 && s_flag[buf] == step) || since == FOLD_STEPS) {      // uniform
            fold();
            if (step == steps) break;
            __syncthreads();
            if (pending) s_scale[wave * 32 + l] = 1.0 / (double)scale;
            pending = false;
            since = 0;
            __syncthreads();
        }
        ++since;
        const int *in = lds + buf * BUF_WORDS + lane * 4;
        auto stage = [&]() __attribute__((always_inline)) {
            // the rows of step + 1 have arrived when no more loads are on their way than those of step + 2; their place
            // is free again when they have been read
            if (wide) asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
            else asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
            read_raw(step + 1);
            mask();
            load_bits(step + 2);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            fetch(step + 3);
            fit(step, buf ^ 1);
#pragma unroll
            for (int g = 0; g < 4; ++g) convert4(buf ^ 1, g);
        };
        auto multiply = [&]() __attribute__((always_inline)) {
            // X's digits from the last, which meets only H's first, up; the digits of the next round are read before the
            // matrix instructions of this one
            auto read_a = [&](int i, int x) __attribute__((always_inline)) { return *reinterpret_cast<const intx4 *>(in + ((i * 8 + 2 * wm + x) * 64) * 4); };
            auto read_b = [&](int j) __attribute__((always_inline)) { return *reinterpret_cast<const intx4 *>(in + ((j * 8 + 4 + wn) * 64) * 4); };
            intx4 b[DIGITS], a[2][2];
            b[0] = read_b(0);
            a[0][0] = read_a(DIGITS - 1, 0);
            a[0][1] = read_a(DIGITS - 1, 1);
#pragma unroll
            for (int g = 0; g < DIGITS; ++g) {
                const int i = DIGITS - 1 - g;
                if (g + 1 < DIGITS) {
                    b[g + 1] = read_b(g + 1);
                    a[(g + 1) & 1][0] = read_a(i - 1, 0);
                    a[(g + 1) & 1][1] = read_a(i - 1, 1);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; i + j < DIGITS; ++j)
#pragma unroll
                    for (int x = 0; x < 2; ++x)
                        acc[x][i + j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[g & 1][x], b[j], acc[x][i + j], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        // wavefronts w and w + 4 share a SIMD: one multiplies while the other stages
        if (!side_b) stage();
        __builtin_amdgcn_sched_barrier(0);
        multiply();
        __builtin_amdgcn_sched_barrier(0);
        if (side_b) stage();
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // no load into LDS outlives the block
    if (bad || (t < 2 * BT && s_small[t] < kSmallest)) s_bad = 1;
    __syncthreads();                                        // and the folded sums are written before they are replaced
    if (!s_bad) return;
    // in double, one output per thread and turn
    for (int o = t; o < BT * BT; o += 512) {
        const int m = m0 + o / BT, n = n0 + o % BT;
        if (m >= M || n >= N) continue;
        double s = 0.0;
        for (long k = kbeg; k < kend; ++k) {
            float x = B[(size_t)k * N + n];
            if constexpr (MASK) {
                const long back = K - 1 - k;                // rows are counted from the end
                if (!((keep[(size_t)(back / STEP) * N + n] >> (STEP - 1 - back % STEP)) & 1)) x = 0.f;
            }
            s += (double)A[(size_t)k * M + m] * (double)x;
        }
        out[(size_t)m * N + n] = s;
    }
}

// The chunks are cut from the last row back: only the first chunk, and in it the first step, can be ragged.
int digit_splits(int64_t M, int64_t N, int64_t K, int64_t *k_chunk) {
    const int64_t tiles = ceil_div(M, BT) * ceil_div(N, BT);
    int64_t s = 256 / tiles;                                // one block per CU
    if (s > K / 512) s = K / 512;
    if (s < 1) s = 1;
    const int64_t c = ceil_div(ceil_div(K, s), STEP) * STEP;
    if (k_chunk) *k_chunk = c;
    return (int)ceil_div(K, c);
}

size_t partial_bytes(int64_t M, int64_t N, int64_t K) {
    return align_up((size_t)digit_splits(M, N, K, nullptr) * M * N * sizeof(double));
}

// bit r of keep[b][n]: Y[row][n] > 0 for row = K - 32 (b + 1) + r
__global__ void __launch_bounds__(256)
pack_signs_kernel(int N, long K, const float *__restrict__ Y, uint32_t *__restrict__ keep) {
    const int n = blockIdx.y * 256 + threadIdx.x;
    if (n >= N) return;
    const long k0 = K - STEP * ((long)blockIdx.x + 1);
    uint32_t w = 0;
#pragma unroll
    for (int r = 0; r < STEP; ++r) {
        const float y = Y[(size_t)max(k0 + r, 0L) * N + n];
        if (y > 0.f && k0 + r >= 0) w |= 1u << r;
    }
    keep[(size_t)blockIdx.x * N + n] = w;
}

}  // namespace

// Where the digits pay: outputs that fill most of a 128 x 128 tile.  Both sides (fp64 instruction / digits, M x N, K):
// 128 x 128, 2^17 92 / 56 us; 128 x 512, 2^17 337 / 201; 256 x 256, 2^17 323 / 199, 2^15 289 / 55; 100 x 256, 2^20 1272 /
// 792; 512 x 512, 2^17 1097 / 683; 128 x 128, 2^13 50 / 41; but 64 x 256, 2^17 91 / 92, 64 x 64, 2^17 33 / 47,
// 256 x 47, 2^20 740 / 743, 100 x 47, 10^5 51 / 72.
bool gemm_tn_digits_shape(int64_t M, int64_t N, int64_t K) { return M > 64 && N > 64 && K >= 8192; }

size_t gemm_tn_digits_workspace_bytes(int64_t M, int64_t N, int64_t K) {
    return partial_bytes(M, N, K) + align_up(((size_t)ceil_div(K, STEP) * N + BT) * sizeof(uint32_t));
}

// Writes *splits partial products of M x N doubles to the workspace.  relu_y: NULL, or B counts only where it is > 0.
gnn_status_t gemm_tn_digits_launch(int64_t M, int64_t N, int64_t K, const float *A, const float *B, const float *relu_y,
                                   void *workspace, int *splits, hipStream_t st) {
    const int tiles_m = (int)ceil_div(M, BT), tiles_n = (int)ceil_div(N, BT);
    int64_t k_chunk;
    *splits = digit_splits(M, N, K, &k_chunk);
    double *P = static_cast<double *>(workspace);
    uint32_t *keep = reinterpret_cast<uint32_t *>(static_cast<char *>(workspace) + partial_bytes(M, N, K));
    if (relu_y) {
        hipLaunchKernelGGL(pack_signs_kernel, dim3((unsigned)ceil_div(K, STEP), (unsigned)ceil_div(N, 256)), dim3(256), 0, st,
                           (int)N, (long)K, relu_y, keep);
        GNN_TRY(launch_status());
    }
    const long total = (long)tiles_m * tiles_n * *splits;
    const dim3 grid((unsigned)(8 * ceil_div(total, 8)));
    const int wide_a = aligned16(A) && M % 4 == 0, wide_b = aligned16(B) && N % 4 == 0;
    const size_t bytes = (size_t)(2 * BUF_WORDS + 2 * 8192) * sizeof(int);
    if (relu_y)
        hipLaunchKernelGGL(gemm_tn_digits_kernel<true>, grid, dim3(512), bytes, st, (int)M, (int)N, (long)K, A, B, keep, P,
                           (long)k_chunk, tiles_m, tiles_n, *splits, wide_a, wide_b);
    else
        hipLaunchKernelGGL(gemm_tn_digits_kernel<false>, grid, dim3(512), bytes, st, (int)M, (int)N, (long)K, A, B, keep, P,
                           (long)k_chunk, tiles_m, tiles_n, *splits, wide_a, wide_b);
    return launch_status();
}

}  // namespace gnn
