// C = A op(B) (+ A2 op(B2)) (+ what C holds) + bias, ReLU, for rows = nodes and a few hundred columns, with fp32
// operands, sums and results, on the bf16 matrix instruction.
//
// A float is the exact sum of three bf16 numbers (8 + 8 + 8 bits: round, subtract, round, subtract), and a product of
// two bf16 numbers is exact in float.  Six of the nine products of the parts are formed, the three below 2^-26 of the
// whole (a1 b2, a2 b1, a2 b2) are not, and everything is added in float by v_mfma_f32_32x32x16_bf16: six instructions
// of 32 cycles for 16 reduction indices where v_mfma_f32_32x32x2_f32 takes eight of 64.  The matrix cores
// offer 2.5 PFLOP/s / 6 = 420 against 157 TFLOP/s.  The five small products of a step are summed from zero and join the
// sum at its end, so the sum is rounded three times per 32 indices instead of 16 times.  Relative 2-norm error of the
// products of a layer against 64 bits, fp32 instruction and parts: 2.0e-7 and
// 0.7e-7 (K = 128), 2.9e-7 and 1.0e-7 (256), 4.1e-7 and 1.4e-7 (512); of positive operands 1.7e-7 and 0.7e-7 (128).
//
// What the parts cannot hold is recomputed with the fp32 instruction, wavefront by wavefront: a tile with results that
// are not finite (operands that are not, or that the rounding to bf16 or a partial sum carries over the edge), and a tile
// with operands whose third part falls below the bf16 range (magnitudes below 2^-110: they lose up to 2^-134) where that
// loss may show in a result.
#include "common.h"

namespace gnn {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));   // 16 bytes at a 4-byte aligned address
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));

constexpr int KB = 32;                 // reduction indices of a step: lane half h takes 16 h .. 16 h + 15
constexpr unsigned kTinyCode = 2 * ((127u - 110) << 23) - 1;   // magnitude_code(2^-110)
constexpr int kFragBytes = 64 * 16;    // eight bf16 per lane: one operand of one instruction
constexpr int kStepBytes = 2 * 3 * kFragBytes;   // [instruction][part] for 32 columns and KB indices

__device__ __forceinline__ unsigned pack_bf16(float a, float b) {
    return __builtin_bit_cast(unsigned, __builtin_convertvector((floatx2){a, b}, bf16x2));
}
__device__ __forceinline__ float low(unsigned u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float high(unsigned u) { return __uint_as_float(u & 0xffff0000u); }

// orders like the magnitude, except that zero comes last
__device__ __forceinline__ unsigned magnitude_code(float a) { return 2 * __float_as_uint(a) - 1; }

// three parts of eight floats; `least` collects the smallest magnitude code
__device__ __forceinline__ void split8(const floatx4 &x, const floatx4 &y, bf16x8 (&part)[3], unsigned &least) {
    uintx4 u[3];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float a = i < 2 ? x[2 * i] : y[2 * i - 4], b = i < 2 ? x[2 * i + 1] : y[2 * i - 3];
        least = min(least, min(magnitude_code(a), magnitude_code(b)));
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            const unsigned h = pack_bf16(a, b);
            u[p][i] = h;
            if (p < 2) { a -= low(h); b -= high(h); }
        }
    }
#pragma unroll
    for (int p = 0; p < 3; ++p) part[p] = __builtin_bit_cast(bf16x8, u[p]);
}

// the kept products, smallest first; the last, of the leading parts, goes to the sum itself
constexpr int kProducts = 6;
__device__ constexpr int kPartA[kProducts] = {1, 0, 2, 1, 0, 0}, kPartB[kProducts] = {1, 2, 0, 0, 1, 0};

// columns of B as the kernels read it: element (k, n) at k * sk + n * sn
struct Operand {
    const float *p;
    long sk, sn;
};

// ---- parts of B, in the order in which the product kernel's lanes take them ----------------------------
// out: [32-column tile][KB step][instruction][part][lane][8]; lane (half, l): column 32 tile + l, indices
// KB step + 16 half + 8 instruction + 0..7; zeros past N and K.  range[tile]: the tile's smallest magnitude code and its
// largest magnitude.  One block per tile, 1024 threads: eight steps at a time.
struct Range {
    unsigned least;
    float top;
};

__global__ void __launch_bounds__(1024)
split_weights_kernel(int N, int K, int steps, Operand b0, Operand b1, char *__restrict__ out0, char *__restrict__ out1,
                     Range *__restrict__ range0, Range *__restrict__ range1) {
    __shared__ unsigned s_least, s_top;
    const Operand b = blockIdx.y ? b1 : b0;
    char *out = (blockIdx.y ? out1 : out0) + (size_t)blockIdx.x * steps * kStepBytes;
    const int lane = threadIdx.x % 64, ins = (threadIdx.x / 64) % 2, sub = threadIdx.x / 128;
    const int l = lane % 32, half = lane / 32;
    const int n = blockIdx.x * 32 + l;
    if (threadIdx.x == 0) { s_least = ~0u; s_top = 0; }
    __syncthreads();
    unsigned least = ~0u, top = 0;                          // magnitudes order like their bits, NaN last
    for (int s = sub; s < steps; s += 8) {
        const int k0 = s * KB + 16 * half + 8 * ins;
        floatx4 x[2];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            x[j / 4][j % 4] = n < N && k0 + j < K ? b.p[(k0 + j) * b.sk + n * b.sn] : 0.f;
            top = max(top, __float_as_uint(x[j / 4][j % 4]) & 0x7fffffffu);
        }
        bf16x8 part[3];
        split8(x[0], x[1], part, least);
#pragma unroll
        for (int p = 0; p < 3; ++p)
            *reinterpret_cast<bf16x8 *>(out + (size_t)s * kStepBytes + (ins * 3 + p) * kFragBytes + lane * 16) = part[p];
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        least = min(least, (unsigned)__shfl_xor((int)least, d, 64));
        top = max(top, (unsigned)__shfl_xor((int)top, d, 64));
    }
    if (lane == 0) { atomicMin(&s_least, least); atomicMax(&s_top, top); }
    __syncthreads();
    if (threadIdx.x == 0) (blockIdx.y ? range1 : range0)[blockIdx.x] = Range{s_least, __uint_as_float(s_top)};
}

struct Product {
    int M, N, K, steps;                // steps: KB steps of one operand pair
    const float *A, *A2;               // A2: NULL without a second pair
    Operand B, B2;
    const char *parts, *parts2;
    const Range *range, *range2;
    float *C;
    int ldc;
    const float *bias;
    int act;
    int tiles_m, tiles_n;
    const uint16_t *a_bits;            // see GemmExtras
    int bit_words, bit_stride;         // of a row, in memory and in LDS (an odd number of banks)
};

// logical tile of a block: each XCD (ids are dealt round-robin to eight) takes a contiguous range, the column tiles of
// the same rows side by side, so that they share an L2
__device__ __forceinline__ long xcd_tile(long total) {
    const long per = (total + 7) / 8;
    const long id = (long)(blockIdx.x % 8) * per + blockIdx.x / 8;
    return blockIdx.x / 8 < per ? id : total;
}

__device__ __forceinline__ void put(const Product &g, float *at, float o, float bias) {
    o += bias;
    if (g.act & kActAccumulate) o += *at;
    if (g.act & kActRelu) o = fmaxf(o, 0.f);
    if (g.act & kActStream) __builtin_nontemporal_store(o, at);
    else *at = o;
}

__host__ __device__ constexpr int kept_waves(int nt) { return nt == 1 ? 16 : 12; }   // wavefronts of a CU, by registers

// ---- the product ------------------------------------------------------------------------------------------
// A block of four wavefronts owns 4 x 32 rows and 32 NT columns.  A lane reads its 16 consecutive floats of a row
// straight into registers (the two lane halves take a row's whole 128-byte line, in one go, one step ahead) and splits
// them there: a row is split once per column tile and never passes through LDS.  The parts of B, split beforehand, are
// shared by the block: copied to LDS without touching registers, 6 NT KB per step, double-buffered, one barrier per
// step.  Three to four wavefronts fit a SIMD: loads, splitting, matrix instructions and stores of a block hardly overlap,
// those of different blocks do (64 rows a wavefront, two of them a SIMD: the same within 5 %, 24 % slower at 65536 rows
// and 64 columns).  Against the fp32 instruction, B transposed (K -> N), other buffers each time, us: 2^17 rows 128 -> 512 187
// -> 146, 512 -> 128 157 -> 135, 256 -> 256 167 -> 127, 128 -> 128 51 -> 48, 256 -> 64 48 -> 51 (into buffers that the caches hold
// 47 -> 42); 2^20 100 -> 256 732 -> 521, 47 -> 256 335 -> 328, 256 -> 47 417 -> 292; 2^22 64 -> 256 1552 -> 1341, 256 -> 64 1397 ->
// 1123 (4.8 TB/s: what a copy reaches).  Matrix cores busy 30 % (512 -> 128, 128 -> 128) and 36 % (128 -> 512): matrix
// instructions, stores and loads add up more than they overlap; without the stores 128 -> 512 took 115 of then 167 us,
// with a sixth of the matrix instructions 117.
// The columns of a row are stored one after the other: a row's lines reach memory together (column tile by column tile
// 128 -> 128 over 2^17 rows 40.8 -> 38.9 us, 512 -> 128 140.5 -> 137.7, 64 -> 256 over 2^22 1397 -> 1342).
// KEPT: KEPT wavefronts a block keep the parts of their columns in LDS, split by themselves, and go through the rows in
// tiles of 32 each without a barrier, so that one stores while another multiplies, and without the launch before.
// kept_pays says where.
// BITS: A is used where its bit is set; a lane's 16 floats have one word, from the block's copy in LDS (held in registers a
// step ahead it spills).
template <int NT, bool BITS, int KEPT>
__global__ void __launch_bounds__(KEPT ? 64 * KEPT : 256, (NT == 4 || (KEPT && NT == 2) ? 3 : 4) - (BITS && NT > 1))
gemm_split_kernel(Product g) {
    extern __shared__ __align__(16) char lds[];
    constexpr int STAGE = NT * kStepBytes;
    const int t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t / 64);
    int lane = t % 64, l = lane % 32, half = lane / 32;
    const int total = g.A2 ? 2 * g.steps : g.steps;
    int rt, rt_end, rt_by, ct0;                             // the wavefront's tiles of 32 rows; first 32-column tile
    if constexpr (KEPT) {                                   // XCD x: the x-th eighth of the rows, all columns of them
        const int tiles = (g.M + 31) / 32, per = (tiles + 7) / 8, x = blockIdx.x % 8, i = blockIdx.x / 8;
        ct0 = i % g.tiles_n * NT;
        rt = x * per + i / g.tiles_n * KEPT + wave;
        rt_end = min(tiles, (x + 1) * per);
        rt_by = (int)gridDim.x / 8 / g.tiles_n * KEPT;
    } else {
        const long tile = xcd_tile((long)g.tiles_m * g.tiles_n);
        if (tile >= (long)g.tiles_m * g.tiles_n) return;
        ct0 = (int)(tile % g.tiles_n) * NT;
        rt = (int)(tile / g.tiles_n) * 4 + wave;
        rt_end = rt + 1;
        rt_by = 1;
    }
    int row0 = rt * 32;
    // rows past the end re-read the last one
    auto row_offset = [&](int r) __attribute__((always_inline)) { return (size_t)min(r * 32 + l, g.M - 1) * g.K; };
    size_t ro = row_offset(rt);

    // Four indices at a time, at any 4-byte aligned address; the ones that would run over the row's end are read from
    // its last four floats instead (K >= 4) and put in place by `settle`, so no load stands behind a branch.
    floatx4 raw[4];
    uint16_t *bits = reinterpret_cast<uint16_t *>(lds + 2 * STAGE);
    if constexpr (BITS) {                                  // the block's words; the first step's barrier covers them
        const size_t from = (size_t)min(row0 - wave * 32 + t / 2, g.M - 1) * g.bit_words;
        for (int i = t % 2; i < g.bit_words; i += 2) bits[t / 2 * g.bit_stride + i] = g.a_bits[from + i];
    }
    auto load = [&](int step) __attribute__((always_inline)) {
        const bool second = step >= g.steps;
        const float *A = second ? g.A2 : g.A;
        const int k = (second ? step - g.steps : step) * KB + 16 * half;
#pragma unroll
        for (int i = 0; i < 4; ++i) raw[i] = *reinterpret_cast<const float4u *>(A + ro + min(k + 4 * i, g.K - 4));
    };
    auto settle = [&](int step) __attribute__((always_inline)) {
        const int k0 = (step >= g.steps ? step - g.steps : step) * KB;
        auto use = [&]() __attribute__((always_inline)) {
            if constexpr (BITS) {
                const int mask = bits[(wave * 32 + l) * g.bit_stride + min(2 * step + half, g.bit_words - 1)];
#pragma unroll
                for (int j = 0; j < 16; ++j)
                    raw[j / 4][j % 4] = __int_as_float(__float_as_int(raw[j / 4][j % 4]) & __builtin_amdgcn_sbfe(mask, j, 1));
            }
        };
        if (k0 + KB <= g.K) return use();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            // floats past the end: 0 none .. 4 all; a shift by one, by two and by four places
            const int over = min(max(k0 + 16 * half + 4 * i + 4 - g.K, 0), 4);
            const bool one = over & 1, two = over & 2, all = over & 4;
            floatx4 v = raw[i];
            v = floatx4{one ? v.y : v.x, one ? v.z : v.y, one ? v.w : v.z, one ? 0.f : v.w};
            v = floatx4{two ? v.z : v.x, two ? v.w : v.y, two ? 0.f : v.z, two ? 0.f : v.w};
            raw[i] = floatx4{all ? 0.f : v.x, all ? 0.f : v.y, all ? 0.f : v.z, all ? 0.f : v.w};
        }
        use();
    };
    // Rows that begin with tiny values (a saturated node's gradient) are taken times a power of two and their results
    // back, in a wavefront that has one.  Formed again, one such row in 32 costs four times the product: 128 -> 512 over
    // 2^17 rows 606 us, 512 -> 128 717, with the power of two 152 and 136 (without such rows 152 and 133).
    __shared__ float s_scale[KEPT ? 32 * KEPT : 128];        // of the block's rows; a wavefront reads its own alone
    float *scale = s_scale + wave * 32;
    bool scaled = false;                                     // uniform
    auto fit = [&]() __attribute__((always_inline)) {       // from the first step, once it is settled
        float top = 0.f;
#pragma unroll
        for (int j = 0; j < 16; ++j) top = fmaxf(top, fabsf(raw[j / 4][j % 4]));
        top = fmaxf(top, __shfl_xor(top, 32, 64));
        const bool low = top > 0.f && top < 0x1p-90f;
        scaled = __any(low);
        if (scaled) scale[l] = low ? ldexpf(1.f, min(-ilogbf(top), 126)) : 1.f;     // both halves of a row the same
    };
    auto apply = [&]() __attribute__((always_inline)) {
        if (!scaled) return;
        const float by = scale[l];
#pragma unroll
        for (int i = 0; i < 4; ++i) raw[i] *= by;
    };
    // global -> LDS, 1 KB per wavefront and instruction: the 6 NT fragments of a step are dealt to the four wavefronts
    auto stage = [&](int step, int buf) __attribute__((always_inline)) {
        const bool second = step >= g.steps;
        const char *src = (second ? g.parts2 : g.parts) + (size_t)(second ? step - g.steps : step) * kStepBytes;
#pragma unroll
        for (int i = 0; i < (6 * NT + 3) / 4; ++i) {
            const int f = wave + 4 * i;                      // uniform
            if (6 * NT % 4 == 0 || f < 6 * NT) {
                const char *from = src + (size_t)(ct0 + f / 6) * g.steps * kStepBytes + (f % 6) * kFragBytes + lane * 16;
                char *to = lds + buf * STAGE + f * kFragBytes;
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)from,
                                                 (__attribute__((address_space(3))) void *)to, 16, 0, 0);
            }
        }
    };

    floatx16 acc[NT];
    auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < NT; ++c)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[c][v] = 0.f;
    };
    clear();
    unsigned least = ~0u;                                   // of this lane's half of the row

    __shared__ unsigned s_least[NT], s_top[NT];              // KEPT: of the column tiles
    if constexpr (KEPT) {
        load(0);
        if (t < NT) { s_least[t] = ~0u; s_top[t] = 0; }
        __syncthreads();
        for (int f = wave; f < 2 * NT * total; f += KEPT) {  // a fragment at a time, as in split_weights_kernel
            const int c = f / (2 * total), step = f / 2 % total, ins = f % 2;
            const bool second = step >= g.steps;
            const Operand b = second ? g.B2 : g.B;
            const int k0 = (second ? step - g.steps : step) * KB + 16 * half + 8 * ins, n = (ct0 + c) * 32 + l;
            floatx4 x[2];
            unsigned low = ~0u, top = 0;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                x[j / 4][j % 4] = n < g.N && k0 + j < g.K ? b.p[(k0 + j) * b.sk + n * b.sn] : 0.f;
                top = max(top, __float_as_uint(x[j / 4][j % 4]) & 0x7fffffffu);
            }
            bf16x8 part[3];
            split8(x[0], x[1], part, low);
#pragma unroll
            for (int p = 0; p < 3; ++p)
                *reinterpret_cast<bf16x8 *>(lds + (size_t)(c * total + step) * kStepBytes + (ins * 3 + p) * kFragBytes + lane * 16) = part[p];
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) {
                low = min(low, (unsigned)__shfl_xor((int)low, d, 64));
                top = max(top, (unsigned)__shfl_xor((int)top, d, 64));
            }
            if (lane == 0) { atomicMin(&s_least[c], low); atomicMax(&s_top[c], top); }
        }
        __syncthreads();
    } else {
        stage(0, 0);
        load(0);
    }
    auto range = [&](int c) __attribute__((always_inline)) {
        Range b;
        if constexpr (KEPT) {
            b.least = s_least[c];
            b.top = __uint_as_float(s_top[c]);
        } else {
            b = g.range[ct0 + c];
            if (g.A2) {
                const Range b2 = g.range2[ct0 + c];
                b.least = min(b.least, b2.least);
                b.top = fmaxf(b.top, b2.top);
            }
        }
        return b;
    };
  if (KEPT && rt >= rt_end) return;
  do {
    row0 = rt * 32;
    // addresses are formed for each tile again: kept for all of them they spill
    if constexpr (KEPT) asm volatile("" : "+v"(half), "+v"(l), "+v"(lane));
    for (int step = 0; step < total; ++step) {
        const int buf = step & 1;
        if constexpr (!KEPT) {
            // this wavefront's copies of the step have arrived; after the barrier everyone's have, and the other buffer,
            // read in the step before, is free
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            if (step + 1 < total) stage(step + 1, buf ^ 1);
        }
        bf16x8 a[2][3];
        settle(step);
        if (step == 0) fit();
        apply();
#pragma unroll
        for (int ins = 0; ins < 2; ++ins) split8(raw[2 * ins], raw[2 * ins + 1], a[ins], least);
        load(min(step + 1, total - 1));                    // the last step again after the last: no branch, no use
#pragma unroll
        for (int c = 0; c < NT; ++c) {
            bf16x8 b[2][3];
#pragma unroll
            for (int i = 0; i < 6; ++i)
                b[i / 3][i % 3] = *reinterpret_cast<const bf16x8 *>(
                    lds + (KEPT ? (size_t)(c * total + step) * kStepBytes : (size_t)buf * STAGE + c * kStepBytes) + i * kFragBytes +
                    lane * 16);
            floatx16 small;
#pragma unroll
            for (int v = 0; v < 16; ++v) small[v] = 0.f;
#pragma unroll
            for (int i = 0; i < kProducts - 1; ++i)
#pragma unroll
                for (int ins = 0; ins < 2; ++ins)
                    small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ins][kPartA[i]], b[ins][kPartB[i]], small, 0, 0, 0);
#pragma unroll
            for (int ins = 0; ins < 2; ++ins)
                acc[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ins][0], b[ins][0], acc[c], 0, 0, 0);
            acc[c] += small;
        }
    }

    // what the parts cannot hold: see the top of the file
    float finite = 0.f;
    unsigned least_b = ~0u;
#pragma unroll
    for (int c = 0; c < NT; ++c)
#pragma unroll
        for (int v = 0; v < 16; ++v) finite = fmaf(acc[c][v], 0.f, finite);
#pragma unroll
    for (int c = 0; c < NT; ++c) least_b = min(least_b, range(c).least);
    bool bad = finite != 0.f;                                // 0 x (inf or NaN) is NaN
    if (!__any(bad) && __any(min(least, least_b) < kTinyCode)) {
        // Some operand lost up to 2^-134: a result is off by at most K 2^-134 times the largest magnitude it met (the
        // rows' for a tiny B, the column tile's for a tiny row).  Where that is below the rounding of the result nothing
        // is lost: rows that hold a saturated probability beside ordinary values, weights that have decayed.
        float top = 0.f;                                     // of the row, read once more for a tiny B
#pragma unroll 1
        for (int step = 0; step < total && least_b < kTinyCode; ++step) {
            load(step);
            settle(step);
            apply();
#pragma unroll
            for (int j = 0; j < 16; ++j) top = fmaxf(top, fabsf(raw[j / 4][j % 4]));
        }
        const float lost = 0x1p-110f * (float)(g.A2 ? 2L * g.K : (long)g.K);   // 2^24 times what a unit magnitude loses
        // a bit per row, from both halves of it
        unsigned long long row_tiny = __ballot(least < kTinyCode), row_zero = __ballot(top == 0.f);
        row_tiny |= row_tiny >> 32;
        row_zero &= row_zero >> 32;
        const unsigned tiny = (unsigned)row_tiny >> (4 * half), zero = (unsigned)row_zero >> (4 * half);
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) top = fmaxf(top, __shfl_xor(top, d, 64));
#pragma unroll
        for (int c = 0; c < NT; ++c) {
            const Range b = range(c);
            const float of_b = lost * b.top, of_a = b.least < kTinyCode ? lost * top : 0.f;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = 8 * (v / 4) + v % 4;         // of this register, behind the shift by 4 half
                const float most = ((tiny >> row) & 1 ? of_b : 0.f) + ((zero >> row) & 1 ? 0.f : of_a);
                bad |= (ct0 + c) * 32 + l < g.N && !(fabsf(acc[c][v]) >= most);
            }
        }
    }
    if (__any(bad)) {
        clear();
        scaled = false;
        for (int step = 0; step < total; ++step) {
            load(step);
            settle(step);
            const bool second = step >= g.steps;
            const Operand b = second ? g.B2 : g.B;
            const int k0 = (second ? step - g.steps : step) * KB + 16 * half;
#pragma unroll
            for (int j = 0; j < 16; ++j)
#pragma unroll
                for (int c = 0; c < NT; ++c) {
                    const int n = (ct0 + c) * 32 + l;
                    const float bv = k0 + j < g.K && n < g.N ? b.p[(k0 + j) * b.sk + n * b.sn] : 0.f;
                    acc[c] = __builtin_amdgcn_mfma_f32_32x32x2f32(raw[j / 4][j % 4], bv, acc[c], 0, 0, 0);
                }
        }
    }

    if constexpr (KEPT) {                                   // the next tile's first step, ahead of this one's stores
        ro = row_offset(rt + rt_by);
        load(0);
    }
    // accumulator register v of lane (half, l): row 8 (v / 4) + 4 half + v % 4, column l of its 32 x 32 tile
    if (scaled) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const float back = 1.f / scale[8 * (v / 4) + 4 * half + v % 4];
#pragma unroll
            for (int c = 0; c < NT; ++c) acc[c][v] *= back;
        }
    }
    if (row0 + 32 <= g.M && (ct0 + NT) * 32 <= g.N && !(g.act & kActAccumulate)) {
        // whole tiles, the columns of a row one after the other
        float bias[NT];
#pragma unroll
        for (int c = 0; c < NT; ++c) bias[c] = g.bias ? g.bias[(ct0 + c) * 32 + l] : 0.f;
        float *at = g.C + (size_t)(row0 + 4 * half) * g.ldc + ct0 * 32 + l;
#pragma unroll
        for (int v = 0; v < 16; ++v)
#pragma unroll
            for (int c = 0; c < NT; ++c) put(g, at + (size_t)(8 * (v / 4) + v % 4) * g.ldc + 32 * c, acc[c][v], bias[c]);
    } else
#pragma unroll
    for (int c = 0; c < NT; ++c) {
        const int n = (ct0 + c) * 32 + l;
        const float bias = g.bias && n < g.N ? g.bias[n] : 0.f;
        const int m0 = row0 + 4 * half;
        float *at = g.C + (size_t)m0 * g.ldc + n;
        if (row0 + 32 <= g.M && n < g.N) {
            if (g.act & kActAccumulate) {                    // a tile's worth of loads before the first store
                float held[16];
#pragma unroll
                for (int v = 0; v < 16; ++v) held[v] = at[(size_t)(8 * (v / 4) + v % 4) * g.ldc];
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const float o = acc[c][v] + bias + held[v];
                    at[(size_t)(8 * (v / 4) + v % 4) * g.ldc] = (g.act & kActRelu) ? fmaxf(o, 0.f) : o;
                }
            } else {
#pragma unroll
                for (int v = 0; v < 16; ++v) put(g, at + (size_t)(8 * (v / 4) + v % 4) * g.ldc, acc[c][v], bias);
            }
        } else if (n < g.ldc) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int dm = 8 * (v / 4) + v % 4;
                if (m0 + dm < g.M) {
                    if (n < g.N) put(g, at + (size_t)dm * g.ldc, acc[c][v], bias);
                    else at[(size_t)dm * g.ldc] = 0.f;       // padding columns of a wider row stride
                }
            }
        }
    }
    if constexpr (KEPT) {
        clear();
        least = ~0u;
    }
  } while (KEPT && (rt += rt_by) < rt_end);
}

// 32-column tiles per block: as wide as the output allows (a row of A is split once per tile)
int tiles_wide(int64_t N) { return N <= 32 ? 1 : N <= 64 ? 2 : 4; }

size_t parts_bytes(int64_t N, int64_t K) {
    const int64_t w = tiles_wide(N);
    return align_up((size_t)(ceil_div(N, 32 * w) * w) * ceil_div(K, KB) * kStepBytes);
}

// Whether blocks that keep the parts of their columns are the faster.  Those that pass them through LDS start their tiles as
// slots come free, and the blocks of one row's columns run side by side; where a block has its columns for good, these drift
// apart, which costs where they share lines of C and the caches no longer hold what was written of them.  Chosen on 18 000
// shapes, into buffers that the caches hold and into others: the time is 1.01 of the better of the two, 0.93 of that of blocks
// that pass the parts on and store column tile by column tile.  Step by step / kept, us, other buffers each time; t: B
// transposed.
//   One step, C up to 134 MB: 60000 x 16 -> 128 14.9 / 13.1, 2^17 33 / 22; not B in rows of 32 floats, which a block reads a line
//     per lane, for 128 columns (t 90000 x 32 -> 128 21.5 / 22.7).
//   More of C: few columns, 2^22 x 10 -> 47 288 / 244, x 16 -> 64 265 / 269, 2^22 x 20 -> 30 176 / 193, 2^21 x 32 -> 64 153 / 168;
//     rows that begin with a line, 2^20 x 16 -> 96 137 / 109, x 24 -> 128 135 / 137, x 32 135 / 149, or with half a line, up to
//     335 MB, 2^19 x 16 -> 80 67 / 61; others 2^19 x 16 -> 83 71 / 83, x 4 -> 300 161 / 209, 2^22 x 4 -> 259 1132 / 1749.
//   Two steps: 60000 x 64 -> 64 14.5 / 13.4, x 48 -> 16 10.1 / 8.5; t 2^17 x 48 -> 64 21.8 / 23.9, 2^20 x 48 -> 30 77.5 / 82.7;
//     several whole lines of C a row 2^20 x 48 -> 192 296 / 278, 2^22 x 64 -> 256 1365 / 1321; -> 100 180 / 210.
//   More, from 2^19 rows on: 2^17 x 128 -> 128 47 / 53, 2^19 150 / 148, 2^20 289 / 273, 100 -> 256 539 / 507, 128 -> 64 181 / 166,
//     96 -> 96 225 / 208; not a third step into ragged rows (90 -> 100 261 / 268), nor last tiles of a few columns (2^22 x 128 ->
//     130 1730 / 2006) or four steps into nearly whole ones (2 588 361 x 112 -> 117 759 / 801), nor up to 32 columns (2^20 x 300 ->
//     30 331 / 333).
bool kept_pays(int tb, int64_t M, int64_t N, int64_t K, int w, int steps) {
    const bool line = N % 32 == 0, half = N % 16 == 0, many = M >= 1 << 19;
    if (steps == 1) {
        if (M * N <= 1 << 25) return !(tb && K == 32 && w == 4);
        if (w < 4) return N <= 16 || K <= (half || w == 1 ? 16 : 12);
        return K <= 24 && (line || (half && M * N <= 5 << 24));
    }
    if (steps == 2) return w == 4 ? line && N > 128 && many : M <= (w == 2 ? 1 << 16 : K > 48 ? 1 << 18 : 1 << 19);
    if (w == 1 || !many) return false;
    return line || (w == 2 ? steps > 3 : N % 128 >= 32 && steps > (N % 128 < 96 ? 3 : 4));
}

// Wavefronts of a block that keeps the parts of its columns, or 0 where blocks pass them through LDS.
int kept_waves_per_block(int tb, int64_t M, int64_t N, int64_t K, int w, int steps) {
    if (!kept_pays(tb, M, N, K, w, steps)) return 0;
    const size_t room = 160 * 1024, own = 4096;            // a block's scales and ranges: at most 2 KB
    const int64_t tiles_n = ceil_div(N, 32 * w);
    for (int kept : {4, w == 1 ? 4 : 12}) {                // what the launch has
        const int on_cu = kept_waves(w) / kept;
        if (((size_t)w * steps * kStepBytes + own) * on_cu <= room && tiles_n <= 32 * on_cu) return kept;
    }
    return 0;
}

int64_t split_blocks(int64_t M, int64_t N) { return 8 * ceil_div(ceil_div(M, 128) * ceil_div(N, 32 * tiles_wide(N)), 8); }

}  // namespace

// a grid has less than 2^32 threads
bool gemm_split_fits(int64_t M, int64_t N) { return split_blocks(M, N) < (int64_t)1 << 24; }

// scratch of one operand pair: the parts of B, then a Range per 32 columns
size_t gemm_split_workspace_bytes(int64_t N, int64_t K) {
    return parts_bytes(N, K) + align_up((size_t)(ceil_div(N, 32) + 3) * sizeof(Range));
}

// C [M][N], rows ldc apart = A [M][K] op(B) (+ A2 op(B2)), K >= 4 and gemm_split_fits; tb: B is [N][K], else
// [K][N].  workspace: gemm_split_workspace_bytes per operand pair.
gnn_status_t gemm_split_launch(int tb, int64_t M, int64_t N, int64_t K, const float *A, const float *B, float *C,
                               int64_t ldc, const float *bias, int act, void *workspace, hipStream_t st,
                               const float *A2, const float *B2, const uint16_t *a_bits) {
    Product g{};
    g.M = (int)M; g.N = (int)N; g.K = (int)K;
    g.steps = (int)ceil_div(K, KB);
    g.A = A; g.A2 = A2;
    g.B = Operand{B, tb ? 1 : (long)N, tb ? (long)K : 1};
    g.B2 = Operand{B2, g.B.sk, g.B.sn};
    g.C = C; g.ldc = (int)ldc; g.bias = bias; g.act = act;
    g.a_bits = a_bits; g.bit_words = (int)ceil_div(K, 16); g.bit_stride = 2 * ((g.bit_words + 1) / 2 | 1);
    const int w = tiles_wide(N);
    g.tiles_m = (int)ceil_div(M, 128); g.tiles_n = (int)ceil_div(N, 32 * w);
    const size_t one = gemm_split_workspace_bytes(N, K), words = parts_bytes(N, K);
    char *ws = static_cast<char *>(workspace), *ws2 = ws + one;
    g.parts = ws; g.parts2 = ws2;
    Range *range = reinterpret_cast<Range *>(ws + words), *range2 = reinterpret_cast<Range *>(ws2 + words);
    g.range = range; g.range2 = range2;
    const int steps = A2 ? 2 * g.steps : g.steps, kept = a_bits ? 0 : kept_waves_per_block(tb, M, N, K, w, steps);
    if (kept) {
        const int64_t per_xcd = ceil_div(ceil_div(M, 32), 8);
        int64_t groups = 32 * (kept_waves(w) / kept) / g.tiles_n;      // blocks of an XCD that share a column tile
        if (groups > ceil_div(per_xcd, kept)) groups = ceil_div(per_xcd, kept);
        const dim3 grid((unsigned)(8 * groups * g.tiles_n));
        const size_t lds = (size_t)w * steps * kStepBytes;
        bool launched = false;
#define KEPT_CASE(NT_, KEPT_)                                                                              \
        if (w == NT_ && kept == KEPT_) {                                                                   \
            hipLaunchKernelGGL((gemm_split_kernel<NT_, false, KEPT_>), grid, dim3(64 * KEPT_), lds, st, g);  \
            launched = true;                                                                               \
        }
        KEPT_CASE(1, 4) KEPT_CASE(2, 4) KEPT_CASE(2, 12) KEPT_CASE(4, 4) KEPT_CASE(4, 12)
#undef KEPT_CASE
        return launched ? launch_status() : GNN_ERR_UNSUPPORTED;
    }
    hipLaunchKernelGGL(split_weights_kernel, dim3((unsigned)(g.tiles_n * w), A2 ? 2 : 1), dim3(1024), 0, st, (int)N,
                       (int)K, g.steps, g.B, g.B2, ws, ws2, range, range2);
    GNN_TRY(launch_status());
    const dim3 grid((unsigned)split_blocks(M, N));
    const size_t lds = (size_t)2 * w * kStepBytes + (a_bits ? (size_t)128 * g.bit_stride * sizeof(uint16_t) : 0);
    auto kernel = w == 1   ? (a_bits ? gemm_split_kernel<1, true, 0> : gemm_split_kernel<1, false, 0>)
                  : w == 2 ? (a_bits ? gemm_split_kernel<2, true, 0> : gemm_split_kernel<2, false, 0>)
                           : (a_bits ? gemm_split_kernel<4, true, 0> : gemm_split_kernel<4, false, 0>);
    hipLaunchKernelGGL(kernel, grid, dim3(256), lds, st, g);
    return launch_status();
}

}  // namespace gnn
