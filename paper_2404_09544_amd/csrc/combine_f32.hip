// Eq. 1 Combine in fp32 for many rows, on the fp16 matrix cores with fp32
// rounding: both operands as two fp16 parts, three part products per fp32
// product (the error-corrected scheme of Ootomo and Yokota, "Recovering single
// precision accuracy from Tensor Cores while surpassing the FP32 theoretical
// peak performance", 2022).
//
// A scaled value y is h + 2^-11 l with h = RN16(y) and l = RN16(2^11 (y - h));
// the products h h' go to one fp32 accumulator, h l' and l h' to a second one
// that joins it at the end, times 2^-11.  fp16 has five exponent bits, so
// values are scaled by powers of two first (exact): every weight column by its
// own maximum, the rows of a workgroup's tile by one scale, from the maximum of
// four of them.  Where y lies within [2^-13, 65504], 29 powers of two, its parts
// miss at most 2^-23 of it, and the product left out, l l', is below 2^-22 of
// the term.  Every term is held to that, about the bound of the six products of
// three bf16 parts (bf16split.hpp; theirs leave out 2^-22 twice):
//   - values of a row outside of that range (zero counts as inside) are taken
//     out and put on a list, and their products with their rows of W added in
//     fp32 at the end;
//   - a tile that meets more than kListMax of them, or whose columns hold such
//     a weight, is taken with the six products instead, in the same workgroup;
//     it gives up at the end of the step that shows it.
// The scale cancels exactly, so inside the range a row's bits do not depend on
// the rows around it; which of the three ways a value takes does.
//
// Relative error against 64 bits of normal data, whole output: 1,204-deep sums
// 2.4e-7 (six products 5.4e-7: their six sums a step round twice as often),
// 400-deep 1.5e-7 (3.0e-7), 80-deep 1.1e-7 (1.7e-7).
//
// Structure: a workgroup owns 32 TM WM rows and 32 WN columns.  Four
// wavefronts bring the rows, global -> registers three steps of 64 k ahead,
// split them once per workgroup and store two fp16 planes in one of three LDS
// stages; eight wavefronts multiply.  The weights, split and laid out as
// fragments beforehand (k_split_weights), go straight from L2 into the
// multiplying wavefronts' registers one step ahead, 1 KB contiguous per
// fragment, and never touch LDS.  Kept apart, the two kinds of loads do not
// wait for each other (loads return in order within a wavefront) and the
// splitting runs beside the matrix cores.  The product is taken transposed
// (weights as the A operand) so a lane stores four consecutive columns at a
// time.
//
// Measured (us, with the weights' launch; k_combine_split with its own):
// 20,902 x 1,204 x 256 97 -> 60, 13,720 rows 73 -> 44, 66,000 x 400 x 256 114 -> 81,
// 107,000 x 256 x 256 100 -> 88, 6,761 x 512 x 256 27.5 -> 18.7.  What is left at
// 20,902 rows: the products alone, without loads, take 45 us at the clock the
// matrix cores hold; the weights' launch 6.  Data that needs the list (one column
// 2^10 times the rest) 64, tiles that all take six products (2^20 and more) 94,
// 66,000 x 400 x 256 134 (113).
#include <algorithm>
#include <type_traits>

#include "bf16split.hpp"
#include "common.hpp"

namespace gnnav {

namespace {

typedef float f32x16c __attribute__((ext_vector_type(16)));
typedef float f32x4c __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4c __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2c __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));

constexpr int kStep = 64;           // k per step
constexpr int kFrags = kStep / 16;  // MFMA k steps per step

// The exponents that scales bring maxima to: the rows' leaves room for rows
// the scale was not taken from; a column's is exact.
constexpr int kRowExp = 13, kColExp = 14;

// A scaled value in [kSmallest, kLargest] has both parts to 2^-23 of it: h and
// the low part, kept times 2^11, are normal fp16 numbers or, where the low part
// is subnormal, its spacing of 2^-24 lies 2^-35 below h's.
constexpr float kSmallest = 0x1p-13f, kLargest = 65504.f, kLowScale = 2048.f;
constexpr int kListMax = 32;   // values outside of it that a tile takes one by one

// 2^(target - floor(log2 m)) and its inverse for a positive finite m (1 and 1
// otherwise), both kept normal numbers.
__device__ __forceinline__ void scale_of(float m, int target, float &scale, float &inv) {
    const int e = (int)((__float_as_uint(m) >> 23) & 255u);
    int f = m == 0.f || e == 255 ? 127 : 254 + target - e;
    f = f > 253 ? 253 : f;
    scale = __uint_as_float((uint32_t)f << 23);
    inv = __uint_as_float((uint32_t)(254 - f) << 23);
}

__device__ __forceinline__ void split2(float y, _Float16 &hi, _Float16 &lo) {
    hi = (_Float16)y;
    lo = (_Float16)__builtin_fmaf((float)hi, -kLowScale, y * kLowScale);   // exact before its rounding
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, kWave));
    return v;
}

}  // namespace

// The weights as fragments: for column group g (32 columns), k step s (16 k;
// each segment's K padded with zeros to a multiple of 64) and plane p, lane l
// = (h, c) holds k = 16 s + 8 h .. + 7 of column 32 g + c at
// [((g * steps + s) * planes + p) * 64 + l], 16 bytes.  Two scaled fp16 planes
// and three unscaled bf16 ones; inv[n] undoes column n's scale.  A workgroup
// takes 8 columns: their maxima first, then the parts; outside[b] tells whether
// a weight of workgroup b's columns lies outside of the fp16 parts' range.
constexpr int kSplitThreads = 1024;
constexpr int kSplitItems = 4;   // fragments a thread keeps between the two passes (d_in up to 2,048)

__global__ void __launch_bounds__(kSplitThreads) k_split_weights(const float *__restrict__ W, int32_t K, int32_t N,
                                                                 int32_t kt, u32x4c *__restrict__ half_planes,
                                                                 u32x4c *__restrict__ bf_planes,
                                                                 float *__restrict__ inv, int32_t *__restrict__ outside) {
    constexpr int NW = kSplitThreads / kWave, PER = kSplitThreads / 8;
    __shared__ float part[NW][8];
    __shared__ int s_outside;
    const int tid = threadIdx.x, c = tid & 7, lane = tid & 63, wid = tid >> 6;
    const int32_t n = blockIdx.x * 8 + c, nn = n < N ? n : N - 1;
    const int32_t steps = 2 * kt * kFrags;
    // item i of a column: k step i / 2, half i % 2; 8 k values, zeros past K or N
    auto load = [&](int32_t i, float (&x)[8]) {
        const int32_t s = i >> 1, seg = s >= kt * kFrags, k0 = (seg ? s - kt * kFrags : s) * 16 + 8 * (i & 1);
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = W[((int64_t)(seg ? K : 0) + (k0 + e < K ? k0 + e : 0)) * N + nn];
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (k0 + e >= K || n >= N) x[e] = 0.f;
    };
    float kept[kSplitItems][8];
    float mx = 0.f;
#pragma unroll
    for (int q = 0; q < kSplitItems; ++q) {
        const int32_t i = (tid >> 3) + q * PER;
        if (i < 2 * steps) load(i, kept[q]);
        else
#pragma unroll
            for (int e = 0; e < 8; ++e) kept[q][e] = 0.f;
    }
#pragma unroll
    for (int q = 0; q < kSplitItems; ++q)
#pragma unroll
        for (int e = 0; e < 8; ++e) mx = fmaxf(mx, fabsf(kept[q][e]));
    for (int32_t i = (tid >> 3) + kSplitItems * PER; i < 2 * steps; i += PER) {
        float x[8];
        load(i, x);
#pragma unroll
        for (int e = 0; e < 8; ++e) mx = fmaxf(mx, fabsf(x[e]));
    }
#pragma unroll
    for (int o = 8; o < kWave; o <<= 1) mx = fmaxf(mx, __shfl_xor(mx, o, kWave));
    if (lane < 8) part[wid][lane] = mx;
    if (tid == 0) s_outside = 0;
    __syncthreads();
    mx = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) mx = fmaxf(mx, part[w][c]);
    float scale, back;
    scale_of(mx, kColExp, scale, back);
    if (tid < 8) inv[n] = back;
    bool out = false;
    auto store = [&](int32_t i, const float (&x)[8]) {
        f16x8 hi, lo;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float y = x[e] * scale;
            out = out || (x[e] != 0.f && !(fabsf(y) >= kSmallest && fabsf(y) <= kLargest));
            _Float16 a, b;
            split2(y, a, b);
            hi[e] = a;
            lo[e] = b;
        }
        bf16x8 p1, p2, p3;
        split3(x, p1, p2, p3);
        const int64_t f = (int64_t)(n >> 5) * steps + (i >> 1);
        const int l = (i & 1) * 32 + (n & 31);
        half_planes[(f * 2 + 0) * 64 + l] = __builtin_bit_cast(u32x4c, hi);
        half_planes[(f * 2 + 1) * 64 + l] = __builtin_bit_cast(u32x4c, lo);
        bf_planes[(f * 3 + 0) * 64 + l] = __builtin_bit_cast(u32x4c, p1);
        bf_planes[(f * 3 + 1) * 64 + l] = __builtin_bit_cast(u32x4c, p2);
        bf_planes[(f * 3 + 2) * 64 + l] = __builtin_bit_cast(u32x4c, p3);
    };
#pragma unroll
    for (int q = 0; q < kSplitItems; ++q) {
        const int32_t i = (tid >> 3) + q * PER;
        if (i < 2 * steps) store(i, kept[q]);
    }
    for (int32_t i = (tid >> 3) + kSplitItems * PER; i < 2 * steps; i += PER) {
        float x[8];
        load(i, x);
        store(i, x);
    }
    if (out) s_outside = 1;
    __syncthreads();
    if (tid == 0) outside[blockIdx.x] = s_outside;
}

constexpr int kMulWaves = 8, kRowWaves = 4;   // wavefronts that multiply, wavefronts that bring rows
constexpr int kRowThreads = 64 * kRowWaves;
constexpr int kSampled = 4;   // rows of a tile that its scale is taken from

// A value outside of the parts' range: row of the tile, row of W, the value.
struct Outlier {
    int32_t row, k;
    float x;
};

// LDS of a workgroup with tiles of BM rows.
template <int BM>
struct F32Shared {
    u32x4c stages[9 * BM * 8];   // three stages of two planes (six products: of three)
    float max[kRowWaves];
    Outlier list[kListMax];
    int count;     // outliers met so far
    int over[3];   // too many: [2] before the first step, [t & 1] in step t, read after its barrier
};

struct F32Args {
    const float *A0;
    int64_t lda0;
    const float *A1;
    int64_t lda1;
    int64_t M;
    const int32_t *m_dev;
    int32_t K, kt;
    const float *W;
    const u32x4c *half_planes, *bf_planes;
    const float *inv;
    const int32_t *outside;
    int32_t N;
    int relu, vec;
    float *C;
    int64_t ldc;
};

// One workgroup's tile: rows from blockIdx.x * 32 TM WM on, of M.
template <int TM, int WM, int WN>
__device__ __forceinline__ void combine_f32_tile(const F32Args &a, int64_t M, F32Shared<32 * TM * WM> &sh) {
    static_assert(WM * WN == kMulWaves, "wavefront grid");
    constexpr int BM = 32 * TM * WM, AJ = BM / 16;   // a row thread loads AJ float4 of a step
    constexpr int PL = BM * 8;                       // 16-byte chunks of one plane of a stage
    const float *__restrict__ A0 = a.A0, *__restrict__ A1 = a.A1, *__restrict__ W = a.W, *__restrict__ inv = a.inv;
    const u32x4c *__restrict__ half_planes = a.half_planes, *__restrict__ bf_planes = a.bf_planes;
    const int32_t *__restrict__ outside = a.outside;
    float *__restrict__ C = a.C;
    const int64_t lda0 = a.lda0, lda1 = a.lda1, ldc = a.ldc;
    const int32_t K = a.K, kt = a.kt, N = a.N;
    const int relu = a.relu, vec = a.vec;
    u32x4c *S = sh.stages;
    float *s_max = sh.max;
    Outlier *s_list = sh.list;
    int &s_count = sh.count;
    int *s_over = sh.over;
    const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t m0 = (int64_t)blockIdx.x * BM;
    if (m0 >= M) return;
    const int32_t T = 2 * kt, steps = T * kFrags;
    // 16-byte chunk (row, c) of a plane sits at c ^ ((row >> 1) & 7): 16
    // consecutive rows' fragment reads touch 16 distinct bank groups
    auto chunk = [](int row, int c) { return row * 8 + (c ^ ((row >> 1) & 7)); };

    if (wid >= kMulWaves) {
        // ---- rows: thread (r, c) = (id / 16, id % 16) loads k = 4 c .. 4 c + 3
        // of rows r, r + 16, ... of a step, three steps ahead
        const int id = tid - 64 * kMulWaves, c4 = id & 15, r0 = id >> 4;
        auto load = [&](int32_t t, f32x4c (&x)[AJ]) {
            // rows' addresses are formed for each load: kept from load to load
            // they would not fit the registers beside three steps' rows
            int from = r0;
            if (AJ > 6) asm volatile("" : "+v"(from));
            t = t < T ? t : T - 1;
            const int seg = t >= kt;
            const int32_t k = (seg ? t - kt : t) * kStep + 4 * c4;
            const float *A = (seg ? A1 : A0) + (k < K ? k : 0);
            const int64_t lda = seg ? lda1 : lda0;
#pragma unroll
            for (int j = 0; j < AJ; ++j) {
                const int64_t row = m0 + from + 16 * j;
                x[j] = *(const f32x4c *)(A + (row < M ? row : M - 1) * lda);
            }
        };
        auto mask = [&](int32_t t, f32x4c (&x)[AJ]) {   // zeros at k >= K
            const int32_t k = (t >= kt ? t - kt : t) * kStep + 4 * c4;
            if (k - 4 * c4 + kStep <= K) return;
#pragma unroll
            for (int j = 0; j < AJ; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) x[j][e] = k + e < K ? x[j][e] : 0.f;
        };
        // the tile's scale, from rows spread over it
        if (id < 3) s_over[id] = 0;
        if (id == 0) s_count = 0;
        float mx = 0.f;
        for (int32_t k = id; k < K; k += kRowThreads)
#pragma unroll
            for (int j = 0; j < kSampled; ++j) {
                const int64_t row = m0 + j * (BM / kSampled) < M ? m0 + j * (BM / kSampled) : M - 1;
                mx = fmaxf(mx, fmaxf(fabsf(A0[row * lda0 + k]), fabsf(A1[row * lda1 + k])));
            }
        f32x4c x0[AJ], x1[AJ], x2[AJ];
        load(0, x0);
        load(1, x1);
        load(2, x2);
        mx = wave_max(mx);
        if (lane == 0) s_max[wid - kMulWaves] = mx;
        __syncthreads();
        mx = fmaxf(fmaxf(s_max[0], s_max[1]), fmaxf(s_max[2], s_max[3]));
        float scale, back;
        scale_of(mx, kRowExp, scale, back);
        // the range of unscaled values (kSmallest / scale may be subnormal, but
        // never zero); twice the bits less one orders magnitudes with 0 on top
        const uint32_t least = (__float_as_uint(kSmallest * back) << 1) - 1u;
        const float most = kLargest * back;

        // columns with weights out of range: six products from the start
        const int32_t blk = (int32_t)blockIdx.y * (4 * WN) + id;
        if (id < 4 * WN && blk < (N + 7) / 8 && outside[blk]) s_over[2] = 1;

        auto outlier = [&](float v) { return (__float_as_uint(v) << 1) - 1u < least || fabsf(v) > most; };
        auto split = [&](int32_t t, f32x4c (&x)[AJ]) {
            mask(t, x);
            uint32_t lo_seen = ~0u;
            float hi_seen = 0.f;
#pragma unroll
            for (int j = 0; j < AJ; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    lo_seen = min(lo_seen, (__float_as_uint(x[j][e]) << 1) - 1u);
                    hi_seen = fmaxf(hi_seen, fabsf(x[j][e]));
                }
            if (lo_seen < least || hi_seen > most) {   // rare: such values leave the parts and go to the list
#pragma unroll
                for (int j = 0; j < AJ; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float v = x[j][e];
                        if (!outlier(v)) continue;
                        x[j][e] = 0.f;
                        if (m0 + r0 + 16 * j >= M) continue;
                        const int at = atomicAdd(&s_count, 1);
                        const int32_t k = (t >= kt ? K + (t - kt) * kStep : t * kStep) + 4 * c4 + e;
                        if (at < kListMax) s_list[at] = Outlier{r0 + 16 * j, k, v};
                        else s_over[t < 2 ? 2 : t & 1] = 1;
                    }
            }
            u32x2c *st = (u32x2c *)(S + t % 3 * 2 * PL);
#pragma unroll
            for (int j = 0; j < AJ; ++j) {
                f16x4 hi, lo;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    _Float16 a, b;
                    split2(x[j][e] * scale, a, b);
                    hi[e] = a;
                    lo[e] = b;
                }
                const int at = 2 * chunk(r0 + 16 * j, c4 >> 1) + (c4 & 1);
                st[at] = __builtin_bit_cast(u32x2c, hi);
                st[2 * PL + at] = __builtin_bit_cast(u32x2c, lo);
            }
        };
        // while step t is multiplied, step t + 2 is split; true: there were too many
        auto pass = [&](auto &&put, auto checked) {
            auto over = [&](int i) { return decltype(checked)::value && __builtin_amdgcn_readfirstlane(s_over[i]) != 0; };
            put(0, x0);
            load(3, x0);
            put(1, x1);   // T is at least 2
            load(4, x1);
            __syncthreads();
            if (over(2)) return true;
            for (int32_t t = 0;; t += 3) {
                if (t + 2 < T) put(t + 2, x2);
                load(t + 5, x2);
                __syncthreads();
                if (over(t & 1)) return true;
                if (t + 1 >= T) return false;
                if (t + 3 < T) put(t + 3, x0);
                load(t + 6, x0);
                __syncthreads();
                if (over((t + 1) & 1)) return true;
                if (t + 2 >= T) return false;
                if (t + 4 < T) put(t + 4, x1);
                load(t + 7, x1);
                __syncthreads();
                if (over(t & 1)) return true;
                if (t + 3 >= T) return false;
            }
        };
        if (!pass(split, std::true_type())) return;
        // the tile again, with three bf16 parts
        auto split_bf = [&](int32_t t, f32x4c (&x)[AJ]) {
            mask(t, x);
            u32x2c *st = (u32x2c *)(S + t % 3 * 3 * PL);
#pragma unroll
            for (int j = 0; j < AJ; ++j) {
                uint16_t q[3][4];
#pragma unroll
                for (int e = 0; e < 4; ++e) split3_bits(x[j][e], q[0][e], q[1][e], q[2][e]);
                const int at = 2 * chunk(r0 + 16 * j, c4 >> 1) + (c4 & 1);
#pragma unroll
                for (int p = 0; p < 3; ++p)
                    st[2 * p * PL + at] = u32x2c{(uint32_t)q[p][0] | ((uint32_t)q[p][1] << 16),
                                                 (uint32_t)q[p][2] | ((uint32_t)q[p][3] << 16)};
            }
        };
        load(0, x0);
        load(1, x1);
        load(2, x2);
        pass(split_bf, std::false_type());
        return;
    }

    // ---- products
    const int wm = wid / WN, wn = wid % WN, h = lane >> 5, lr = lane & 31;
    // column group; a wavefront past the last one repeats it and stores nothing
    // (no branches around loads, so that their waits can be counted)
    const int32_t groups = (N + 31) / 32, gw = (int32_t)blockIdx.y * WN + wn, g = gw < groups ? gw : groups - 1;
    const u32x4c *bh = half_planes + (int64_t)g * steps * 128 + lane;
    f16x8 w[kFrags][2];
    auto load_w = [&](int32_t t, int u) {
#pragma unroll
        for (int p = 0; p < 2; ++p)
            w[u][p] = __builtin_bit_cast(f16x8, bh[(int64_t)t * (kFrags * 128) + (u * 2 + p) * 64]);
    };
#pragma unroll
    for (int u = 0; u < kFrags; ++u) load_w(0, u);
    f32x16c acc[TM], low[TM];   // high times high; the two products with a low part, 2^11 times
#pragma unroll
    for (int m = 0; m < TM; ++m)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[m][r] = low[m][r] = 0.f;
    __syncthreads();
    const float mx = fmaxf(fmaxf(s_max[0], s_max[1]), fmaxf(s_max[2], s_max[3]));
    float scale, back;
    scale_of(mx, kRowExp, scale, back);
    __syncthreads();
    // A step's 16 k take three products a block; the next 16 k's high parts are
    // read before the last of them and its low parts after it, each into the
    // registers just used (two sets would not fit), across the step's end too:
    // the next step's stage was complete a barrier ago.  The order is fixed by
    // scheduling barriers: the compiler's own put reads right before their use.
    f16x8 ah[TM], al[TM];
    auto fetch = [&](f16x8 (&f)[TM], const u32x4c *st, int u) {
#pragma unroll
        for (int m = 0; m < TM; ++m) f[m] = __builtin_bit_cast(f16x8, st[chunk((wm * TM + m) * 32 + lr, 2 * u + h)]);
    };
    fetch(ah, S, 0);
    fetch(al, S + PL, 0);
    int32_t stage = 0;
    // (read as scalars: both outcomes' registers are not needed at once)
    bool redo = __builtin_amdgcn_readfirstlane(s_over[2]) != 0;
    for (int32_t t = 0; t < T && !redo; ++t) {
        const u32x4c *st = S + stage * 2 * PL;
        stage = stage == 2 ? 0 : stage + 1;
        const u32x4c *next = S + stage * 2 * PL;   // (after the last step: read, not used)
        const int32_t tn = t + 1 < T ? t + 1 : t;
#pragma unroll
        for (int u = 0; u < kFrags; ++u) {
            const u32x4c *from = u + 1 < kFrags ? st : next;
            const int un = (u + 1) % kFrags;
#pragma unroll
            for (int m = 0; m < TM; ++m) low[m] = __builtin_amdgcn_mfma_f32_32x32x16_f16(w[u][1], ah[m], low[m], 0, 0, 0);
#pragma unroll
            for (int m = 0; m < TM; ++m) acc[m] = __builtin_amdgcn_mfma_f32_32x32x16_f16(w[u][0], ah[m], acc[m], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            fetch(ah, from, un);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int m = 0; m < TM; ++m) low[m] = __builtin_amdgcn_mfma_f32_32x32x16_f16(w[u][0], al[m], low[m], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            fetch(al, from + PL, un);
            load_w(tn, u);   // a whole step ahead of its use, into the registers just used
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
        redo = __builtin_amdgcn_readfirstlane(s_over[t & 1]) != 0;
    }
#pragma unroll
    for (int m = 0; m < TM; ++m)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[m][r] += low[m][r] * (1.f / kLowScale);
    if (redo) {   // six products of three bf16 parts
#pragma unroll
        for (int m = 0; m < TM; ++m)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[m][r] = 0.f;
        const u32x4c *bb = bf_planes + (int64_t)g * steps * 192 + lane;
        bf16x8 b[2][3], r1[TM], r2[TM], r3[TM];
        auto load_b = [&](int32_t i, bf16x8 (&f)[3]) {   // 16 k, one ahead of their use
            i = i < steps ? i : steps - 1;
#pragma unroll
            for (int p = 0; p < 3; ++p) f[p] = __builtin_bit_cast(bf16x8, bb[(int64_t)i * 192 + p * 64]);
        };
        auto fetch_b = [&](bf16x8 (&f)[TM], const u32x4c *st, int u) {
#pragma unroll
            for (int m = 0; m < TM; ++m) f[m] = __builtin_bit_cast(bf16x8, st[chunk((wm * TM + m) * 32 + lr, 2 * u + h)]);
        };
        auto mul = [&](const bf16x8 &x, const bf16x8 (&y)[TM]) {
#pragma unroll
            for (int m = 0; m < TM; ++m) acc[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, y[m], acc[m], 0, 0, 0);
        };
        load_b(0, b[0]);
        __syncthreads();
        fetch_b(r3, S + 2 * PL, 0);
        fetch_b(r2, S + PL, 0);
        fetch_b(r1, S, 0);
        stage = 0;
        for (int32_t t = 0; t < T; ++t) {
            const u32x4c *st = S + stage * 3 * PL;
            stage = stage == 2 ? 0 : stage + 1;
            const u32x4c *next = S + stage * 3 * PL;
#pragma unroll
            for (int u = 0; u < kFrags; ++u) {
                const u32x4c *from = u + 1 < kFrags ? st : next;
                const int un = (u + 1) % kFrags;
                const bf16x8(&c)[3] = b[u & 1];
                load_b(t * kFrags + u + 1, b[(u + 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);
                mul(c[0], r3);
                __builtin_amdgcn_sched_barrier(0);
                fetch_b(r3, from + 2 * PL, un);
                mul(c[1], r2);
                mul(c[0], r2);
                __builtin_amdgcn_sched_barrier(0);
                fetch_b(r2, from + PL, un);
                mul(c[2], r1);
                mul(c[1], r1);
                mul(c[0], r1);
                __builtin_amdgcn_sched_barrier(0);
                fetch_b(r1, from, un);
            }
            __syncthreads();
        }
    }
    // acc[m][4 q + e]: row lr of block m, column 8 q + 4 h + e of the group
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const f32x4c s = *(const f32x4c *)(inv + g * 32 + 8 * q + 4 * h);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            // both scales at once: one after the other could leave fp32's range on the way
            const int exp = redo ? 0 : (int)(__float_as_uint(back) >> 23) + (int)(__float_as_uint(s[e]) >> 23) - 254;
#pragma unroll
            for (int m = 0; m < TM; ++m) acc[m][4 * q + e] = ldexpf(acc[m][4 * q + e], exp);
        }
    }
    const int n_list = redo ? 0 : __builtin_amdgcn_readfirstlane(s_count);
    if (n_list > 0) {
        // the list's values, each with its row of W, in fp32; in the order of
        // their places, so that the sum does not depend on who came first
        Outlier o{INT_MAX, INT_MAX, 0.f};
        if (lane < n_list) o = s_list[lane];
        int rank = 0;
        for (int i = 0; i < n_list; ++i) {
            const Outlier p = s_list[i];
            rank += p.row < o.row || (p.row == o.row && p.k < o.k);
        }
        rank = lane < n_list ? rank : lane;
        const int row_s = __builtin_amdgcn_ds_permute(4 * rank, o.row);
        const int k_s = __builtin_amdgcn_ds_permute(4 * rank, o.k);
        const int x_s = __builtin_amdgcn_ds_permute(4 * rank, __builtin_bit_cast(int, o.x));
        // their rows of W, 32 columns each, all on the way together, then
        // through this wavefront's share of the stages (no longer read)
        static_assert(kMulWaves * kListMax * 32 * sizeof(float) <= sizeof(sh.stages), "the list's weights fit the stages");
        float *wl = (float *)S + wid * (kListMax * 32);
        const int32_t col = g * 32 + lr < N ? g * 32 + lr : N - 1;
        float v[kListMax / 2];
#pragma unroll
        for (int q = 0; q < kListMax / 2; ++q) {
            const int k = __shfl(k_s, 2 * q + h, kWave);
            v[q] = 2 * q + h < n_list ? W[(int64_t)k * N + col] : 0.f;
        }
#pragma unroll
        for (int q = 0; q < kListMax / 2; ++q) wl[(2 * q + h) * 32 + lr] = v[q];
        for (int i = 0; i < n_list; ++i) {
            const int row = __builtin_amdgcn_readlane(row_s, i);
            const float x = __builtin_bit_cast(float, __builtin_amdgcn_readlane(x_s, i));
#pragma unroll
            for (int m = 0; m < TM; ++m) {
                if (row >> 5 != wm * TM + m || lr != (row & 31)) continue;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f32x4c y = *(const f32x4c *)&wl[i * 32 + 8 * q + 4 * h];
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[m][4 * q + e] = fmaf(x, y[e], acc[m][4 * q + e]);
                }
            }
        }
    }
    if (gw >= groups) return;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int32_t n = g * 32 + 8 * q + 4 * h;
#pragma unroll
        for (int m = 0; m < TM; ++m) {
            const int64_t row = m0 + (wm * TM + m) * 32 + lr;
            if (row >= M) continue;
            f32x4c v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = relu ? fmaxf(acc[m][4 * q + e], 0.f) : acc[m][4 * q + e];
            float *o = C + row * ldc + n;
            if (vec && n + 4 <= N) {
                *(f32x4c *)o = v;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (n + e < N) o[e] = v[e];
            }
        }
    }
}

template <int TM, int WM, int WN>
__global__ void __launch_bounds__(64 * (kMulWaves + kRowWaves)) k_combine_f32(F32Args a) {
    __shared__ F32Shared<32 * TM * WM> sh;
    combine_f32_tile<TM, WM, WN>(a, a.m_dev ? *a.m_dev : a.M, sh);
}

// Rows of 32 on the busiest of `units` compute units (one workgroup each at a
// time) with tiles of 32 blocks rows and `groups` column groups, half a
// block's work of overhead a workgroup.
__host__ __device__ inline int64_t f32_cost(int64_t m, int blocks, int64_t groups, int64_t units) {
    const int64_t wgs = (m + 32 * blocks - 1) / (32 * blocks) * groups;
    return (wgs + units - 1) / units * (2 * blocks + 1);
}

// The same for a row count on the device, with its tile height, 64 or 96 rows,
// by the count and not by its bound: a sampled frontier's 20,900 rows under a
// bound of 26,624 took 82 us in the two rounds of the bound's 64-row tiles.
__global__ void __launch_bounds__(64 * (kMulWaves + kRowWaves)) k_combine_f32_counted(F32Args a, int32_t units) {
    __shared__ F32Shared<96> sh;
    const int64_t M = *a.m_dev;
    if (f32_cost(M, 2, gridDim.y, units) < f32_cost(M, 3, gridDim.y, units))
        combine_f32_tile<2, 1, 8>(a, M, (F32Shared<64> &)sh);
    else
        combine_f32_tile<3, 1, 8>(a, M, sh);
}

namespace {
// k steps of 64 per segment; columns padded to the 32 WN of a workgroup
int64_t f32_kt(int64_t d_in) { return (d_in + kStep - 1) / kStep; }
int64_t f32_cols(int64_t d_out) { return (d_out + 255) / 256 * 256; }
}  // namespace

// Where k_combine_f32 beats k_combine_split, measured over d_in 16 .. 602, d_out
// 32 .. 700 and 2,600 .. 500,000 rows (us, k_combine_split first).  It takes
// whole groups of 256 columns, one workgroup per compute unit and 64 k a step:
//   d_in <= 64: 100,000 x 32 x 32 20 against 36, 66,000 x 64 x 384 63 against 71,
//     at best 20,900 x 64 x 256 25 against 21;
//   d_out <= 64: 100,000 x 200 x 64 62 against 85, at best 50.6 against 46.4;
//   d_out <= 128 in one round of tiles (128 rows by 256 units) 1.1 to 1.4 times as
//     fast, in more rounds 0.8 to 1.1 times unless the rows are long;
//   d_out in (128, 256]: 1.1 to 1.6 times as fast everywhere (20,902 x 602 x 256 94
//     against 61, 100,000 x 100 x 256 100 against 89);
//   d_out > 256: 1.0 to 1.5 times where more than 3/4 of the groups' columns are
//     used or the rows are long, 0.8 to 1.4 times elsewhere.
// (By the whole chip's units on every stream, so that a call's bits do not depend
// on its stream's share.)
bool combine_f32_parts(int64_t m, int64_t d_in, int64_t d_out) {
    if (d_in <= 64 || d_out <= 64) return false;
    const bool long_rows = d_in > 256;
    if (d_out <= 128) return long_rows || m <= 256 * 128;
    return d_out <= 256 || long_rows || 4 * d_out > 3 * f32_cols(d_out);
}

size_t combine_f32_workspace(int64_t d_in, int64_t d_out) {
    const size_t values = (size_t)(f32_cols(d_out) * 2 * f32_kt(d_in) * kStep);
    return values * 2 * 5 + (size_t)f32_cols(d_out) * sizeof(float) + (size_t)f32_cols(d_out) / 8 * sizeof(int32_t);
}

void launch_split_weights(const float *w, int64_t d_in, int64_t d_out, void *ws, hipStream_t s) {
    const int64_t kt = f32_kt(d_in), nc = f32_cols(d_out), values = nc * 2 * kt * kStep;
    char *p = (char *)ws;
    hipLaunchKernelGGL(k_split_weights, dim3((unsigned)((d_out + 31) / 32 * 4)), dim3(kSplitThreads), 0, s, w, (int32_t)d_in,
                       (int32_t)d_out, (int32_t)kt, (u32x4c *)p, (u32x4c *)(p + 4 * values), (float *)(p + 10 * values),
                       (int32_t *)(p + 10 * values + 4 * nc));
    GNNAV_HIP(hipGetLastError());
}

void launch_combine_f32(const float *self, int64_t ld_self, const float *agg, int64_t ld_agg, int64_t m,
                        const int32_t *m_dev, int64_t d_in, const float *w, int64_t d_out, const void *ws, bool relu,
                        float *out, int64_t ld_out, hipStream_t s) {
    const int64_t kt = f32_kt(d_in), nc = f32_cols(d_out), values = nc * 2 * kt * kStep;
    const char *p = (const char *)ws;
    const int vec = ld_out % 4 == 0 && ((uintptr_t)out & 15u) == 0;
    const F32Args a{self, ld_self, agg, ld_agg, m, m_dev, (int32_t)d_in, (int32_t)kt, w, (const u32x4c *)p,
                    (const u32x4c *)(p + 4 * values), (const float *)(p + 10 * values),
                    (const int32_t *)(p + 10 * values + 4 * nc), (int32_t)d_out, (int)relu, vec, out, ld_out};
    const dim3 threads(64 * (kMulWaves + kRowWaves));
    auto grid = [&](int rows, int cols) { return dim3((unsigned)((m + rows - 1) / rows), (unsigned)((d_out + cols - 1) / cols)); };
    const int64_t units = stream_units(s);
    if (d_out > 128) {
        const int64_t groups = (d_out + 255) / 256;
        int best = 3;
        for (int b = 2; b >= 1; --b)
            if (f32_cost(m, b, groups, units) < f32_cost(m, best, groups, units)) best = b;
        if (best == 1)
            hipLaunchKernelGGL((k_combine_f32<1, 1, 8>), grid(32, 256), threads, 0, s, a);
        else if (m_dev)
            hipLaunchKernelGGL(k_combine_f32_counted, grid(64, 256), threads, 0, s, a, (int32_t)units);
        else if (best == 2)
            hipLaunchKernelGGL((k_combine_f32<2, 1, 8>), grid(64, 256), threads, 0, s, a);
        else
            hipLaunchKernelGGL((k_combine_f32<3, 1, 8>), grid(96, 256), threads, 0, s, a);
    } else {
        if (f32_cost(m, 2, 1, units) < f32_cost(m, 4, 1, units))
            hipLaunchKernelGGL((k_combine_f32<1, 2, 4>), grid(64, 128), threads, 0, s, a);
        else
            hipLaunchKernelGGL((k_combine_f32<2, 2, 4>), grid(128, 128), threads, 0, s, a);
    }
    GNNAV_HIP(hipGetLastError());
}

}  // namespace gnnav
