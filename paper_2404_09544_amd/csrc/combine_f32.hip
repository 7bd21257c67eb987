// Eq. 1 Combine in fp32 for many rows, on the fp16 matrix cores with fp32
// rounding: both operands as two fp16 parts, three part products per fp32
// product (the error-corrected scheme of Ootomo and Yokota, "Recovering single
// precision accuracy from Tensor Cores while surpassing the FP32 theoretical
// peak performance", 2022).
//
// A scaled value x = h + l + e with h = RN16(x) and l = RN16(x - h) has
// |e| <= 2^-23 |x| while l is a normal fp16 number, and the dropped product
// l l' is below 2^-22 |x x'| (rms 2^-24): both far below the rounding of a
// sum of tens of products in fp32, and three accumulations per 16 k instead
// of the six of a three-way bf16 split round half as often.  fp16 has five
// exponent bits, so the values are scaled by powers of two first (exact):
//   - every weight column by its own maximum;
//   - the rows of a workgroup's tile by one scale, from the maximum of two of
//     its rows, which leaves 16 times that maximum before fp16 overflows;
//   - while the tile is split, each row's maximum in each of the two segments
//     is tracked.  A row that overflowed, or whose maximum lies more than
//     about 2^12 below the scale's target (where its l parts turn subnormal),
//     sends the tile back through the three-way bf16 split (bf16split.hpp, six
//     products, bf16's full exponent range), in the same workgroup.
// Against 64 bits the rms row error is below that of the six-product scheme at
// every width from 16 up (1,204-deep sums of normal data 3.9e-7 against
// 5.0e-7, 32-deep 8.7e-8 against 9.2e-8) and within it where the fallback
// takes over.
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
// Measured (us, both with their weights launch; the six-product kernel before):
// 20,902 x 1,204 x 256 98.0 -> 62.4 (the kernel alone 89 -> 53, its weights
// 4.6 -> 5.9, no tail sum), 13,720 rows 84 -> 50, 66,000 x 200 x 256 85 -> 73,
// 6,761 x 256 x 256 20 -> 16; 12,000 x 128 x 41 and other launch-bound sizes
// within 1 us.  What is left at 20,902 rows: the products alone, without
// loads, take 45 us at the clock the matrix cores hold; rows add 10 us, the
// weights' L2 reads (64 KB a step and workgroup) nothing measurable.
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
// the scale was not taken from; a column's is exact and takes the top of
// fp16's range, which keeps the l parts of its small weights normal.
constexpr int kRowExp = 11, kColExp = 14;

// 2^(target - floor(log2 m)) and its inverse for a positive finite m (1 and 1
// otherwise), both kept normal numbers.
__device__ __forceinline__ void scale_of(float m, int target, float &scale, float &inv) {
    const int e = (int)((__float_as_uint(m) >> 23) & 255u);
    int f = m == 0.f || e == 255 ? 127 : 254 + target - e;
    f = f > 253 ? 253 : f;
    scale = __uint_as_float((uint32_t)f << 23);
    inv = __uint_as_float((uint32_t)(254 - f) << 23);
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, kWave));
    return v;
}

// Maximum over the 16 lanes of a DPP row, on every lane of it.
__device__ __forceinline__ float row16_max(float v) {
    v = fmaxf(v, __uint_as_float((uint32_t)__builtin_amdgcn_mov_dpp((int)__float_as_uint(v), 0xB1, 0xf, 0xf, true)));
    v = fmaxf(v, __uint_as_float((uint32_t)__builtin_amdgcn_mov_dpp((int)__float_as_uint(v), 0x4E, 0xf, 0xf, true)));
    v = fmaxf(v, __uint_as_float((uint32_t)__builtin_amdgcn_mov_dpp((int)__float_as_uint(v), 0x141, 0xf, 0xf, true)));
    v = fmaxf(v, __uint_as_float((uint32_t)__builtin_amdgcn_mov_dpp((int)__float_as_uint(v), 0x140, 0xf, 0xf, true)));
    return v;
}

}  // namespace

// The weights as fragments: for column group g (32 columns), k step s (16 k;
// each segment's K padded with zeros to a multiple of 64) and plane p, lane l
// = (h, c) holds k = 16 s + 8 h .. + 7 of column 32 g + c at
// [((g * steps + s) * planes + p) * 64 + l], 16 bytes.  Two scaled fp16 planes
// and three unscaled bf16 ones; inv[n] undoes column n's scale.  A workgroup
// takes 8 columns: their maxima first, then the parts.
constexpr int kSplitThreads = 1024;
constexpr int kSplitItems = 4;   // fragments a thread keeps between the two passes (d_in up to 2,048)

__global__ void __launch_bounds__(kSplitThreads) k_split_weights(const float *__restrict__ W, int32_t K, int32_t N,
                                                                 int32_t kt, u32x4c *__restrict__ half_planes,
                                                                 u32x4c *__restrict__ bf_planes,
                                                                 float *__restrict__ inv) {
    constexpr int NW = kSplitThreads / kWave, PER = kSplitThreads / 8;
    __shared__ float part[NW][8];
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
    __syncthreads();
    mx = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) mx = fmaxf(mx, part[w][c]);
    float scale, back;
    scale_of(mx, kColExp, scale, back);
    if (tid < 8) inv[n] = back;
    auto store = [&](int32_t i, const float (&x)[8]) {
        f16x8 hi, lo;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float y = x[e] * scale;
            hi[e] = (_Float16)y;
            lo[e] = (_Float16)(y - (float)hi[e]);
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
}

constexpr int kMulWaves = 8, kRowWaves = 4;   // wavefronts that multiply, wavefronts that bring rows
constexpr int kRowThreads = 64 * kRowWaves;
constexpr int kDepth = 3;                     // row steps in flight

// LL: the product of the low parts too (four part products), for sums so short
// (d_in <= 64) that its rms 2^-24 shows beside the sum's own rounding.
template <int TM, int WM, int WN, bool LL>
__global__ void __launch_bounds__(64 * (kMulWaves + kRowWaves))
    k_combine_f32(const float *__restrict__ A0, int64_t lda0, const float *__restrict__ A1, int64_t lda1, int64_t M,
                  const int32_t *__restrict__ m_dev, int32_t K, int32_t kt, const u32x4c *__restrict__ half_planes,
                  const u32x4c *__restrict__ bf_planes, const float *__restrict__ inv, int32_t N, int relu, int vec,
                  float *__restrict__ C, int64_t ldc) {
    static_assert(WM * WN == kMulWaves, "wavefront grid");
    constexpr int BM = 32 * TM * WM, AJ = BM / 16;   // a row thread loads AJ float4 of a step
    constexpr int PL = BM * 8;                       // 16-byte chunks of one plane of a stage
    __shared__ u32x4c S[6 * PL];                     // three stages of two planes (the fallback: one of three)
    __shared__ float s_max[kRowWaves];
    __shared__ int s_bad;
    const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (m_dev) M = *m_dev;
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
            t = t < T ? t : T - 1;
            const int seg = t >= kt;
            const int32_t k = (seg ? t - kt : t) * kStep + 4 * c4;
            const float *A = (seg ? A1 : A0) + (k < K ? k : 0);
            const int64_t lda = seg ? lda1 : lda0;
#pragma unroll
            for (int j = 0; j < AJ; ++j) {
                const int64_t row = m0 + r0 + 16 * j;
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
        // the tile's scale, from its first and middle rows
        if (id == 0) s_bad = 0;
        float mx = 0.f;
        const int64_t rb = m0 + BM / 2 < M ? m0 + BM / 2 : M - 1;
        for (int32_t k = id; k < K; k += kRowThreads)
            mx = fmaxf(mx, fmaxf(fmaxf(fabsf(A0[m0 * lda0 + k]), fabsf(A1[m0 * lda1 + k])),
                                 fmaxf(fabsf(A0[rb * lda0 + k]), fabsf(A1[rb * lda1 + k]))));
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

        float row_mx[AJ];
#pragma unroll
        for (int j = 0; j < AJ; ++j) row_mx[j] = 0.f;
        bool bad = false;
        auto split = [&](int32_t t, f32x4c (&x)[AJ]) {
            mask(t, x);
            u32x2c *st = (u32x2c *)(S + t % 3 * 2 * PL);
#pragma unroll
            for (int j = 0; j < AJ; ++j) {
                f16x4 hi, lo;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float y = x[j][e] * scale;
                    row_mx[j] = fmaxf(row_mx[j], fabsf(y));
                    hi[e] = (_Float16)y;
                    lo[e] = (_Float16)(y - (float)hi[e]);
                }
                const int at = 2 * chunk(r0 + 16 * j, c4 >> 1) + (c4 & 1);
                st[at] = __builtin_bit_cast(u32x2c, hi);
                st[2 * PL + at] = __builtin_bit_cast(u32x2c, lo);
            }
            if (t == kt - 1 || t == T - 1) {   // a segment is complete: each row's range in it
#pragma unroll
                for (int j = 0; j < AJ; ++j) {
                    const float m = row16_max(row_mx[j]);
                    bad = bad || !(m < 65504.f) || (m != 0.f && m < 0.5f);
                    row_mx[j] = 0.f;
                }
                if (bad) s_bad = 1;
            }
        };
        split(0, x0);
        load(3, x0);
        split(1, x1);   // T is at least 2
        load(4, x1);
        __syncthreads();
        // while step t is multiplied, step t + 2 is split
        for (int32_t t = 0;; t += 3) {
            if (t + 2 < T) split(t + 2, x2);
            load(t + 5, x2);
            __syncthreads();
            if (t + 1 >= T) break;
            if (t + 3 < T) split(t + 3, x0);
            load(t + 6, x0);
            __syncthreads();
            if (t + 2 >= T) break;
            if (t + 4 < T) split(t + 4, x1);
            load(t + 7, x1);
            __syncthreads();
            if (t + 3 >= T) break;
        }
        if (!s_bad) return;
        for (int32_t t = 0; t < T; ++t) {   // out of fp16's range: three bf16 parts
            load(t, x0);
            mask(t, x0);
            __syncthreads();   // the step before is multiplied
#pragma unroll
            for (int j = 0; j < AJ; ++j) {
                uint16_t q[3][4];
#pragma unroll
                for (int e = 0; e < 4; ++e) split3_bits(x0[j][e], q[0][e], q[1][e], q[2][e]);
                const int at = 2 * chunk(r0 + 16 * j, c4 >> 1) + (c4 & 1);
#pragma unroll
                for (int p = 0; p < 3; ++p)
                    ((u32x2c *)(S + p * PL))[at] = u32x2c{(uint32_t)q[p][0] | ((uint32_t)q[p][1] << 16),
                                                          (uint32_t)q[p][2] | ((uint32_t)q[p][3] << 16)};
            }
            __syncthreads();
        }
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
    f32x16c acc[TM];
#pragma unroll
    for (int m = 0; m < TM; ++m)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[m][r] = 0.f;
    __syncthreads();
    const float mx = fmaxf(fmaxf(s_max[0], s_max[1]), fmaxf(s_max[2], s_max[3]));
    float scale, back;
    scale_of(mx, kRowExp, scale, back);
    __syncthreads();
    // Row fragments are read 16 k ahead of their products, across the step's
    // end too: the next step's stage was complete a barrier ago.
    f16x8 ah[2][TM], al[2][TM];
    auto fetch = [&](const u32x4c *st, int u) {
#pragma unroll
        for (int m = 0; m < TM; ++m) {
            const int r = chunk((wm * TM + m) * 32 + lr, 2 * u + h);
            ah[u & 1][m] = __builtin_bit_cast(f16x8, st[r]);
            al[u & 1][m] = __builtin_bit_cast(f16x8, st[PL + r]);
        }
    };
    fetch(S, 0);
    int32_t stage = 0;
    for (int32_t t = 0; t < T; ++t) {
        const u32x4c *st = S + stage * 2 * PL;
        stage = stage == 2 ? 0 : stage + 1;
        const u32x4c *next = S + stage * 2 * PL;   // (after the last step: read, not used)
        const int32_t tn = t + 1 < T ? t + 1 : t;
#pragma unroll
        for (int u = 0; u < kFrags; ++u) {
            if (u + 1 < kFrags) fetch(st, u + 1);
            else fetch(next, 0);
            const int b = u & 1;
            if constexpr (LL) {
#pragma unroll
                for (int m = 0; m < TM; ++m)
                    acc[m] = __builtin_amdgcn_mfma_f32_32x32x16_f16(w[u][1], al[b][m], acc[m], 0, 0, 0);
            }
#pragma unroll
            for (int m = 0; m < TM; ++m) acc[m] = __builtin_amdgcn_mfma_f32_32x32x16_f16(w[u][1], ah[b][m], acc[m], 0, 0, 0);
#pragma unroll
            for (int m = 0; m < TM; ++m) acc[m] = __builtin_amdgcn_mfma_f32_32x32x16_f16(w[u][0], al[b][m], acc[m], 0, 0, 0);
#pragma unroll
            for (int m = 0; m < TM; ++m) acc[m] = __builtin_amdgcn_mfma_f32_32x32x16_f16(w[u][0], ah[b][m], acc[m], 0, 0, 0);
            load_w(tn, u);   // a whole step ahead of its use, into the registers just used
        }
        __syncthreads();
    }
    const bool redo = s_bad != 0;
    if (redo) {   // out of fp16's range: three bf16 parts, six products
        back = 1.f;
#pragma unroll
        for (int m = 0; m < TM; ++m)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[m][r] = 0.f;
        const u32x4c *bb = bf_planes + (int64_t)g * steps * 192 + lane;
        for (int32_t t = 0; t < T; ++t) {
            __syncthreads();
            __syncthreads();
#pragma unroll 1
            for (int u = 0; u < kFrags; ++u) {
                bf16x8 b[3];
#pragma unroll
                for (int p = 0; p < 3; ++p) b[p] = __builtin_bit_cast(bf16x8, bb[(int64_t)((t * kFrags + u) * 3 + p) * 64]);
#pragma unroll
                for (int m = 0; m < TM; ++m) {
                    const int r = chunk((wm * TM + m) * 32 + lr, 2 * u + h);
                    acc[m] = mfma_split6(b[0], b[1], b[2], __builtin_bit_cast(bf16x8, S[r]),
                                         __builtin_bit_cast(bf16x8, S[PL + r]), __builtin_bit_cast(bf16x8, S[2 * PL + r]),
                                         acc[m]);
                }
            }
        }
    }
    if (gw >= groups) return;
    // acc[m][4 q + e]: row lr of block m, column 8 q + 4 h + e of the group
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int32_t n = g * 32 + 8 * q + 4 * h;
        f32x4c s = {1.f, 1.f, 1.f, 1.f};
        if (!redo) s = *(const f32x4c *)(inv + n);
        // both scales at once: one after the other could leave fp32's range on the way
        int exp[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) exp[e] = (int)(__float_as_uint(back) >> 23) + (int)(__float_as_uint(s[e]) >> 23) - 254;
#pragma unroll
        for (int m = 0; m < TM; ++m) {
            const int64_t row = m0 + (wm * TM + m) * 32 + lr;
            if (row >= M) continue;
            f32x4c v;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[e] = ldexpf(acc[m][4 * q + e], exp[e]);
                if (relu) v[e] = fmaxf(v[e], 0.f);
            }
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

namespace {
// k steps of 64 per segment; columns padded to the 32 WN of a workgroup
int64_t f32_kt(int64_t d_in) { return (d_in + kStep - 1) / kStep; }
int64_t f32_cols(int64_t d_out) { return (d_out + 255) / 256 * 256; }
}  // namespace

size_t combine_f32_workspace(int64_t d_in, int64_t d_out) {
    const size_t values = (size_t)(f32_cols(d_out) * 2 * f32_kt(d_in) * kStep);
    return values * 2 * 5 + (size_t)f32_cols(d_out) * sizeof(float);
}

void launch_split_weights(const float *w, int64_t d_in, int64_t d_out, void *ws, hipStream_t s) {
    const int64_t kt = f32_kt(d_in), nc = f32_cols(d_out), values = nc * 2 * kt * kStep;
    char *p = (char *)ws;
    hipLaunchKernelGGL(k_split_weights, dim3((unsigned)((d_out + 31) / 32 * 4)), dim3(kSplitThreads), 0, s, w, (int32_t)d_in,
                       (int32_t)d_out, (int32_t)kt, (u32x4c *)p, (u32x4c *)(p + 4 * values), (float *)(p + 10 * values));
    GNNAV_HIP(hipGetLastError());
}

void launch_combine_f32(const float *self, int64_t ld_self, const float *agg, int64_t ld_agg, int64_t m,
                        const int32_t *m_dev, int64_t d_in, int64_t d_out, const void *ws, bool relu, float *out,
                        int64_t ld_out, hipStream_t s) {
    const int64_t kt = f32_kt(d_in), nc = f32_cols(d_out), values = nc * 2 * kt * kStep;
    const char *p = (const char *)ws;
    const int vec = ld_out % 4 == 0 && ((uintptr_t)out & 15u) == 0;
    auto run = [&](auto tm_, auto wm_, auto wn_) {
        constexpr int tm = decltype(tm_)::value, wm = decltype(wm_)::value, wn = decltype(wn_)::value;
        const dim3 grid((unsigned)((m + 32 * tm * wm - 1) / (32 * tm * wm)), (unsigned)((d_out + 32 * wn - 1) / (32 * wn)));
        auto kern = kt == 1 ? k_combine_f32<tm, wm, wn, true> : k_combine_f32<tm, wm, wn, false>;
        hipLaunchKernelGGL(kern, grid, dim3(64 * (kMulWaves + kRowWaves)), 0, s, self, ld_self, agg, ld_agg, m, m_dev,
                           (int32_t)d_in, (int32_t)kt, (const u32x4c *)p, (const u32x4c *)(p + 4 * values),
                           (const float *)(p + 10 * values), (int32_t)d_out, (int)relu, vec, out, ld_out);
    };
    const std::integral_constant<int, 1> i1;
    const std::integral_constant<int, 2> i2;
    const std::integral_constant<int, 3> i3;
    const std::integral_constant<int, 4> i4;
    const std::integral_constant<int, 8> i8;
    // rows of 32 on the busiest of 256 compute units (one workgroup each at a
    // time), half a block's work of overhead a workgroup
    auto cost = [&](int blocks, int wn) {
        const int64_t wgs = ((m + 32 * blocks - 1) / (32 * blocks)) * ((d_out + 32 * wn - 1) / (32 * wn));
        return (wgs + 255) / 256 * (2 * blocks + 1);
    };
    if (d_out > 128) {
        int best = 3;
        for (int b = 2; b >= 1; --b)
            if (cost(b, 8) < cost(best, 8)) best = b;
        if (best == 3) run(i3, i1, i8);
        else if (best == 2) run(i2, i1, i8);
        else run(i1, i1, i8);
    } else if (d_out > 64) {
        if (cost(2, 4) < cost(4, 4)) run(i1, i2, i4);
        else run(i2, i2, i4);
    } else {
        run(i1, i4, i2);
    }
    GNNAV_HIP(hipGetLastError());
}

}  // namespace gnnav
