// Eq. 1 Combine in bf16 for many rows and weights that fit the registers: a
// persistent workgroup per compute unit keeps its weight columns in registers
// for the whole launch and streams row tiles of [self | agg] through LDS.
//
// The combine of a sampled layer reads 4 d_in bytes a row and writes 2 d_out,
// a few dozen multiply-adds per byte, so HBM bounds it.  Tiled as an ordinary
// GEMM (k_combine_ring) every 128-row tile pulled its weight columns from L2
// again (as many bytes as its rows), walked a k loop of four latency-bound
// steps, and needed a transposed copy of the weights made by a launch of its
// own.  Here:
//   - wavefront w owns 32 output columns and holds their weights as MFMA
//     fragments, 4 registers per 16 k (64 for 256 k, 128 for 512), loaded once
//     straight from the row-major W while the first row tiles are in flight;
//   - a row tile is BM rows of both segments, 32 KB, by LDS DMA into a ring of
//     three: two tiles (64 KB per compute unit) are always on their way;
//   - the product is taken transposed (weights as the A operand), so a lane
//     holds consecutive columns of one output row; bf16 rows gather in the LDS
//     stage the tile has just left and go out as whole lines (stored straight
//     from registers, 32 bytes of a row at a time, they took 15% longer).
// Stores are raw buffer stores that drop what lies past the last row or
// column: every wavefront issues the same number of them per tile, which lets
// the wait for a tile's DMAs count them (vmcnt runs in issue order).
//
// Measured against k_combine_ring with its transpose launch: 107,000 x 256 x
// 256 51.3 -> 32.4 us (110 MB, 3.4 TB/s; 400,000 rows 152 -> 91 us, 4.5 TB/s),
// 24,000 x 512 x 256 23.0 -> 21.0 us (three tiles a workgroup, half of the time
// is the weights' way to 256 compute units), 20,000 x 128 x 128 14.3 -> 9.0 us.
// With weights gathered column by column, 2 bytes a load, the prologue took
// 6 us longer; with the products branching on the step count 20% more in all.
#include <algorithm>
#include <type_traits>

#include "bf16split.hpp"
#include "common.hpp"
#include "dma.hpp"

namespace gnnav {

namespace {

typedef float f32x16s __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4s __attribute__((ext_vector_type(4)));

// 8 x 8 transpose of 16-bit values over the lanes that differ in bits 0, 1 and
// 4: lane (b4 b1 b0) passes row 4 b4 + 2 b1 + b0 of 8 values and receives
// column 4 b4 + 2 b1 + b0.
__device__ __forceinline__ void transpose8(uint32_t (&d)[4], int lane) {
    // bit 0 against the halves of a dword
    const uint32_t sel = (lane & 1) ? 0x03020706u : 0x05040100u;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint32_t o = (uint32_t)__builtin_amdgcn_mov_dpp((int)d[q], 0xB1, 0xf, 0xf, true);   // lane ^ 1
        d[q] = __builtin_amdgcn_perm(o, d[q], sel);
    }
    // bit 1 against dwords q, q + 1
#pragma unroll
    for (int q = 0; q < 4; q += 2) {
        const uint32_t give = (lane & 2) ? d[q] : d[q + 1];
        const uint32_t got = (uint32_t)__builtin_amdgcn_mov_dpp((int)give, 0x4E, 0xf, 0xf, true);   // lane ^ 2
        d[q] = (lane & 2) ? got : d[q];
        d[q + 1] = (lane & 2) ? d[q + 1] : got;
    }
    // bit 4 against dwords q, q + 2
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const auto z = __builtin_amdgcn_permlane16_swap(d[q], d[q + 2], false, false);
        d[q] = z[0];
        d[q + 2] = z[1];
    }
}

// two floats as a pair of bf16, rounded to nearest even
__device__ __forceinline__ uint32_t bf16_pair(float lo, float hi) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    bf16x2 v;   // one v_cvt_pk_bf16_f32, the same bits as bf16_rne
    v[0] = (__bf16)lo;
    v[1] = (__bf16)hi;
    return __builtin_bit_cast(uint32_t, v);
}

// KT: 16-deep k steps the fragments have room for (both segments); TM: 32-row
// blocks per wavefront; WM x WN wavefronts over rows x 32-column groups.  FULL:
// every step is used (d_in 8 KT), so the product loop has no branches.
template <int KT, int TM, int WM, int WN, bool FULL, class OutT>
__global__ void __launch_bounds__(64 * WM * WN) k_combine_stream(const uint16_t *__restrict__ A0, int64_t lda0,
                                                                 const uint16_t *__restrict__ A1, int64_t lda1,
                                                                 int64_t M, const int32_t *__restrict__ m_dev,
                                                                 int32_t K, const uint16_t *__restrict__ W, int32_t N,
                                                                 int relu, OutT *__restrict__ C, int64_t ldc) {
    constexpr int NW = WM * WN, BM = 32 * TM * WM, PITCH = 2 * KT, STAGES = 3;
    constexpr int PER = BM * PITCH / 64 / NW;                           // DMAs per wavefront and tile
    constexpr int ST = TM * (sizeof(OutT) == 2 ? 2 : 4);                // stores per wavefront and tile
    static_assert(BM * PITCH % (64 * NW) == 0 && PITCH % 16 == 0 && 2 * ST + PER < 64, "tile shape");
    __shared__ u32x4s S[STAGES][BM * PITCH];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int wm = wid / WN, wn = wid % WN, h = lane >> 5, lr = lane & 31;
    if (m_dev) M = *m_dev;
    const int64_t tiles = (M + BM - 1) / BM, G = gridDim.x;
    int64_t tile = blockIdx.x;
    if (tile >= tiles) return;
    if constexpr (FULL) K = 8 * KT;
    const int32_t kts = FULL ? KT / 2 : (K + 15) / 16, kt = 2 * kts;   // k steps per segment, in all

    // LDS slot (row, c) holds chunk c ^ (row & 15) of the row: 16 consecutive
    // rows' fragment reads touch 16 distinct 16-byte bank groups
    int r_[PER], k_[PER];
    bool s1[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int s = (wid * PER + q) * 64 + lane;
        r_[q] = s / PITCH;
        const int ch = (s % PITCH) ^ (r_[q] & 15);
        s1[q] = ch >= 2 * kts;
        k_[q] = 8 * (s1[q] ? ch - 2 * kts : ch);
    }
    auto issue = [&](int64_t t, int stage) {
        const int64_t m0 = t * BM;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int64_t row = m0 + r_[q] < M ? m0 + r_[q] : M - 1;
            const uint16_t *p = s1[q] ? A1 + row * lda1 : A0 + row * lda0;
            dma16(p + (k_[q] < K ? k_[q] : 0), &S[stage][(wid * PER + q) * 64]);
        }
    };
    // elements at k >= K of the last chunks of a segment (row padding, or a
    // reread of the row's start) become zero, by the lane that loaded them
    auto fixup = [&](int stage) {
        if (K % 16 == 0) return;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            if (k_[q] + 8 <= K) continue;
            uint16_t *e = (uint16_t *)&S[stage][(wid * PER + q) * 64 + lane];
#pragma unroll
            for (int x = 0; x < 8; ++x)
                if (k_[q] + x >= K) e[x] = 0;
        }
    };

    issue(tile, 0);
    if (tile + G < tiles) issue(tile + G, 1);

    const int32_t n0 = (int32_t)(blockIdx.y * WN + wn) * 32;
    // Weights: lane l loads 8 columns of one k row (16 bytes) and the lanes
    // transpose 8 x 8 among themselves, an eighth of the loads of gathering a
    // column's k values one by one.  Lane l ends with column col of the
    // wavefront's 32 and k = 16 t + 8 h .. + 7.
    const int cb = (lr >> 2) & 3, kr = (lr & 3) + 4 * (lr >> 4);   // loaded: column block, k row
    bf16x8 b[KT];
#pragma unroll
    for (int t = 0; t < KT; ++t) {
        uint32_t d[4] = {0u, 0u, 0u, 0u};
        if (t < kt) {
            const int32_t k = (t >= kts ? t - kts : t) * 16 + 8 * h + kr, n = n0 + 8 * cb;
            if (k < K && n < N) {   // N is a multiple of 8
                const u32x4s v = *(const u32x4s *)(W + ((int64_t)(t >= kts ? K : 0) + k) * N + n);
                d[0] = v[0], d[1] = v[1], d[2] = v[2], d[3] = v[3];
            }
        }
        b[t] = __builtin_bit_cast(bf16x8, u32x4s{d[0], d[1], d[2], d[3]});
    }
#pragma unroll
    for (int t = 0; t < KT; ++t) {
        const u32x4s v = __builtin_bit_cast(u32x4s, b[t]);
        uint32_t d[4] = {v[0], v[1], v[2], v[3]};
        transpose8(d, lane);
        b[t] = __builtin_bit_cast(bf16x8, u32x4s{d[0], d[1], d[2], d[3]});
    }

    int stage = 0;
    for (int64_t i = 0;; ++i, tile += G) {
        const bool next = tile + G < tiles;
        // issued after this tile's DMAs: the stores of the two tiles before
        // and the next tile's DMAs
        if (i >= 2 && next) wait_vm<2 * ST + PER>();
        else if (next) wait_vm<PER>();
        else wait_vm<0>();
        fixup(stage);
        lds_barrier();   // the tile is visible to all; everyone is done with the one before
        if (tile + 2 * G < tiles) issue(tile + 2 * G, stage == 0 ? 2 : stage - 1);
        f32x16s acc[TM];
#pragma unroll
        for (int m = 0; m < TM; ++m)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[m][r] = 0.f;
        u32x4s *buf = S[stage];
        // Row fragments are read a group of GRP steps ahead of the products
        // that use them (clamped, so no branch holds the reads back).
        constexpr int GRP = 4;
        bf16x8 a[2][GRP][TM];
        auto fetch = [&](int g, bf16x8 (&f)[GRP][TM]) {
#pragma unroll
            for (int u = 0; u < GRP; ++u) {
                const int t = FULL || g * GRP + u < kt ? g * GRP + u : 0;
#pragma unroll
                for (int m = 0; m < TM; ++m) {
                    const int r = (wm * TM + m) * 32 + lr;
                    f[u][m] = __builtin_bit_cast(bf16x8, buf[r * PITCH + ((2 * t + h) ^ (r & 15))]);
                }
            }
        };
        fetch(0, a[0]);
#pragma unroll
        for (int g = 0; g < KT / GRP; ++g) {
            if (g + 1 < KT / GRP) fetch(g + 1, a[(g + 1) & 1]);
#pragma unroll
            for (int u = 0; u < GRP; ++u) {
                if (FULL || g * GRP + u < kt) {
#pragma unroll
                    for (int m = 0; m < TM; ++m)
                        acc[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[g * GRP + u], a[g & 1][u][m], acc[m], 0, 0, 0);
                }
            }
        }
        // acc[m][4 q + e]: output row lr of block m, column
        // 8 (h + 2 (q % 2)) + 4 (q / 2) + e of the wavefront's 32
        const int64_t m0 = tile * BM;
        const int32_t left = (int32_t)(M - m0 < BM ? M - m0 : BM);
        const uint32_t pitch = (uint32_t)(ldc * (int64_t)sizeof(OutT));
        const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(C + m0 * ldc), (short)0, (int)((uint32_t)left * pitch),
                                                            0x00027000);
#pragma unroll
        for (int m = 0; m < TM; ++m)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (relu) acc[m][r] = fmaxf(acc[m][r], 0.f);
        if constexpr (sizeof(OutT) == 2) {
            constexpr int CPR = 4 * WN;   // 16-byte chunks of an output row in this workgroup's columns
            static_assert(BM * CPR <= BM * PITCH && BM * CPR / (64 * NW) == ST, "the output tile fits its stage");
            lds_barrier();   // every wavefront is done reading the tile
#pragma unroll
            for (int m = 0; m < TM; ++m) {
                const int r = (wm * TM + m) * 32 + lr;
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    u32x4s v;
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        v[e] = bf16_pair(acc[m][4 * p + 2 * e], acc[m][4 * p + 2 * e + 1]);
                        v[2 + e] = bf16_pair(acc[m][8 + 4 * p + 2 * e], acc[m][8 + 4 * p + 2 * e + 1]);
                    }
                    buf[r * CPR + ((4 * wn + h + 2 * p) ^ (r & (CPR - 1)))] = v;
                }
            }
            lds_barrier();
            const int32_t nb = (int32_t)blockIdx.y * WN * 32;
#pragma unroll
            for (int q = 0; q < ST; ++q) {
                const int i2 = q * 64 * NW + tid, r = i2 / CPR;
                const int32_t n = nb + 8 * ((i2 % CPR) ^ (r & (CPR - 1)));
                __builtin_amdgcn_raw_buffer_store_b128(buf[i2], rsrc,
                                                       n < N ? (int)((uint32_t)r * pitch + 2u * (uint32_t)n) : INT_MAX, 0,
                                                       0);
            }
        } else {
#pragma unroll
            for (int m = 0; m < TM; ++m) {
                const uint32_t row = (uint32_t)((wm * TM + m) * 32 + lr) * pitch;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int32_t n = n0 + 8 * (h + 2 * (q & 1)) + 4 * (q >> 1);
                    const u32x4s v = {__float_as_uint(acc[m][4 * q]), __float_as_uint(acc[m][4 * q + 1]),
                                      __float_as_uint(acc[m][4 * q + 2]), __float_as_uint(acc[m][4 * q + 3])};
                    __builtin_amdgcn_raw_buffer_store_b128(v, rsrc, n < N ? (int)(row + 4u * (uint32_t)n) : INT_MAX, 0,
                                                           0);
                }
            }
        }
        if (!next) break;
        stage = stage == 2 ? 0 : stage + 1;
    }
}

}  // namespace

// Whether the streaming kernel takes a bf16 combine of many rows: the weights
// of 32 columns fit 128 registers (d_in <= 256), weight and output rows move 16
// bytes at a time, and it is the faster one.  Ratios are the ring's time over its
// own, measured over d_in 8 .. 256, d_out 8 .. 768 and 2,600 .. 300,000 rows:
//   d_out in (128, 256]: 1.0 to 2.4 everywhere;
//   d_out in (64, 128]: 1.1 to 2.1; 0.7 to 0.95 past 32,768 rows where d_in > 128
//     is no multiple of 16 (every tile's last chunks are then masked in LDS);
//   d_out <= 64 has two or four wavefronts to a workgroup: d_in <= 128 1.1 to 1.9, not
//     a multiple of 16 below 1 past 65,536 rows (0.7 at 300,000 x 40); d_in in
//     (128, 256) 1.3 to 1.5 up to 16,384 rows, 0.7 at 300,000, and 0.3 to 0.95 where
//     it is no multiple of 16; d_in = 256 (no bound in the loop) 1.06 to 1.8;
//   d_out > 256 reads the rows again for every 256 columns: d_in <= 128 1.1 to 2.1,
//     fp32 results 0.8 to 1.3 unless there are few rows or d_in is small; d_in > 128
//     1.2 to 1.7 up to 4,096 rows of two groups, 0.6 to 1.2 above, 1.0 to 1.7 from
//     200,000.
bool combine_streams(int64_t m, int64_t d_in, const void *w, int64_t d_out, bool out_bf16, const void *out,
                     int64_t ld_out) {
    if (!(d_in <= 256 && d_out % 8 == 0 && ld_out % (out_bf16 ? 8 : 4) == 0 &&
          (((uintptr_t)w | (uintptr_t)out) & 15u) == 0 && ld_out < (1 << 20) && d_out < (1 << 20)))
        return false;
    const bool ragged = d_in % 16 != 0, deep = d_in > 128;
    if (d_out > 256) {
        const int64_t groups = (d_out + 255) / 256;
        if (deep) return m * groups <= 8192 || m >= 200000;
        return out_bf16 || d_in <= 48 || m <= 8192;
    }
    if (d_out > 128) return true;
    if (d_out > 64) return !(deep && ragged) || m <= 32768;
    if (deep) return d_in == 256 || (!ragged && m <= 16384);
    return !ragged || m <= 65536;
}

void launch_combine_stream(const uint16_t *self, int64_t ld_self, const uint16_t *agg, int64_t ld_agg, int64_t m,
                           const int32_t *m_dev, int64_t d_in, const uint16_t *w, int64_t d_out, bool relu,
                           bool out_bf16, void *out, int64_t ld_out, hipStream_t s) {
    // as many workgroups as units to run on: more would come in a second round
    // that loads the weights again (on half of the units, one workgroup for each
    // of the chip's against so: 6,000 x 512 x 256 22.4 -> 14.0 us, 24,000 rows 31.6
    // -> 22.6, 107,000 x 256 x 256 45 -> 40)
    const int units = stream_units(s);
    auto run = [&](auto kt_, auto tm_, auto wm_, auto wn_) {
        constexpr int KT = decltype(kt_)::value, TM = decltype(tm_)::value, WM = decltype(wm_)::value,
                      WN = decltype(wn_)::value, BM = 32 * TM * WM;
        const dim3 grid((unsigned)std::min<int64_t>((m + BM - 1) / BM, units), (unsigned)((d_out + 32 * WN - 1) / (32 * WN)));
        auto go = [&](auto kern, auto *o) {
            hipLaunchKernelGGL(kern, grid, dim3(64 * WM * WN), 0, s, self, ld_self, agg, ld_agg, m, m_dev, (int32_t)d_in, w,
                               (int32_t)d_out, (int)relu, o, ld_out);
        };
        const bool full = d_in == 8 * KT;
        if (out_bf16)
            full ? go(k_combine_stream<KT, TM, WM, WN, true, uint16_t>, (uint16_t *)out)
                 : go(k_combine_stream<KT, TM, WM, WN, false, uint16_t>, (uint16_t *)out);
        else
            full ? go(k_combine_stream<KT, TM, WM, WN, true, float>, (float *)out)
                 : go(k_combine_stream<KT, TM, WM, WN, false, float>, (float *)out);
    };
    using std::integral_constant;
    integral_constant<int, 1> i1;
    integral_constant<int, 2> i2;
    integral_constant<int, 4> i4;
    integral_constant<int, 8> i8;
    integral_constant<int, 16> i16;
    integral_constant<int, 32> i32;
    if (d_in <= 128) {
        if (d_out > 128) run(i16, i2, i1, i8);
        else if (d_out > 64) run(i16, i1, i2, i4);
        else run(i16, i1, i2, i2);
    } else {
        if (d_out > 128) run(i32, i1, i1, i8);
        else if (d_out > 64) run(i32, i1, i1, i4);
        else run(i32, i1, i1, i2);
    }
    GNNAV_HIP(hipGetLastError());
}

}  // namespace gnnav
