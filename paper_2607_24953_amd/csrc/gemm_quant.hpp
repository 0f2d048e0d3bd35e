// FP4-quantizing epilogue of the GEMM kernels.
#pragma once

#include "gemm_common.hpp"

namespace q2d {
namespace {

// Quantize a wave's accumulator block into 2D-block FP4 with round to
// nearest (the quantizer's scale rule and codec, applied to the float32
// result): each 32 x 32 MFMA tile is exactly one block.
//   1. block maxima: each lane's maximum over the 16 values it holds of every
//      tile, then the 16 maxima reduced across the wave together (quad and row
//      permutes, then two lane exchanges), so the reductions overlap; with
//      CHECK, values outside rows_left x cols_left count as 0 (padding gets
//      zero codes, an all-zero block the byte 0x00);
//   2. per 32-row strip i, per tile j:
//      codes_t: a lane holds one column's rows 8q + 4h + 0..3 (h = lane / 32),
//               two bytes per q; the halves h swap one word so that each lane
//               stores 8 consecutive bytes of its column's 16-byte run;
//      codes:   neighbouring columns meet through a quad permute; the even lane
//               packs rows q = 0, 1 and the odd lane rows q = 2, 3, one byte per
//               row, into the wave's LDS strip (32 rows x 16 TJ bytes);
//      scales:  one byte per tile in each grid;
//      then the strip leaves as 16-byte row segments.
// Only the written extent of the layout is touched: codes rows < M, bytes below
// roundup(N, 128) / 2; codes_t rows < N, bytes below roundup(M, 128) / 2.
//
// Stochastic rounding (SR): element (r, c) of the M x N result takes the draw of
// storage index r N + c of a row-major M x N tensor (half (idx & 1) of word
// (idx & 7) >> 1 of the Philox block for counter (idx >> 3, offset)), the draw
// q2d_quantize would give it, and is converted on its own with seed r16 << 16
// (first element of a pair) or r16 << 15 (second).  N is a multiple of 8, so a
// Philox block covers 8 consecutive columns of one row: the wave computes each
// of a tile's 128 blocks once (two per lane) into its LDS table, and every lane
// reads back the 16-bit draws of the 16 elements it holds.
constexpr int q_pitch(int tj) { return 16 * tj + 16; }      // LDS strip row pitch
constexpr int q_strip(int tj) { return 32 * q_pitch(tj); }  // per wave
constexpr int kPRow = 80;                       // Philox table row: four 16-byte blocks + pad
constexpr int kPTab = 32 * kPRow;               // per wave

typedef float f32x2 __attribute__((ext_vector_type(2)));

// SR conversion of a pair into byte `sel` of a zero word (only the nibble the
// caller keeps is defined)
__device__ __forceinline__ uint32_t sr_cvt(int sel, f32x2 v, uint32_t seed, float scale)
{
    switch (sel) {
    case 0: return __builtin_amdgcn_cvt_scalef32_sr_pk_fp4_f32(0u, v, seed, scale, 0);
    case 1: return __builtin_amdgcn_cvt_scalef32_sr_pk_fp4_f32(0u, v, seed, scale, 1);
    case 2: return __builtin_amdgcn_cvt_scalef32_sr_pk_fp4_f32(0u, v, seed, scale, 2);
    default: return __builtin_amdgcn_cvt_scalef32_sr_pk_fp4_f32(0u, v, seed, scale, 3);
    }
}

// byte `sel` of `old` gets the SR codes of the pair (a, b): a with seed ra
// (= r16 << 16) in the low nibble, b with seed rb >> 1 (= r16 << 15) in the high
__device__ __forceinline__ uint32_t sr_pair_into(uint32_t old, int sel, float a, float b, uint32_t ra, uint32_t rb,
                                                 float scale)
{
    const f32x2 v = {a, b};
    const uint32_t lo = sr_cvt(sel, v, ra, scale), hi = sr_cvt(sel, v, rb >> 1, scale);
    return old | (lo & (0x0Fu << (8 * sel))) | (hi & (0xF0u << (8 * sel)));
}

//
// TI x TJ: MFMA tiles of the wave (its block is 32 TI x 32 TJ); AGPR: the accumulators
// live there and are read one by one (the persistent kernel has no registers to
// copy them to).
template <bool CHECK, bool SR, int TI, int TJ, bool AGPR>
__device__ __forceinline__ void store_qblock(v16f (&acc)[TI][TJ], const GemmArgs &g, uint8_t *strip, uint8_t *ptab,
                                             int r0, int c0, int rows_left, int cols_left)
{
    const int lane = threadIdx.x & 63;
    const int col = lane & 31, h = lane >> 5, odd = lane & 1;
    const int padm = (int)((g.M + 127) / 128 * 128), padn = (int)((g.N + 127) / 128 * 128);
    if (AGPR) {
        int dummy = 0;
        asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" : "+s"(dummy));   // the last MFMA results settle
    }
    auto value = [&](int i, int j, int r) __attribute__((always_inline)) -> float {
        float v;
        if constexpr (AGPR) asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v) : "a"(acc[i][j][r]));
        else v = acc[i][j][r];
        if (CHECK) {
            const int rr = 32 * i + 8 * (r >> 2) + 4 * h + (r & 3);
            if (rr >= rows_left || 32 * j + col >= cols_left) v = 0.0f;
        }
        return v;
    };
    uint32_t am[TI][TJ];
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j) {
            uint32_t m = 0;
#pragma unroll
            for (int r = 0; r < 16; ++r) m = max(m, f_bits(value(i, j, r)) & 0x7FFFFFFFu);
            am[i][j] = m;
        }
    // quad_perm [1,0,3,2], quad_perm [2,3,0,1], row_half_mirror, row_mirror
    auto perm_max = [&](auto ctrl) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j)
                am[i][j] = max(am[i][j], (uint32_t)__builtin_amdgcn_update_dpp((int)am[i][j], (int)am[i][j],
                                                                               decltype(ctrl)::value, 0xF, 0xF, false));
    };
    perm_max(std::integral_constant<int, 0xB1>{});
    perm_max(std::integral_constant<int, 0x4E>{});
    perm_max(std::integral_constant<int, 0x141>{});
    perm_max(std::integral_constant<int, 0x140>{});
#pragma unroll
    for (int m = 16; m < 64; m <<= 1)
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j) am[i][j] = max(am[i][j], (uint32_t)__shfl_xor((int)am[i][j], m));

    // compile-time tile indices: a runtime loop here would put acc in scratch memory
    unroll<TI>([&](auto ic) __attribute__((always_inline)) {
        constexpr int i = decltype(ic)::value;
        const int tr = r0 + 32 * i;                     // strip origin row in C
        unroll<TJ>([&](auto jc) __attribute__((always_inline)) {
            constexpr int j = decltype(jc)::value;
            const int tc = c0 + 32 * j;                 // tile origin column
            const bool finite = am[i][j] < 0x7F800000u;
            const int e = fp4_block_exponent(am[i][j]);
            const float scale = bits_f((uint32_t)(127 + e) << 23);
            float v[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) v[r] = value(i, j, r);
            // SR draws of the lane's elements (rows 8 (r / 4) + 4 h + r % 4, column col),
            // packed two to a register: rw[k] = draw(2k) | draw(2k + 1) << 16
            uint32_t rw[8];
            if constexpr (SR) {
                // the previous tile's reads of the table come first (in program order)
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const int b = lane + 64 * t, brow = b >> 2, bcg = b & 3;
                    const uint64_t idx = (uint64_t)(uint32_t)(tr + brow) * (uint64_t)g.N + (uint64_t)(tc + 8 * bcg);
                    uint32_t w[4];
                    philox4x32_10((uint32_t)(idx >> 3), (uint32_t)(idx >> 35), (uint32_t)g.offset,
                                  (uint32_t)(g.offset >> 32), (uint32_t)g.seed, (uint32_t)(g.seed >> 32), w);
                    *reinterpret_cast<uint4 *>(ptab + brow * kPRow + 16 * bcg) = make_uint4(w[0], w[1], w[2], w[3]);
                }
                // LDS accesses of one wave complete in order: the reads below see the table.
                // All 16 reads issue back to back, so their latency is paid once.
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_sched_barrier(0);
                const uint8_t *cp = ptab + 16 * (col >> 3) + 4 * ((col & 7) >> 1) + 2 * (col & 1);
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const int rl = 8 * (k >> 1) + 4 * h + 2 * (k & 1);        // row of element 2k
                    const uint32_t d0 = *reinterpret_cast<const uint16_t *>(cp + rl * kPRow);
                    const uint32_t d1 = *reinterpret_cast<const uint16_t *>(cp + (rl + 1) * kPRow);
                    rw[k] = d0 | (d1 << 16);
                }
            }
            // the draw of element r, shifted to bits 31..16
            auto rr = [&](int r) __attribute__((always_inline)) -> uint32_t {
                return (r & 1) ? (rw[r >> 1] & 0xFFFF0000u) : (rw[r >> 1] << 16);
            };
            // column-packed: word q/2 byte 2 (q % 2) + k holds rows (8q + 4h + 2k, +1)
            uint32_t w0 = 0, w1 = 0;
            if constexpr (SR) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    w0 = sr_pair_into(w0, k, v[2 * k], v[2 * k + 1], rr(2 * k), rr(2 * k + 1), scale);
                    w1 = sr_pair_into(w1, k, v[8 + 2 * k], v[9 + 2 * k], rr(8 + 2 * k), rr(9 + 2 * k), scale);
                }
            } else {
                w0 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w0, v[0], v[1], scale, 0);
                w0 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w0, v[2], v[3], scale, 1);
                w0 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w0, v[4], v[5], scale, 2);
                w0 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w0, v[6], v[7], scale, 3);
                w1 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w1, v[8], v[9], scale, 0);
                w1 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w1, v[10], v[11], scale, 1);
                w1 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w1, v[12], v[13], scale, 2);
                w1 = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w1, v[14], v[15], scale, 3);
            }
            if (!finite) w0 = w1 = 0;
            // half 0 stores bytes 0..7 of the run (q = 0, 1 of both halves), half 1
            // bytes 8..15 (q = 2, 3)
            const uint32_t mine = h ? w1 : w0;
            const uint32_t other = (uint32_t)__shfl_xor((int)(h ? w0 : w1), 32);
            const uint32_t first = h ? other : mine, second = h ? mine : other;
            const uint2 run = make_uint2((first & 0xFFFFu) | (second << 16), (first >> 16) | (second & 0xFFFF0000u));
            if (tc + col < g.N && tr < padm)
                *reinterpret_cast<uint2 *>(g.qct + (int64_t)(tc + col) * g.ldqct + tr / 2 + 8 * h) = run;
            // row-packed: both layouts hold the same code for an element (one block
            // scale; under SR the element's own draw either way), so the row bytes
            // come from the column words.  Nibble r & 7 of w0 (w1) is the code of
            // v[r] for r < 8 (r >= 8).  Of a column pair, the even lane packs rows
            // v[0..7] (its own column low, the neighbour's high), the odd lane rows
            // v[8..15] (the neighbour's low, its own high): one word from the
            // neighbour, then the two words' nibbles zipped into bytes.
            const uint32_t send = odd ? w0 : w1;
            const uint32_t recv = (uint32_t)__builtin_amdgcn_update_dpp((int)send, (int)send, 0xB1, 0xF, 0xF, false);
            const uint32_t lo = odd ? recv : w0, hi = odd ? w1 : recv;
            const uint32_t ev = (lo & 0x0F0F0F0Fu) | ((hi << 4) & 0xF0F0F0F0u);     // byte k: row 2k
            const uint32_t od = ((lo >> 4) & 0x0F0F0F0Fu) | (hi & 0xF0F0F0F0u);     // byte k: row 2k + 1
            uint32_t rowb[2] = {__builtin_amdgcn_perm(od, ev, 0x05010400u), __builtin_amdgcn_perm(od, ev, 0x07030602u)};
            if (!finite) rowb[0] = rowb[1] = 0;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int rk = odd ? 8 + k : k;
                const int rl = 8 * (rk >> 2) + 4 * h + (rk & 3);
                strip[rl * q_pitch(TJ) + 16 * j + (col >> 1)] = (uint8_t)(rowb[k >> 2] >> (8 * (k & 3)));
            }
            if (lane == 0) {
                const uint8_t sbyte = finite ? (uint8_t)(e + 127) : (uint8_t)0xFF;
                if (tr < g.M && tc < padn) g.qs[(int64_t)(tr / 32) * g.ldqs + tc / 32] = sbyte;
                if (tc < g.N && tr < padm) g.qst[(int64_t)(tc / 32) * g.ldqst + tr / 32] = sbyte;
            }
        });
        // the strip's 32 rows as 16-byte row segments (LDS accesses of
        // one wave complete in order, so the reads see the writes above)
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int k = 0; k < TJ / 2; ++k) {
            const int rl = lane / TJ + 64 / TJ * k, chunk = lane % TJ;
            const uint4 w = *reinterpret_cast<const uint4 *>(strip + rl * q_pitch(TJ) + 16 * chunk);
            if (tr + rl < g.M && c0 + 32 * chunk < padn)
                *reinterpret_cast<uint4 *>(g.qc + (int64_t)(tr + rl) * g.ldqc + c0 / 2 + 16 * chunk) = w;
        }
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_sched_barrier(0);
    });
}

}  // namespace
}  // namespace q2d
