// Fused 2D-block FP4 quantizer (Sec. 3, Sec. 3.1; App. D, App. E).
//
// One pass over the input: block maximum, truncation-free E8M0 scale, round to
// nearest or Philox stochastic rounding, and both packed layouts (row-packed
// codes and column-packed codes_t) plus the scale grid and its transpose.
//
// Work split: a workgroup owns a 128-row tile of WC x 128 columns (small inputs:
// a strip of its own); each wave owns a 32 x 128 strip (four 32 x 32 blocks side by side).  Lane l owns an
// 8 x 8 sub-block: rows 8*(l/16) .. +7 and columns 8*(l%16) .. +7 of the strip.
// A row of the sub-block is one 16-byte load (bf16), so every load
// instruction of the wave reads four 256-byte row segments.  The 8 x 8
// sub-block makes the transposition local: each lane packs eight nibbles per
// row for codes and eight per column for codes_t without data exchange.  The
// block maximum is a max over the lane's 64 values followed by four cross-lane
// butterflies (the 16 lanes of a 32 x 32 block differ in lane bits 0, 1, 4, 5).
// bfloat16 rows stay packed two elements per register.
//
// The packed codes go through LDS and leave as 16-byte stores: full 128-byte
// lines of codes when the tile is 256 columns wide (WC = 2, round to nearest),
// 64-byte runs of codes_t.
//
// Round to nearest uses gfx950's v_cvt_scalef32_pk_fp4_{bf16,f32}: the E2M1
// code of x / S rounded to nearest even, two elements per instruction, which
// is the round-to-nearest definition exactly.
//
// Stochastic rounding uses v_cvt_scalef32_sr_pk_fp4_f32.  It converts a pair
// with one 32-bit seed: the first element adds seed >> 10 below its kept
// mantissa bit (after aligning subnormal E2M1 results) and truncates, the
// second element adds (seed << 1) >> 10.  A seed of r16 << 16 for the first
// element, or r16 << 15 for the second, therefore rounds the magnitude up
// exactly when floor(2^16 d / delta) + r16 >= 2^16 -- the rounding contract of
// this library.  Each element is converted in an instruction where it has its
// own draw; the other nibble of that result is dropped.  The parity tests
// compare every bfloat16 value under every scale, in both modes, bit for bit
// with the CPU definition.
//
// The same kernel emits 1D FP4 for activations (ONED; Sec. 3, "Application to
// linear layers"; App. C, "Activations"): 1 x 32 row blocks for the codes copy
// and 32 x 1 column blocks for the codes_t copy, each with its own
// truncation-free scale.  A row block spans the 4 lanes that differ in lane
// bits 0-1, a column block the 4 lanes that differ in bits 4-5; the codes are
// packed and stored exactly as for 2D blocks, and the scales (one byte per row
// and K-group) go through LDS and leave as 4-byte words in K-tile-major order.
#include "device_common.hpp"
#include "kernels.hpp"

namespace q2d {

namespace {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f2v __attribute__((ext_vector_type(2)));
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

template <typename T>
struct Elem;

template <>
struct Elem<float> {
    static __device__ __forceinline__ uint32_t bits(const float *p) { return f_bits(*p); }
};

template <>
struct Elem<uint16_t> {
    static __device__ __forceinline__ uint32_t bits(const uint16_t *p) { return (uint32_t)*p << 16; }
};

// Round-to-nearest E2M1 pair into byte SEL of `old`: f32 sources as two
// float32 bit patterns, bf16 sources as one packed register (low half first).
template <int SEL>
__device__ __forceinline__ uint32_t rtn_pair_f32(uint32_t old, uint32_t lo, uint32_t hi, float scale)
{
    return __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(old, bits_f(lo), bits_f(hi), scale, SEL);
}
template <int SEL>
__device__ __forceinline__ uint32_t rtn_pair_bf16(uint32_t old, uint32_t packed, float scale)
{
    return __builtin_amdgcn_cvt_scalef32_pk_fp4_bf16(old, __builtin_bit_cast(bf16x2, packed), scale, SEL);
}

// Stochastic E2M1 conversion of a pair into byte `sel`; the other bytes of the
// result are not defined and the caller masks them.
__device__ __forceinline__ uint32_t sr_pair(int sel, f2v v, uint32_t seed, float scale)
{
    switch (sel) {
    case 0: return __builtin_amdgcn_cvt_scalef32_sr_pk_fp4_f32(0u, v, seed, scale, 0);
    case 1: return __builtin_amdgcn_cvt_scalef32_sr_pk_fp4_f32(0u, v, seed, scale, 1);
    case 2: return __builtin_amdgcn_cvt_scalef32_sr_pk_fp4_f32(0u, v, seed, scale, 2);
    default: return __builtin_amdgcn_cvt_scalef32_sr_pk_fp4_f32(0u, v, seed, scale, 3);
    }
}

// Stochastic E2M1 conversion of the pair (columns 2k, 2k+1) of one sub-block
// row into byte `sel` (bf16 rows are one packed register, float32 rows two bit
// patterns).  Both go through the float32 conversion: the bf16-source form
// rounds differently near the carry boundary (its parity against the rounding
// contract fails), so bf16 pairs are widened first.  As for sr_pair, the other
// bytes of the result are not defined.
template <typename T>
__device__ __forceinline__ uint32_t sr_row_pair(int sel, const uint32_t *row, uint32_t seed, float scale)
{
    f2v p;
    if constexpr (sizeof(T) == 2) p = f2v{bits_f(row[sel] << 16), bits_f(row[sel] & 0xFFFF0000u)};
    else p = f2v{bits_f(row[2 * sel]), bits_f(row[2 * sel + 1])};
    return sr_pair(sel, p, seed, scale);
}

// 8 x 8 transpose of 4-bit elements: nibble j of in[i] becomes nibble i of
// out[j].  Three exchange stages of doubling width (nibbles within row pairs,
// bytes across distance 2, half-words across distance 4).
__device__ __forceinline__ void nibble_transpose8(const uint32_t in[8], uint32_t out[8])
{
    uint32_t m[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) m[i] = in[i];
#pragma unroll
    for (int p = 0; p < 8; p += 2) {
        const uint32_t t = ((m[p] >> 4) ^ m[p + 1]) & 0x0F0F0F0Fu;
        m[p + 1] ^= t;
        m[p] ^= t << 4;
    }
#pragma unroll
    for (int i = 0; i < 8; i += (i & 1) ? 3 : 1) {         // 0, 1, 4, 5
        const uint32_t x = m[i], y = m[i + 2];
        m[i] = __builtin_amdgcn_perm(y, x, 0x06020400u);     // bytes x0 y0 x2 y2
        m[i + 2] = __builtin_amdgcn_perm(y, x, 0x07030501u); // bytes x1 y1 x3 y3
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t x = m[i], y = m[i + 4];
        out[i] = __builtin_amdgcn_perm(y, x, 0x05040100u);       // x.lo, y.lo
        out[i + 4] = __builtin_amdgcn_perm(y, x, 0x07060302u);   // x.hi, y.hi
    }
}

// Philox4x32-10 block of counter (g lo, g hi, o0, o1), one 32x32->64 multiply per
// product (v_mad_u64_u32) and one three-input xor per output word.  The offset and,
// unless WIDE, the upper counter word (0) are the same for every lane, so one product
// of each of the first two rounds is scalar: 18 vector products instead of 20 (WIDE 19).
template <bool WIDE>
__device__ __forceinline__ void philox_block(uint64_t g, uint32_t o0, uint32_t o1, uint32_t k0, uint32_t k1,
                                             uint32_t w[4])
{
    const uint64_t s0 = (uint64_t)0xCD9E8D57u * o0, p0 = (uint64_t)0xD2511F53u * (uint32_t)g;
    // round 0: words 0 and 1
    const uint32_t u0 = (uint32_t)(s0 >> 32) ^ k0 ^ (WIDE ? (uint32_t)(g >> 32) : 0u), u1 = (uint32_t)s0;
    const uint32_t v2 = (uint32_t)(p0 >> 32) ^ (o1 ^ k1), v3 = (uint32_t)p0;          // words 2 and 3
    k0 += 0x9E3779B9u; k1 += 0xBB67AE85u;
    const uint64_t s1 = (uint64_t)0xD2511F53u * u0, p1 = (uint64_t)0xCD9E8D57u * v2;
    uint32_t c0 = (uint32_t)(p1 >> 32) ^ (u1 ^ k0), c1 = (uint32_t)p1;                // round 1
    uint32_t c2 = v3 ^ ((uint32_t)(s1 >> 32) ^ k1), c3 = (uint32_t)s1;
#pragma unroll
    for (int r = 2; r < 10; ++r) {
        k0 += 0x9E3779B9u; k1 += 0xBB67AE85u;
        const uint64_t q0 = (uint64_t)0xD2511F53u * c0;
        const uint64_t q1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t n0 = xor3_uniform((uint32_t)(q1 >> 32), c1, k0);
        const uint32_t n2 = r == 2 && !WIDE ? (uint32_t)(q0 >> 32) ^ (c3 ^ k1) : xor3_uniform((uint32_t)(q0 >> 32), c3, k1);
        c0 = n0; c1 = (uint32_t)q1; c2 = n2; c3 = (uint32_t)q0;
    }
    w[0] = c0; w[1] = c1; w[2] = c2; w[3] = c3;
}

// One 128-row tile (row tile tr, column tile tc) of the quantization described
// by `a` (for a grouped tensor, `a` is already narrowed to the tile's segment).
// VEC: 0 -- element by element; 1 -- contiguous rows (stride_c == 1) of any pitch and
// alignment, read as 16-byte windows; 2 -- rows on 16-byte boundaries (with SR, also
// on storage indices that are multiples of 8).  1 and 2 with SR: every storage
// index is below 2^35, so the upper Philox counter word is 0.  3 and 4 (SR only): as 1
// and 2 with larger indices.
// SR: stochastic rounding.
// GROUPED: the rows are expert segments (see QuantArgs).  WR x WC:
// 32 x 128 strips per tile, one a wave.  ONED: 1 x 32 / 32 x 1 blocks.
template <typename T, int VECW, bool SR, int WR, bool GROUPED, int WC, bool ONED>
__device__ __forceinline__ void quantize_tile(QuantArgs a, const int64_t tr, const int64_t tc)
{
    constexpr bool WIDE = VECW > 2;
    constexpr int VEC = WIDE ? VECW - 2 : VECW;
    static_assert(SR || !WIDE, "only the draws depend on the storage index");
    constexpr int kTC = 128 * WC, kTile = 32 * WR;
    constexpr int kThreads = 64 * WR * WC;
    constexpr bool PK = sizeof(T) == 2;     // bf16: two elements per register
    constexpr int NV = PK ? 4 : 8;
    // pauses between the row loads of a large tensor's tiles (see load_sub_block).  Without
    // and with them: 196608 x 2048 bf16 RTN 236.9 / 231.7 us, 16384 x 4096 bf16 RTN 39.7 /
    // 39.1, 8192 x 4096 float32 RTN 41.6 / 41.2, SR 46.5 / 45.1, 1D RTN 47.1 / 43.8.  Better
    // without: bf16 SR (8192 x 5632 32.2 / 34.7), 1D bf16 (16384 x 4096 40.5 / 41.2) and 1D
    // float32 SR (8192 x 4096 52.0 / 52.8); strips wait for one tile's latency
    constexpr int kPace = VEC != 2 || WR != 4 || (ONED && (PK || SR)) ? 0 : PK ? (SR ? 0 : 1) : 3;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int wr = wave / WC, wc = wave % WC;
    const int64_t strip_r = tr * kTile + wr * 32;
    const int rg = lane >> 4, cc = lane & 15;
    const int64_t r0 = strip_r + 8 * rg;
    const int64_t c0 = tc * kTC + wc * 128 + 8 * cc;
    const T *x = reinterpret_cast<const T *>(a.x);

    // ---- load the 8 x 8 sub-block (0 outside R x C).  bf16: v[i][k] holds
    // columns 2k (low half) and 2k+1 (high half) of row i; fp32: bit patterns.
    uint32_t v[8][NV];
    if constexpr (VEC != 0) {
        load_sub_block<(int)sizeof(T), VEC == 2, kPace>(v, reinterpret_cast<const uint8_t *>(x + r0 * a.stride_r + c0),
                                                 a.stride_r * (int64_t)sizeof(T), a.rows - r0, a.cols - c0);
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int64_t r = r0 + i;
            auto at = [&](int64_t c) __attribute__((always_inline)) -> uint32_t {
                return r < a.rows && c < a.cols ? Elem<T>::bits(x + r * a.stride_r + c * a.stride_c) : 0u;
            };
#pragma unroll
            for (int k = 0; k < NV; ++k) v[i][k] = PK ? (at(c0 + 2 * k) >> 16) | at(c0 + 2 * k + 1) : at(c0 + k);
        }
    }
    // float32 bit pattern of element (i, j)
    auto elem = [&](int i, int j) -> uint32_t {
        if (PK) return (j & 1) ? (v[i][j >> 1] & 0xFFFF0000u) : (v[i][j >> 1] << 16);
        return v[i][j];
    };

    // ---- block maximum on |bits| (NaN > inf > finite, as unsigned integers).
    // 2D: one per lane group of 16; 1D: one per row (rm) and per column (cm).
    uint32_t am = 0;
    uint32_t rm[8], cm[8];
    if (!ONED) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int k = 0; k < NV; ++k) {
                if (PK) {
                    const uint32_t w = v[i][k] & 0x7FFF7FFFu;
                    am = max(am, max(w & 0xFFFFu, w >> 16));
                } else {
                    am = max(am, v[i][k] & 0x7FFFFFFFu);
                }
            }
        if (PK) am <<= 16;
        am = max(am, (uint32_t)__shfl_xor((int)am, 1));
        am = max(am, (uint32_t)__shfl_xor((int)am, 2));
        am = max(am, (uint32_t)__shfl_xor((int)am, 16));
        am = max(am, (uint32_t)__shfl_xor((int)am, 32));
    } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) cm[j] = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            uint32_t m = 0;
#pragma unroll
            for (int k = 0; k < NV; ++k) {
                if (PK) {
                    const uint32_t w = v[i][k] & 0x7FFF7FFFu;
                    m = max(m, max(w & 0xFFFFu, w >> 16));
                    cm[2 * k] = max(cm[2 * k], w & 0xFFFFu);
                    cm[2 * k + 1] = max(cm[2 * k + 1], w >> 16);
                } else {
                    const uint32_t w = v[i][k] & 0x7FFFFFFFu;
                    m = max(m, w);
                    cm[k] = max(cm[k], w);
                }
            }
            rm[i] = PK ? m << 16 : m;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            rm[i] = max(rm[i], (uint32_t)__shfl_xor((int)rm[i], 1));
            rm[i] = max(rm[i], (uint32_t)__shfl_xor((int)rm[i], 2));
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (PK) cm[j] <<= 16;
            cm[j] = max(cm[j], (uint32_t)__shfl_xor((int)cm[j], 16));
            cm[j] = max(cm[j], (uint32_t)__shfl_xor((int)cm[j], 32));
        }
    }
    if (WR > 1 && !ONED && !GROUPED && a.block == 64) {
        // 64 x 64 blocks: the 32 x 32 block beside it in this wave (lane bit 2), then
        // the 32-row strip of the paired wave through LDS
        __shared__ uint32_t am64[WR][2 * WC];
        am = max(am, (uint32_t)__shfl_xor((int)am, 4));
        if (rg == 0 && (cc & 7) == 0) am64[wr][wc * 2 + (cc >> 3)] = am;
        __syncthreads();
        am = max(am, am64[wr ^ 1][wc * 2 + (cc >> 3)]);
    }
    const bool finite = am < 0x7F800000u;
    const bool floor_rule = !ONED && a.floor_scale;
    const int e = floor_rule ? fp4_floor_exponent(am) : fp4_block_exponent(am);
    const float scale = bits_f((uint32_t)(127 + e) << 23);       // 2^e
    if (floor_rule && finite) {
        // saturate magnitudes above 6 * 2^e (exact in bf16: 1.5 * 2^(e+2)): the
        // magnitude bits take their minimum with the limit's, the sign stays
        // (bf16: both halves of a word at once, in place)
        const uint32_t lim = ((uint32_t)(e + 129) << 23) | 0x400000u;
        const u16x2 l16 = {(uint16_t)(lim >> 16), (uint16_t)(lim >> 16)};
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int k = 0; k < NV; ++k) {
                if (PK) {
                    const u16x2 mag = __builtin_bit_cast(u16x2, v[i][k] & 0x7FFF7FFFu);
                    v[i][k] = (v[i][k] & 0x80008000u) | __builtin_bit_cast(uint32_t, __builtin_elementwise_min(mag, l16));
                } else {
                    v[i][k] = (v[i][k] & 0x80000000u) | min(v[i][k] & 0x7FFFFFFFu, lim);
                }
            }
    }
    // scale of row i / column j of the sub-block (the block scale for 2D)
    auto rscale = [&](int i) -> float {
        return ONED ? bits_f((uint32_t)(127 + fp4_block_exponent(rm[i])) << 23) : scale;
    };
    auto cscale = [&](int j) -> float {
        return ONED ? bits_f((uint32_t)(127 + fp4_block_exponent(cm[j])) << 23) : scale;
    };

    // ---- encode: rowp[i] = eight nibbles of row i, colp[j] = eight nibbles of column j
    uint32_t rowp[8], colp[8];
    if (!SR) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            uint32_t w = 0;
            const float sc = rscale(i);
            if (PK) {
                w = rtn_pair_bf16<0>(w, v[i][0], sc);
                w = rtn_pair_bf16<1>(w, v[i][1], sc);
                w = rtn_pair_bf16<2>(w, v[i][2], sc);
                w = rtn_pair_bf16<3>(w, v[i][3], sc);
            } else {
                w = rtn_pair_f32<0>(w, elem(i, 0), elem(i, 1), sc);
                w = rtn_pair_f32<1>(w, elem(i, 2), elem(i, 3), sc);
                w = rtn_pair_f32<2>(w, elem(i, 4), elem(i, 5), sc);
                w = rtn_pair_f32<3>(w, elem(i, 6), elem(i, 7), sc);
            }
            rowp[i] = w;
        }
        if constexpr (!ONED) {
            // 2D blocks: one scale for both layouts, so the column-packed words are
            // the nibble transpose of the row-packed ones (each element converted
            // once, and the inputs are dead after the row pass)
            nibble_transpose8(rowp, colp);
        } else {
            // 1D: every column has its own scale and is converted on its own
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                uint32_t w = 0;
                const float sc = cscale(j);
                if (PK) {
                    // rows (2m, 2m+1) of column j as one packed pair
                    const int k = j >> 1;
                    auto pr = [&](int m) -> uint32_t {
                        const uint32_t lo = v[2 * m][k], hi = v[2 * m + 1][k];
                        return (j & 1) ? ((lo >> 16) | (hi & 0xFFFF0000u)) : ((lo & 0xFFFFu) | (hi << 16));
                    };
                    w = rtn_pair_bf16<0>(w, pr(0), sc);
                    w = rtn_pair_bf16<1>(w, pr(1), sc);
                    w = rtn_pair_bf16<2>(w, pr(2), sc);
                    w = rtn_pair_bf16<3>(w, pr(3), sc);
                } else {
                    w = rtn_pair_f32<0>(w, elem(0, j), elem(1, j), sc);
                    w = rtn_pair_f32<1>(w, elem(2, j), elem(3, j), sc);
                    w = rtn_pair_f32<2>(w, elem(4, j), elem(5, j), sc);
                    w = rtn_pair_f32<3>(w, elem(6, j), elem(7, j), sc);
                }
                colp[j] = w;
            }
        }
    } else {
        const uint32_t k0 = (uint32_t)a.seed, k1 = (uint32_t)(a.seed >> 32);
        const uint32_t o0 = (uint32_t)a.offset, o1 = (uint32_t)(a.offset >> 32);
        // Rows that start off a Philox block (VEC 1): a row's eight draws
        // straddle two blocks, the second of which is the first of the lane to the
        // right.  Only the strip's last lane of a row lacks a neighbour: lane i < 8 of
        // the 16 lanes of a row group computes the block behind row i for it.
        uint32_t xw[4] = {0, 0, 0, 0};
        if (VEC == 1) {
            const int64_t idx = a.index_base + (r0 + (cc & 7)) * a.stride_r + (c0 - 8 * cc) + 128;
            philox_block<WIDE>((uint64_t)idx >> 3, o0, o1, k0, k1, xw);
        }
        // the draws of row i (storage index idx_row of its first element) as
        // seeds r16 << 16
        auto row_draws = [&](auto ic, int64_t idx_row, uint32_t s16[8]) __attribute__((always_inline)) {
            constexpr int i = decltype(ic)::value;
            uint32_t w[8] = {0, 0, 0, 0, 0, 0, 0, 0};
            if (VEC) {
                philox_block<WIDE>((uint64_t)idx_row >> 3, o0, o1, k0, k1, w);
                if constexpr (VEC == 1) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        // row_newbcast:i, then row_shl:1 (lane 15 keeps the first operand)
                        const int edge = __builtin_amdgcn_update_dpp(0, (int)xw[j], 0x150 + i, 0xF, 0xF, false);
                        w[4 + j] = (uint32_t)__builtin_amdgcn_update_dpp(edge, (int)w[j], 0x101, 0xF, 0xF, false);
                    }
                    // halves sh .. sh + 7 of the sixteen; sh is the same for every lane
                    // (r0 and c0 are multiples of 8)
                    const int sh = (int)((a.index_base + i * a.stride_r) & 7);
                    // (both operands as values: a choice between array elements would keep
                    // the array in scratch memory)
#pragma unroll
                    for (int j = 0; j < 6; ++j) { const uint32_t a0 = w[j], a1 = w[j + 2]; w[j] = (sh & 4) ? a1 : a0; }
#pragma unroll
                    for (int j = 0; j < 5; ++j) { const uint32_t a0 = w[j], a1 = w[j + 1]; w[j] = (sh & 2) ? a1 : a0; }
#pragma unroll
                    for (int j = 0; j < 4; ++j) { const uint32_t a0 = w[j], a1 = w[j + 1]; w[j] = (sh & 1) ? (a0 >> 16) | (a1 << 16) : a0; }
                }
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                uint32_t r;
                if (VEC) {
                    r = (j & 1) ? (w[j >> 1] & 0xFFFF0000u) : (w[j >> 1] << 16);
                } else {
                    const uint64_t idx = (uint64_t)(a.index_base + (r0 + i) * a.stride_r + (c0 + j) * a.stride_c);
                    r = sr_draw(idx, k0, k1, o0, o1) << 16;
                }
                s16[j] = r;
            }
        };
        int64_t idx0 = a.index_base + r0 * a.stride_r + c0;
        if constexpr (!ONED) {
            // 2D blocks: both layouts share the block scale, so every element is
            // converted once, row by row; the column-packed words are the 8 x 8
            // nibble transpose of the row-packed ones
            unroll<8>([&](auto ic) __attribute__((always_inline)) {
                constexpr int i = decltype(ic)::value;
                uint32_t s16[8];
                row_draws(ic, idx0, s16);
                idx0 += a.stride_r;
                uint32_t w = 0;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    // element 2k from a conversion with its draw, element 2k + 1 from
                    // one with its own (the second element reads seed << 1)
                    const uint32_t lo = sr_row_pair<T>(k, v[i], s16[2 * k], scale);
                    const uint32_t hi = sr_row_pair<T>(k, v[i], s16[2 * k + 1] >> 1, scale);
                    w |= ((lo & 0x0F0F0F0Fu) | (hi & 0xF0F0F0F0u)) & (0xFFu << (8 * k));
                }
                rowp[i] = w;
            });
            nibble_transpose8(rowp, colp);
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) { rowp[i] = 0; colp[i] = 0; }
            unroll<4>([&](auto mc) __attribute__((always_inline)) {
                constexpr int m = decltype(mc)::value;
                // draws of rows 2m and 2m+1 as seeds r16 << 16
                uint32_t s16[2][8];
                unroll<2>([&](auto hc) __attribute__((always_inline)) {
                    row_draws(std::integral_constant<int, 2 * m + decltype(hc)::value>{}, idx0, s16[decltype(hc)::value]);
                    idx0 += a.stride_r;
                });
                // rows 2m and 2m+1: pairs (2k, 2k+1) into byte k
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int i = 2 * m + h;
                    const float sc = rscale(i);
                    uint32_t acc = 0;
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const f2v pr = {bits_f(elem(i, 2 * k)), bits_f(elem(i, 2 * k + 1))};
                        const uint32_t lo = sr_pair(k, pr, s16[h][2 * k], sc);
                        const uint32_t hi = sr_pair(k, pr, s16[h][2 * k + 1] >> 1, sc);
                        acc |= (lo & (0x0Fu << (8 * k))) | (hi & (0xF0u << (8 * k)));
                    }
                    rowp[i] = acc;
                }
                // every column: rows (2m, 2m+1) into byte m, each with its column's scale
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const f2v pr = {bits_f(elem(2 * m, j)), bits_f(elem(2 * m + 1, j))};
                    const float sc = cscale(j);
                    const uint32_t lo = sr_pair(m, pr, s16[0][j], sc);
                    const uint32_t hi = sr_pair(m, pr, s16[1][j] >> 1, sc);
                    colp[j] |= (lo & (0x0Fu << (8 * m))) | (hi & (0xF0u << (8 * m)));
                }
            });
        }
    }
    if (!ONED && !finite) {
#pragma unroll
        for (int i = 0; i < 8; ++i) { rowp[i] = 0; colp[i] = 0; }
    }
    if (ONED) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (rm[i] >= 0x7F800000u) rowp[i] = 0;
            if (cm[i] >= 0x7F800000u) colp[i] = 0;
        }
    }

    // ---- stores through LDS: 16 bytes per lane, codes rows r < store_rows as
    // WC * 64-byte runs, codes_t rows c < C as 64-byte runs
    __shared__ uint32_t st_r[kTile][16 * WC + 1];
    __shared__ uint32_t st_c[kTC][4 * WR + 1];
    __shared__ uint8_t st_rs[ONED ? kTile : 1][4 * WC];     // 1D: row scales of the tile
    __shared__ uint8_t st_cs[ONED ? kTC : 1][WR];            // 1D: column scales of the tile
    {
        // the lane geometry again, from the thread index: cheaper than keeping it
        // live across the conversion (the opaque copy stops the compiler from
        // reusing the values computed at the top)
        int t = threadIdx.x;
        asm volatile("" : "+v"(t));
        const int wr = (t >> 6) / WC, wc = (t >> 6) % WC, rg = (t & 63) >> 4, cc = t & 15;
        const int rl = wr * 32 + 8 * rg;
#pragma unroll
        for (int i = 0; i < 8; ++i) st_r[rl + i][wc * 16 + cc] = rowp[i];
#pragma unroll
        for (int j = 0; j < 8; ++j) st_c[wc * 128 + 8 * cc + j][wr * 4 + rg] = colp[j];
        if (ONED) {
            auto sbyte = [](uint32_t m) -> uint8_t {
                return m < 0x7F800000u ? (uint8_t)(127 + fp4_block_exponent(m)) : (uint8_t)0xFF;
            };
            if ((cc & 3) == 0) {
#pragma unroll
                for (int i = 0; i < 8; ++i) st_rs[rl + i][wc * 4 + (cc >> 2)] = sbyte(rm[i]);
            }
            if (rg == 0) {
#pragma unroll
                for (int j = 0; j < 8; ++j) st_cs[wc * 128 + 8 * cc + j][wr] = sbyte(cm[j]);
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int item = threadIdx.x + kThreads * q;
        if (a.codes) {
            const int line = item / (4 * WC), part = item % (4 * WC);
            const int64_t r = tr * kTile + line;
            if (r < a.store_rows && tc * kTC + part * 32 < a.cols_pad) {
                const uint4 w = make_uint4(st_r[line][4 * part], st_r[line][4 * part + 1],
                                           st_r[line][4 * part + 2], st_r[line][4 * part + 3]);
                *reinterpret_cast<uint4 *>(a.codes + r * a.ld_codes + tc * (kTC / 2) + part * 16) = w;
            }
        }
        if (a.codes_t) {
            const int line = item / WR, part = item % WR;
            const int64_t c = tc * kTC + line;
            if (c < a.cols) {
                const uint4 w = make_uint4(st_c[line][4 * part], st_c[line][4 * part + 1],
                                           st_c[line][4 * part + 2], st_c[line][4 * part + 3]);
                *reinterpret_cast<uint4 *>(a.codes_t + c * a.ld_codes_t + tr * (kTile / 2) + part * 16) = w;
            }
        }
    }
    if (ONED) {
        // scale words, K-tile major: row r's word of each 128-column strip k at
        // (k, r); column c's word of this 128-row tile at (tr, c)
        const int t = threadIdx.x;
        if (t < kTile) {
            const int64_t r = tr * kTile + t;
            if (a.scales && r < a.rows) {
#pragma unroll
                for (int w = 0; w < WC; ++w)
                    if (tc * kTC + w * 128 < a.cols_pad)
                        *reinterpret_cast<uint32_t *>(a.scales + ((tc * kTC + w * 128) / 128) * a.ld_scales + 4 * r) =
                            *reinterpret_cast<const uint32_t *>(&st_rs[t][4 * w]);
            }
        } else if (t >= kThreads - kTC) {
            const int cl = t - (kThreads - kTC);
            const int64_t c = tc * kTC + cl;
            if (a.scales_t && c < a.cols)
                *reinterpret_cast<uint32_t *>(a.scales_t + tr * a.ld_scales_t + 4 * c) =
                    *reinterpret_cast<const uint32_t *>(&st_cs[cl][0]);
        }
        return;
    }
    // the block's scale byte, from one lane per 32 x 32 block (lane geometry
    // recomputed, as above)
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    const int tw = t >> 6, tl = t & 63;
    if (tc * kTC + (tw % WC) * 128 < a.cols_pad && (tl >> 4) == 0 && (tl & 3) == 0) {
        const uint8_t sbyte = finite ? (uint8_t)(e + 127) : (uint8_t)0xFF;
        const int64_t rb = (tr * kTile + (tw / WC) * 32) >> 5, cb = (tc * kTC + (tw % WC) * 128 + 8 * (tl & 15)) >> 5;
        if (a.scales && rb < a.nbr) a.scales[rb * a.ld_scales + cb] = sbyte;
        if (a.scales_t && cb < a.nbc) a.scales_t[cb * a.ld_scales_t + rb] = sbyte;
    }
}

// A lane holds its 8 x 8 sub-block (32 registers of bf16 pairs, 64 of float32)
// and converts each element once, so the bf16 2D variants take 42-61 VGPRs (grouped
// 69-85) with nothing spilled.  Of the bounds below (at most 168 VGPRs for stochastic
// rounding, whose Philox latency needs three waves per SIMD; at most 128 for round to
// nearest) only the float32 round-to-nearest variants reach theirs.
// Spilled registers cost HBM writes here, not only latency: every wave's spill
// lines end up evicted by the streaming traffic.
template <typename T, int VEC, bool SR, int WR, bool GROUPED, int WC, bool ONED, bool PAIR>
__global__ __launch_bounds__(64 * WR * WC)
__attribute__((amdgpu_waves_per_eu(VEC && SR ? 3 : (VEC ? 4 : 1)))) void fp4_quantize_kernel(QuantArgs a, QuantArgs a2, uint32_t first)
{
    static_assert(!(ONED && GROUPED), "grouped tensors use 2D blocks");
    static_assert(WR == 4 || (WR == 1 && !ONED && !GROUPED), "a strip of its own: dense 2D blocks of 32");
    constexpr int kTC = 128 * WC, kTile = 32 * WR;
    if constexpr (GROUPED) {
        const int64_t tiles_c = (a.cols_pad + kTC - 1) / kTC;
        // padded start rows of the segments, built once per workgroup; the
        // workgroup then walks the row tiles of all segments (tile = blockIdx.x,
        // + gridDim.x, ...) and narrows `a` to each tile's segment
        __shared__ int32_t pad_start[kMaxSegs + 1];
        __shared__ int32_t off[kMaxSegs + 1];
        if ((threadIdx.x >> 6) == 0) {
            wave_offsets(a.nseg, a.seg_offsets, a.rows, off);
            __builtin_amdgcn_wave_barrier();
            wave_prefix(a.nseg, [&](int i) { return (off[i + 1] - off[i] + 127) / 128 * 128; }, pad_start);
        }
        __syncthreads();
        const int64_t tiles = (int64_t)(pad_start[a.nseg] / kTile) * tiles_c;
        for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
            const int64_t rt = tile / tiles_c, tc = tile - rt * tiles_c;
            const int32_t prow = (int32_t)(rt * kTile);
            // the tile's segment (wave-uniform: scalar registers for the narrowed arguments)
            const int e = __builtin_amdgcn_readfirstlane(seg_search(pad_start, a.nseg, prow));
            const int32_t o_e = __builtin_amdgcn_readfirstlane(off[e]);
            const int64_t r_begin = o_e, n_e = (int64_t)__builtin_amdgcn_readfirstlane(off[e + 1]) - o_e;
            const int32_t p_e = __builtin_amdgcn_readfirstlane(pad_start[e]);
            QuantArgs b = a;
            b.x = reinterpret_cast<const uint8_t *>(a.x) + r_begin * a.stride_r * (int64_t)sizeof(T);
            b.index_base += r_begin * a.stride_r;
            b.rows = n_e;
            b.store_rows = (n_e + 127) / 128 * 128;
            b.nbr = b.store_rows / 32;
            if (b.codes) b.codes += (int64_t)p_e * a.ld_codes;
            if (b.codes_t) b.codes_t += p_e / 2;
            if (b.scales) b.scales += (int64_t)(p_e / 32) * a.ld_scales;
            if (b.scales_t) b.scales_t += p_e / 32;
            quantize_tile<T, VEC, SR, WR, GROUPED, WC, ONED>(b, (prow - p_e) / kTile, tc);
            __syncthreads();                // the tile's LDS staging is reused by the next
        }
    } else {
        // PAIR: workgroups from `first` on belong to the second tensor of the launch.  A
        // launch of one tensor has a kernel of its own: the choice at the start of each
        // workgroup cost it 2 % (16384 x 12288 bf16 SR 119.1 us against 116.7 for the
        // one-tensor kernel before it, alternating; without it 115.3 against 115.5)
        const bool second = PAIR && blockIdx.x >= first;
        const QuantArgs &b = second ? a2 : a;
        const uint32_t tile = blockIdx.x - (second ? first : 0u), tiles_c = (uint32_t)((b.cols_pad + kTC - 1) / kTC);
        const uint32_t tr = tile / tiles_c;
        quantize_tile<T, VEC, SR, WR, GROUPED, WC, ONED>(b, tr, tile - tr * tiles_c);
    }
}

// 128 x 256 tiles of a quantization
int64_t tiles_of(const QuantArgs &a) { return (a.rows_pad / 128) * ((a.cols_pad + 255) / 256); }

template <typename T, int VEC, bool SR, bool G, int WR, int WC, bool ONED>
hipError_t launch_w(const QuantArgs &a, const QuantArgs *a2, hipStream_t s)
{
    auto blocks = [](const QuantArgs &q) { return (q.rows_pad / (32 * WR)) * ((q.cols_pad + 128 * WC - 1) / (128 * WC)); };
    int64_t nb = blocks(a);
    // grouped: each workgroup walks several tiles, so that the segment table is
    // built once per few tiles (the bound covers every padded segment's tiles);
    // 8 per CU keeps the last round of tiles short
    if (G) nb = nb < 8 * (int64_t)cu_count() ? nb : 8 * (int64_t)cu_count();
    const int64_t all = nb + (a2 ? blocks(*a2) : 0);
    if (all > INT32_MAX) return hipErrorInvalidValue;           // (beyond any device's memory)
    // An input of 96 MB or more streams from HBM, and two workgroups (16 waves) a CU
    // read it faster than the three or four that fit: 124.1 against 127.2 us for 16384 x
    // 12288 bf16, round to nearest (123.0 against 133.4, stochastic); below that size
    // more waves hide more latency (8192 x 5632 SR: 32.4 against 33.8 us).  Unused
    // dynamic LDS fills a workgroup's share up to half of the CU's.  The 1D kernels' own
    // registers already hold them at two (41.5 us for 16384 x 4096 bf16, with or without
    // the fill).  64 x 64 blocks rounded stochastically wait for their maximum at a
    // barrier between the loads and a long conversion, and more workgroups fill that wait:
    // 16384 x 4096 43.1 us without the fill, 47.8 with it, 16384 x 12288 129.6 / 134.1.
    constexpr int kHalf = 81920, kStatic = G ? 42516 : 34368;   // the kernel's own LDS
    auto streams = [](const QuantArgs &q) { return q.rows * q.cols * (int64_t)sizeof(T) >= (int64_t(96) << 20); };
    const bool two = WR == 4 && !ONED && !(SR && a.block == 64) && (streams(a) || (a2 && streams(*a2)));
    const unsigned lds = two ? (unsigned)(kHalf - kStatic) : 0;
    const dim3 grid((unsigned)all), block(64 * WR * WC);
    if constexpr (!G && !ONED && VEC <= 2) {
        if (a2) {
            hipLaunchKernelGGL((fp4_quantize_kernel<T, VEC, SR, WR, G, WC, ONED, true>), grid, block, lds, s, a, *a2, (uint32_t)nb);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((fp4_quantize_kernel<T, VEC, SR, WR, G, WC, ONED, false>), grid, block, lds, s, a, a, (uint32_t)nb);
    return hipGetLastError();
}

constexpr int64_t kStripTiles = 128;

template <typename T, int VEC, bool SR, bool G, bool ONED>
hipError_t launch_t(const QuantArgs &a, const QuantArgs *a2, hipStream_t s)
{
    // 128 x 256 tiles of 8 waves in both rounding modes: the row-packed codes leave
    // as whole 128-byte lines.  Up to kStripTiles of them, one wave a workgroup (a 32 x
    // 128 strip): a strip alone on its SIMD takes 3-4 us where a tile's two waves a
    // SIMD take 6 (128 x 256 float32 SR 5.8 -> 4.1 us, 1024 x 2048 bf16 SR 6.3 -> 4.7;
    // 2000 x 2048, 128 tiles: 6.8 -> 5.8; 2048 x 4096, 256 tiles: 9.1 -> 9.7)
    if constexpr (!G && !ONED) {
        if (a.block == 32 && (!a2 || a2->block == 32) && tiles_of(a) + (a2 ? tiles_of(*a2) : 0) <= kStripTiles)
            return launch_w<T, VEC, SR, G, 1, 1, ONED>(a, a2, s);
    }
    return launch_w<T, VEC, SR, G, 4, 2, ONED>(a, a2, s);
}

template <typename T, bool G, bool ONED>
hipError_t launch_dtype(const QuantArgs &a, const QuantArgs *a2, int vec, bool sr, hipStream_t s)
{
    switch (vec) {
    case 4: return launch_w<T, 4, true, G, 4, 2, ONED>(a, nullptr, s);
    case 3: return launch_w<T, 3, true, G, 4, 2, ONED>(a, nullptr, s);
    case 2: return sr ? launch_t<T, 2, true, G, ONED>(a, a2, s) : launch_t<T, 2, false, G, ONED>(a, a2, s);
    case 1: return sr ? launch_t<T, 1, true, G, ONED>(a, a2, s) : launch_t<T, 1, false, G, ONED>(a, a2, s);
    default: return sr ? launch_t<T, 0, true, G, ONED>(a, a2, s) : launch_t<T, 0, false, G, ONED>(a, a2, s);
    }
}

// How a tensor's rows can be read: contiguous rows of any pitch and alignment take
// the vector loads; 2: rows start on 16-byte boundaries and, for SR, on Philox blocks.
// SR from storage index 2^35 on (a Philox block past the end included) needs the upper
// counter word: 3 and 4, so that the smaller tensors do not pay for it (4096 x 4096 bf16
// rows that reach past that index: 15.5 us, element by element 49.4).
int vec_of(const QuantArgs &a, int dtype_bytes, bool sr)
{
    if (a.stride_c != 1) return 0;
    const bool aligned = reinterpret_cast<uintptr_t>(a.x) % 16 == 0 && (a.stride_r * dtype_bytes) % 16 == 0;
    const bool a8 = a.stride_r % 8 == 0 && a.index_base % 8 == 0;
    const int vec = aligned && (a8 || !sr) ? 2 : a.cols >= 8 ? 1 : 0;
    const bool wide = sr && a.index_base + a.rows * a.stride_r + a.cols >= (int64_t(1) << 35) - 4096;
    return vec && wide ? vec + 2 : vec;
}

}  // namespace

hipError_t launch_fp4_quantize(const QuantArgs &a, int dtype_bytes, bool sr, bool oned, hipStream_t stream)
{
    const int vec = vec_of(a, dtype_bytes, sr);
    if (a.also) {
        // Two tensors in one launch: the second one's tiles fill the CUs that the
        // first one's last round leaves, and a launch (3 us of the host, 2-3 us of the
        // device) is saved: 8192 x 2048 and 5632 x 2048 bf16 SR 30.9 -> 27 us.  Beyond
        // 128 MB together they are better read one after the other (16384 x 4096 and
        // 12288 x 4096: 4 us slower in one launch).
        QuantArgs one = a;
        one.also = nullptr;
        const int64_t bytes = (a.rows * a.cols + a.also->rows * a.also->cols) * dtype_bytes;
        if (vec != vec_of(*a.also, dtype_bytes, sr) || vec > 2 || bytes > (int64_t(128) << 20)) {
            const hipError_t e = launch_fp4_quantize(one, dtype_bytes, sr, false, stream);
            return e != hipSuccess ? e : launch_fp4_quantize(*a.also, dtype_bytes, sr, false, stream);
        }
        return dtype_bytes == 4 ? launch_dtype<float, false, false>(one, a.also, vec, sr, stream)
                                : launch_dtype<uint16_t, false, false>(one, a.also, vec, sr, stream);
    }
    const bool grouped = a.seg_offsets != nullptr;
    if (oned) {
        if (grouped) return hipErrorInvalidValue;
        return dtype_bytes == 4 ? launch_dtype<float, false, true>(a, nullptr, vec, sr, stream)
                                : launch_dtype<uint16_t, false, true>(a, nullptr, vec, sr, stream);
    }
    if (dtype_bytes == 4)
        return grouped ? launch_dtype<float, true, false>(a, nullptr, vec, sr, stream)
                       : launch_dtype<float, false, false>(a, nullptr, vec, sr, stream);
    return grouped ? launch_dtype<uint16_t, true, false>(a, nullptr, vec, sr, stream)
                   : launch_dtype<uint16_t, false, false>(a, nullptr, vec, sr, stream);
}

}  // namespace q2d
