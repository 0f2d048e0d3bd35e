// Device-side helpers shared by the libq2d kernels (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>
#include <utility>

namespace q2d {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));

typedef unsigned int u4v __attribute__((ext_vector_type(4)));

// 16-byte streaming load: a quantizer's input is read once, so it should not
// displace cache lines that are reused
__device__ __forceinline__ uint4 load_stream16(const uint8_t *p)
{
    const u4v v = __builtin_nontemporal_load(reinterpret_cast<const u4v *>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
}

// 16-byte load from an address aligned to 4 bytes only; cached, since neighbouring
// loads meet in one line
typedef u4v u4v_a4 __attribute__((aligned(4)));
__device__ __forceinline__ uint4 load_words16(const uint8_t *p)
{
    const u4v v = *reinterpret_cast<const u4v_a4 *>(p);
    return make_uint4(v.x, v.y, v.z, v.w);
}

// f(std::integral_constant<int, 0>) ... f(std::integral_constant<int, N - 1>), in order
template <typename F, int... Is>
__device__ __forceinline__ void unroll_seq(F &&f, std::integer_sequence<int, Is...>)
{
    (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void unroll(F &&f)
{
    unroll_seq(f, std::make_integer_sequence<int, N>{});
}

__device__ __forceinline__ float bits_f(uint32_t u) { return __uint_as_float(u); }
__device__ __forceinline__ uint32_t f_bits(float f) { return __float_as_uint(f); }

// a ^ b ^ k in one v_bitop3_b32 (truth table 0x96, symmetric in its inputs);
// k is wave-uniform
__device__ __forceinline__ uint32_t xor3_uniform(uint32_t a, uint32_t b, uint32_t k)
{
    uint32_t r;
    asm("v_bitop3_b32 %0, %1, %2, %3 bitop3:0x96" : "=v"(r) : "v"(a), "v"(b), "s"(k));
    return r;
}

// Philox4x32 with 10 rounds (Salmon, Moraes, Dror, Shaw, SC 2011): two 32x32->64
// multiplies per round, key bumped by the Weyl constants between rounds.  The
// key is wave-uniform, so the bumps stay scalar.  Each product is formed as one
// 64-bit result (v_mad_u64_u32) rather than separate low and high multiplies:
// about a quarter fewer cycles per block on gfx950.
__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                              uint32_t k0, uint32_t k1, uint32_t out[4])
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r) { k0 += 0x9E3779B9u; k1 += 0xBB67AE85u; }
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0, p1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t lo0 = (uint32_t)p0, hi0 = (uint32_t)(p0 >> 32);
        const uint32_t lo1 = (uint32_t)p1, hi1 = (uint32_t)(p1 >> 32);
        const uint32_t n0 = xor3_uniform(hi1, c1, k0);
        const uint32_t n2 = xor3_uniform(hi0, c3, k1);
        c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
    }
    out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

// The 16-bit stochastic-rounding draw of storage index idx: half (idx & 1) of
// word (idx & 7) >> 1 of the block for counter (idx >> 3, offset).
__device__ __forceinline__ uint32_t sr_draw(uint64_t idx, uint32_t k0, uint32_t k1,
                                            uint32_t off_lo, uint32_t off_hi)
{
    const uint64_t g = idx >> 3;
    uint32_t w[4];
    philox4x32_10((uint32_t)g, (uint32_t)(g >> 32), off_lo, off_hi, k0, k1, w);
    const uint32_t j = (uint32_t)idx & 7u;
    const uint32_t word = (j & 4u) ? ((j & 2u) ? w[3] : w[2]) : ((j & 2u) ? w[1] : w[0]);
    return (word >> ((j & 1u) * 16u)) & 0xFFFFu;
}

// Truncation-free E2M1 block exponent from the block maximum's float32 bit
// pattern (sign cleared): the smallest e with 6 * 2^e >= M.  For M = 1.f * 2^p
// that is p - 2, plus one when f > 1.5; subnormal and tiny maxima clamp to -127.
__device__ __forceinline__ int fp4_block_exponent(uint32_t amax_bits)
{
    const int eb = (int)(amax_bits >> 23);
    if (eb == 0) return -127;
    const int e = eb - 129 + ((amax_bits & 0x7FFFFFu) > 0x400000u ? 1 : 0);
    return e < -127 ? -127 : e;
}

// Scale rule of the truncation-free ablation (the shared-exponent rule of the
// OCP microscaling formats): e = floor(log2 M) - 2, the exponent of M's leading
// bit minus E2M1's largest exponent (6 = 1.5 * 2^2), clamped to -127.  Block
// maxima with a mantissa above 1.5 then exceed 6 * 2^e and saturate to +-6.
__device__ __forceinline__ int fp4_floor_exponent(uint32_t amax_bits)
{
    const int e = (int)(amax_bits >> 23) - 129;
    return e < -127 ? -127 : e;
}

// Same rule for E4M3 (largest magnitude 448 = 1.75 * 2^8): e = p - 8, plus one
// when f > 1.75.
__device__ __forceinline__ int fp8_block_exponent(uint32_t amax_bits)
{
    const int eb = (int)(amax_bits >> 23);
    if (eb == 0) return -127;
    const int e = eb - 135 + ((amax_bits & 0x7FFFFFu) > 0x600000u ? 1 : 0);
    return e < -127 ? -127 : e;
}

// 2^-e as a float for e in [-127, 126].
__device__ __forceinline__ float inv_pow2(int e) { return bits_f((uint32_t)(127 - e) << 23); }

// E4M3FN code magnitude of v in [0, 448], round to nearest even.  Below 2^-6
// the spacing is 2^-9 (subnormals); above it the 3-bit mantissa is rounded on
// the float32 bit pattern.
__device__ __forceinline__ uint32_t e4m3_rne(float v)
{
    if (v < 0.015625f) return (uint32_t)(int)__builtin_rintf(v * 512.0f);
    uint32_t b = f_bits(v);
    b += 0x7FFFFu + ((b >> 20) & 1u);
    return (b >> 20) - (120u << 3);
}

__device__ __forceinline__ float bf16_to_f(uint16_t h) { return bits_f((uint32_t)h << 16); }

__device__ __forceinline__ uint16_t f_to_bf16_rne(float f)
{
    uint32_t b = f_bits(f);
    if ((b & 0x7F800000u) == 0x7F800000u) return (uint16_t)((b >> 16) | ((b & 0xFFFFu) ? 0x40u : 0u));
    b += 0x7FFFu + ((b >> 16) & 1u);
    return (uint16_t)(b >> 16);
}

// A lane's 8 x 8 sub-block of a matrix with contiguous rows of `pitch` bytes, from
// address p, as 32-bit words (E = 2: bf16 pairs, v[i][k] holds columns 2k and
// 2k + 1 of row i; E = 4: float32).  rows, cols: what the matrix has from p on (at
// most 0: nothing); words outside it are 0.
//
// ALIGNED: p and the pitch are multiples of 16 bytes.  Otherwise loads of aligned
// 4-byte words, and a matrix of at least 8 columns.
//
// No load is skipped, so that all are in flight together: past the edge they go to
// the matrix's last row and its last 16-byte piece (ALIGNED: the one that holds the
// last column) or last 8 columns, and the words are put in place afterwards.
//
// PACE: pauses of 16 cycles between the rows of interior waves.  The rows of a wide
// matrix lie a power of two apart more often than not, and eight of them asked for
// back to back queue on few memory channels.
template <int E, bool ALIGNED, int PACE, int NV>
__device__ __forceinline__ void load_sub_block(uint32_t (&v)[8][NV], const uint8_t *p, int64_t pitch, int64_t rows,
                                               int64_t cols)
{
    static_assert(NV == 2 * E, "8 elements");
    constexpr int NB = E / 2;                   // 16-byte pieces of a row
    const bool edge = __builtin_amdgcn_ballot_w64(rows < 8 || cols < 8) != 0;
    // Rows step from one to the next by adding the pitch (a 64-bit product for each row
    // held the loads back: 64 x 64 blocks, whose conversion waits for all of them at a
    // barrier, 16384 x 12288 bf16 SR 143.0 us, now 134.2).
    const int64_t last = (cols * E - 1) & ~int64_t(15);
    auto load = [&](auto edge_c) __attribute__((always_inline)) {
        constexpr bool EDGE = decltype(edge_c)::value;
        const uint8_t *r = p;
        if (EDGE && !ALIGNED && cols < 8) r += (cols - 8) * E;
        if (EDGE && rows < 1) r += (rows - 1) * pitch;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
#pragma unroll
            for (int t = 0; t < NB; ++t) {
                uint4 x;
                if constexpr (ALIGNED) {
                    x = load_stream16(r + (!EDGE || 16 * t <= last ? 16 * t : last));
                } else if constexpr (E == 4) {
                    x = load_words16(r + 16 * t);
                } else {
                    // the words that hold the eight bf16 values: four from the word of the
                    // first one on and, if that is its upper half, the one behind them
                    // (16-byte loads at 2-byte addresses run at less than half the rate)
                    const bool odd = (reinterpret_cast<uintptr_t>(r) & 2) != 0;
                    const uint8_t *rw = odd ? r - 2 : r;
                    const uint4 y = load_words16(rw);
                    const uint32_t z = *reinterpret_cast<const uint32_t *>(odd ? rw + 16 : rw + 12);
                    x = odd ? make_uint4((y.x >> 16) | (y.y << 16), (y.y >> 16) | (y.z << 16), (y.z >> 16) | (y.w << 16),
                                         (y.w >> 16) | (z << 16))
                            : y;
                }
                v[i][4 * t] = x.x; v[i][4 * t + 1] = x.y; v[i][4 * t + 2] = x.z; v[i][4 * t + 3] = x.w;
            }
            r += !EDGE || i + 1 < rows ? pitch : 0;
            if constexpr (PACE > 0 && !EDGE) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int n = 0; n < PACE; ++n) asm volatile("s_nop 15");
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    // interior waves straight on: between GEMMs a kernel's code is not cached, and a jump
    // over the edge's loads costs 0.3 us of 15 (4096 x 4096 bf16 1D)
    if (__builtin_expect(!edge, 1)) {
        load(std::false_type{});
        return;
    }
    load(std::true_type{});
    const int nr = rows < 8 ? (int)(rows < 0 ? 0 : rows) : 8, nc = cols < 8 ? (int)(cols < 0 ? 0 : cols) : 8;
    if (!ALIGNED) {
        // the lane that holds the last columns read 8 - nc earlier ones before them
        const int s = (8 - nc) & 7;
        // words move down by D if `on`.  Both operands are values before the choice: a
        // choice between two array elements takes their addresses and puts the whole
        // array into scratch memory, for interior waves too (272 bytes a lane for
        // float32; 4096 x 4097 float32, round to nearest, 55.4 us with it, 16.2 without)
        auto down = [&](auto dc, bool on) __attribute__((always_inline)) {
            constexpr int D = decltype(dc)::value;
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int k = 0; k + D < NV; ++k) {
                    const uint32_t here = v[i][k], there = v[i][k + D];
                    v[i][k] = on ? there : here;
                }
        };
        down(std::integral_constant<int, E>{}, (s & 4) != 0);
        down(std::integral_constant<int, E / 2>{}, (s & 2) != 0);
        if constexpr (E == 4) {
            down(std::integral_constant<int, 1>{}, (s & 1) != 0);
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int k = 0; k < NV; ++k) {
                    const uint32_t here = v[i][k], next = k + 1 < NV ? v[i][k + 1 < NV ? k + 1 : k] : 0u;
                    v[i][k] = (s & 1) ? (here >> 16) | (next << 16) : here;
                }
        }
    }
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const uint32_t keep = E == 4 ? (k < nc ? ~0u : 0u)
                                     : (2 * k < nc ? 0xFFFFu : 0u) | (2 * k + 1 < nc ? 0xFFFF0000u : 0u);
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i][k] = i < nr ? v[i][k] & keep : 0u;
    }
}

// ---- grouped (MoE) segment tables, built per workgroup in LDS

constexpr int kMaxSegs = 1024;

// Inclusive prefix over `n` values produced by f(i) (i < n), written to out[1..n]
// with out[0] = 0.  Run by one full wave; n <= kMaxSegs.
template <typename F>
__device__ __forceinline__ void wave_prefix(int n, F f, int32_t *out)
{
    const int lane = threadIdx.x & 63;
    int32_t carry = 0;
    if (lane == 0) out[0] = 0;
    for (int base = 0; base < n; base += 64) {
        const int i = base + lane;
        int32_t v = i < n ? f(i) : 0;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int32_t u = __shfl_up(v, d);
            if (lane >= d) v += u;
        }
        if (i < n) out[i + 1] = carry + v;
        carry += __shfl(v, 63);
    }
}

// Segment offsets as the kernels use them: out[i] = min(max(0, off[0], ..,
// off[i]), total) for i = 0 .. n.  A valid table (ascending from 0 to total) is
// unchanged; any other one becomes ascending and inside [0, total], so the
// segments stay inside the input rows and their padded sizes inside the
// grouped capacity.  Run by one full wave; n <= kMaxSegs.
__device__ __forceinline__ void wave_offsets(int n, const int64_t *off, int64_t total, int32_t *out)
{
    const int lane = threadIdx.x & 63;
    int32_t carry = 0;
    for (int base = 0; base <= n; base += 64) {
        const int i = base + lane;
        int64_t o = i <= n ? off[i] : 0;
        o = o < 0 ? 0 : (o > total ? total : o);
        int32_t v = (int32_t)o;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int32_t u = __shfl_up(v, d);
            if (lane >= d) v = max(v, u);
        }
        v = max(v, carry);
        if (i <= n) out[i] = v;
        carry = __shfl(v, 63);
    }
}

// Largest e < n with table[e] <= x (table ascending, table[0] = 0 <= x).
__device__ __forceinline__ int seg_search(const int32_t *table, int n, int32_t x)
{
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (table[mid] <= x) lo = mid; else hi = mid - 1;
    }
    return lo;
}

}  // namespace q2d
