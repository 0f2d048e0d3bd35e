// Device helpers shared by the GEMM kernels: operand formats, the XCD-aware tile
// order, global -> LDS loads and their hand-counted waits.
#pragma once

#include <type_traits>
#include <utility>
#include "device_common.hpp"
#include "kernels.hpp"

namespace q2d {
namespace {

constexpr int BK = 128;                     // K extents are padded to this
constexpr int kThreads = 256;
constexpr int kXcds = 8;

template <int FMT>
struct Fmt;

// Operand placement measured on gfx950 for v_mfma_scale_f32_32x32x64_f8f6f4:
// with E2M1 operands (4 VGPRs) lane l holds 32 consecutive K values of K-group
// l / 32; with E4M3 operands (8 VGPRs) the first 16 bytes of every lane belong
// to K-group 0 and the last 16 bytes to K-group 1, the two lane halves splitting
// each group.  In both cases lane half h supplies the scale of K-group h.
//
// LDS stages hold 64 bytes of every operand row (128 E2M1 or 64 E4M3 values);
// lane half h reads the 16-byte chunks h and 2 + h of a row: for E2M1 the two
// K-substeps of 64 values, for E4M3 the two register halves of one.
template <>
struct Fmt<kFmtFp4Block2D> {
    static constexpr int kStepK = 128;            // K values per 64-byte row stage
    static constexpr int kCbsz = 4;               // E2M1
};

template <>
struct Fmt<kFmtMxfp8> {
    static constexpr int kStepK = 64;
    static constexpr int kCbsz = 0;               // E4M3
};

// 16-byte chunk swizzle of 64-byte LDS rows, conflict-free for the fragment
// reads: rows r and r + 2 (read together with both lane halves) differ in
// chunk bit 1, and rows r, r + 4, r + 8, r + 12 get four distinct chunks
// (zero LdsBankConflict measured with rocprofv3)
__device__ __forceinline__ int swz(int r) { return ((r & 2) ^ (r >> 2)) & 3; }

// Tile of workgroup bid: `group` row tiles sweep all column tiles together (I: an
// integer type that holds the number of tiles).
template <typename I>
__device__ __forceinline__ void tile_coords_of(I bid, I tiles_m, I tiles_n, I group, I &tm, I &tn)
{
    // Hardware dispatch sends consecutive workgroups to consecutive XCDs; give
    // every XCD a contiguous range of the tile order instead.
    const I nb = tiles_m * tiles_n;
    const I xcd = bid % kXcds, local = bid / kXcds;
    const I per = nb / kXcds, rem = nb % kXcds;
    const I t = xcd * per + (xcd < rem ? xcd : rem) + local;
    // grouped order: `group` row tiles sweep all column tiles together
    const I span = group * tiles_n;
    const I grp = t / span;
    const I first = grp * group;
    const I gsz = (tiles_m - first) < group ? (tiles_m - first) : group;
    const I in = t - grp * span;
    tm = first + in % gsz;
    tn = in / gsz;
}

// Wave-uniform 64-bit value (moves it to SGPRs).
__device__ __forceinline__ uint64_t uniform64(uint64_t v)
{
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// global -> LDS, 16 bytes per lane at M0 + 16 * lane; address = sbase + voff
// with a wave-uniform base
__device__ __forceinline__ void lds_dma16(const uint8_t *sbase, uint32_t voff, uint32_t lds_addr)
{
    const uint64_t base = uniform64(reinterpret_cast<uint64_t>(sbase));
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_addr), "v"(voff), "s"(base)
                 : "memory");
}

// the same with a per-lane 64-bit address
__device__ __forceinline__ void lds_dma16(const uint8_t *src, uint32_t lds_addr)
{
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_addr), "v"(src) : "memory");
}

// global -> LDS, 4 bytes per lane at M0 + 4 * lane, per-lane 64-bit address
__device__ __forceinline__ void lds_dma4(const uint8_t *src, uint32_t lds_addr)
{
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dword %1, off" ::"s"(lds_addr), "v"(src) : "memory");
}

template <int N>
__device__ __forceinline__ void wait_vmcnt() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// every LDS read of this wave has returned: the builtin tells the compiler's wait
// counting, the empty asm keeps reads and loads on their sides of it
__device__ __forceinline__ void wait_lgkm()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);
    asm volatile("" ::: "memory");
}

__device__ __forceinline__ void block_barrier() { asm volatile("s_barrier" ::: "memory"); }

// Row of B (within a 256-row tile) that feeds MFMA row slot t = 128 h + 32 j + l
// of the interleaved-column layout: 128 h + 64 (j / 2) + 2 l + j % 2.
__device__ __forceinline__ int interleaved_row(int t)
{
    const int j = (t >> 5) & 3, l = t & 31;
    return (t & ~127) + 64 * (j >> 1) + 2 * l + (j & 1);
}

}  // namespace
}  // namespace q2d
