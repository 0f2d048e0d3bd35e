// Block-scaled GEMMs with few output tiles: C[M][N] (+)= A . B^T as in gemm.hip
// (FP4 with 2D or 1D blocks, MXFP8), on tiles small enough to fill the chip.
//
// Both kernels stage XOR-swizzled operand rows in LDS with the global -> LDS loads
// of the large-tile kernels.
//
// gemm_tile_kernel: 128 x 128 tiles, 2 x 2 waves, a ring of three stages shared by
// the workgroup, or of two with two workgroups a CU.  What bounds it: at 256
// workgroups the loads -- an L2 channel serves one request a cycle whether it is 64
// or 128 bytes, so stages hold whole 128-byte lines (with 64-byte rows a stage of
// 128 values took 920 cycles against 722 on 2048 x 4096 x 4096), and a load
// instruction costs the CU 16-20 cycles whatever its size, so 2D scale words come
// with one load per wave and stage (a load per 64 rows: 74 of the 722 cycles).
// Alone on a CU it is bound by its own issue: the next fragments' reads and the
// loads sit between MFMAs (all loads in one group: 14.4 us for 128 x 4096 x 4096,
// spread 10.9 us).
//
// gemm_ksplit_kernel: 32 x 32 or 64 x 64 tiles; the four waves of a workgroup
// split K.  Each wave runs its own ring (64-byte rows, four stages, a scale word
// per row) over its K range, so the K loop has no barrier, and the partial tiles
// meet in LDS at the end, added in wave order (the result does not depend on
// timing).  It is bound by load latency and, from a few hundred tiles on, by the
// operand bytes each small tile loads for itself.
//
// Before these kernels a 128 x 128 register-staged kernel took 47.9 us for 16 x
// 12288 x 4096 (now 8.0), 34 us for 2000 x 2048 x 2048 (11.2), 8 us for 128 x 256
// x 256 (2.9), kernel trace against launches in a graph.
#include "gemm_quant.hpp"

namespace q2d {

namespace {

constexpr int kRing = 4;                        // stages of gemm_ksplit_kernel's rings

struct Frag {
    uint4 q0, q1;                               // chunks h and 2 + h of the row's 64 bytes
    uint32_t w;                                 // the row's scale word
};

// row r of a stage (WORD: with its scale word)
template <bool WORD>
__device__ __forceinline__ void read_frag(Frag &f, const uint8_t *rows, const uint8_t *words, int r, int half)
{
    const int sw = swz(r);
    f.q0 = *reinterpret_cast<const uint4 *>(rows + r * 64 + ((half ^ sw) * 16));
    f.q1 = *reinterpret_cast<const uint4 *>(rows + r * 64 + (((2 + half) ^ sw) * 16));
    if (WORD) f.w = *reinterpret_cast<const uint32_t *>(words + r * 4);
}

// Product ks of a stage for a 32-row A fragment and a 32-row B fragment (E2M1:
// two products of 64 values; E4M3: one).  wa, wb: the scale words shifted right
// by 8 * half, so that bytes 0 and 2 belong to this lane half.  E4M3: PAR is the
// stage's half of the 128 values of its word.
template <int FMT, int PAR, int KS>
__device__ __forceinline__ void mfma_stage(v16f &acc, const Frag &a, const Frag &b, uint32_t wa, uint32_t wb)
{
    constexpr int C = Fmt<FMT>::kCbsz;
    if constexpr (FMT == kFmtFp4Block2D) {
        const uint4 qa = KS ? a.q1 : a.q0, qb = KS ? b.q1 : b.q0;
        const v8i av = {(int)qa.x, (int)qa.y, (int)qa.z, (int)qa.w, 0, 0, 0, 0};
        const v8i bv = {(int)qb.x, (int)qb.y, (int)qb.z, (int)qb.w, 0, 0, 0, 0};
        acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, bv, acc, C, C, 2 * KS, (int)wa, 2 * KS, (int)wb);
    } else {
        const v8i av = {(int)a.q0.x, (int)a.q0.y, (int)a.q0.z, (int)a.q0.w,
                        (int)a.q1.x, (int)a.q1.y, (int)a.q1.z, (int)a.q1.w};
        const v8i bv = {(int)b.q0.x, (int)b.q0.y, (int)b.q0.z, (int)b.q0.w,
                        (int)b.q1.x, (int)b.q1.y, (int)b.q1.z, (int)b.q1.w};
        acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, bv, acc, C, C, 2 * PAR, (int)wa, 2 * PAR, (int)wb);
    }
}

// The MFMAs of one stage, with the next stage's fragment reads (read(k), k < TI +
// TJ: A fragments, then B) and the loads into the freed slot (load(k), k < LOADS)
// spread between them (a wave issues in order, and a global -> LDS load may wait
// for the ones before it: back to back they would hold up the MFMAs behind them);
// sched_barrier pins the order.
template <int FMT, int PAR, int TI, int TJ, int LOADS, typename RD, typename LD>
__device__ __forceinline__ void stage_products(v16f (&acc)[TI][TJ], const Frag (&fa)[TI], const Frag (&fb)[TJ], int half,
                                               RD &&read, LD &&load)
{
    constexpr int KS = FMT == kFmtFp4Block2D ? 2 : 1, NM = KS * TI * TJ, NR = TI + TJ, NI = NR + LOADS;
    uint32_t wa[TI], wb[TJ];
#pragma unroll
    for (int i = 0; i < TI; ++i) wa[i] = fa[i].w >> (8 * half);
#pragma unroll
    for (int j = 0; j < TJ; ++j) wb[j] = fb[j].w >> (8 * half);
    unroll<NM>([&](auto mc) __attribute__((always_inline)) {
        constexpr int m = decltype(mc)::value, ks = m / (TI * TJ), i = m / TJ % TI, j = m % TJ;
        mfma_stage<FMT, PAR, ks>(acc[i][j], fa[i], fb[j], wa[i], wb[j]);
        __builtin_amdgcn_sched_barrier(0);
        constexpr int k0 = m * NI / NM, k1 = (m + 1) * NI / NM;
        unroll<k1 - k0>([&](auto kc) __attribute__((always_inline)) {
            constexpr int k = k0 + decltype(kc)::value;
            if constexpr (k < NR) read(std::integral_constant<int, k>{});
            else load(std::integral_constant<int, k - NR>{});
        });
        __builtin_amdgcn_sched_barrier(0);
    });
}

// Scale word of operand row r for stage t at scales + word_row(r) + t * step: 2D
// blocks: grid row r / 32, step 4; 1D blocks: K-tile-major words, step ld; MXFP8:
// one word per row and two stages, step 4 for two.
template <int FMT>
__device__ __forceinline__ int64_t word_row(int64_t r, int64_t ld, bool oned)
{
    if (FMT == kFmtMxfp8) return r * ld;
    return oned ? 4 * r : (r >> 5) * ld;
}

// gemm_ksplit_kernel's wait in the body of stage s: the next stage has landed.  left: stages
// after s (as many as the ring holds are in flight).  CODES and WORDS: this wave's
// loads of codes and of scale words; MXFP8 stages bring words only where their
// number is even (PAR: s's parity).
template <int FMT, int PAR, int CODES, int WORDS>
__device__ __forceinline__ void wait_next(uint32_t left)
{
    constexpr bool F8 = FMT == kFmtMxfp8;
    static_assert(kRing == 4, "two stages may stay in flight behind the next one");
    if (left >= 3) wait_vmcnt<2 * CODES + (F8 ? 1 : 2) * WORDS>();
    else if (left == 2) wait_vmcnt<CODES + (F8 && PAR ? 0 : WORDS)>();
    else wait_vmcnt<0>();
}
// the same before the first stage: n stages in all
template <int FMT, int CODES, int WORDS>
__device__ __forceinline__ void wait_first(uint32_t n)
{
    constexpr bool F8 = FMT == kFmtMxfp8;
    if (n >= 4) wait_vmcnt<3 * CODES + (F8 ? 1 : 3) * WORDS>();
    else if (n == 3) wait_vmcnt<2 * CODES + (F8 ? 1 : 2) * WORDS>();
    else if (n == 2) wait_vmcnt<CODES + (F8 ? 0 : WORDS)>();
    else wait_vmcnt<0>();
}

typedef __bf16 bf2_t __attribute__((ext_vector_type(2)));

// bf16 output: interleaved columns (MFMA tiles 2 p and 2 p + 1 of a wave take B
// rows 64 p + 2 l and 64 p + 2 l + 1), so that a lane holds neighbouring columns
// and 32 lanes store a 128-byte run; pair stores need C and its pitch aligned.
__device__ __forceinline__ bool pair_stores(const GemmArgs &g)
{
    return ((reinterpret_cast<uintptr_t>(g.c) | (uintptr_t)(g.ldc * 2)) & 3u) == 0;
}

// One element of C
template <bool BF16OUT>
__device__ __forceinline__ void store_one(const GemmArgs &g, int64_t row, int64_t col, float v)
{
    if (BF16OUT) {
        __bf16 *p = reinterpret_cast<__bf16 *>(g.c) + row * g.ldc + col;
        *p = (__bf16)(g.accumulate ? v + (float)*p : v);
    } else {
        float *p = reinterpret_cast<float *>(g.c) + row * g.ldc + col;
        *p = g.accumulate ? v + *p : v;
    }
}

// 16-byte chunk swizzle of 128-byte LDS rows, conflict-free for the fragment
// reads: the four rows read together with both lane halves map to distinct chunk
// pairs, and eight consecutive rows to distinct chunks
__device__ __forceinline__ int swz128(int r)
{
    return ((r & 2) << 1) | (((r ^ (r >> 3)) & 1) << 1) | ((r >> 2) & 1);
}

// (64 TI) x (64 TJ) tiles, each wave (32 TI) x (32 TJ); RING stages of 128-byte
// operand rows (256 E2M1 or 128 E4M3 values), i.e. two units of 64 bytes.  A unit
// is the MFMAs on one set of fragments while the next unit's are read; the loads
// of stage s + RING go out over the second unit of stage s and the first of
// stage s + 1.  WM: how the scale words come: 0 -- both operands in 2D blocks: each
// wave loads its own block rows' words of both units at once; 1 -- one word per
// row (1D blocks, MXFP8).
template <int FMT, int TI, int TJ, int RING, int WM>
constexpr int tile_lds_bytes()
{
    const int rows = 64 * (TI + TJ);
    return RING * (128 * rows + (WM ? 4 * (FMT == kFmtMxfp8 ? 1 : 2) * rows : 4 * 256));
}

// QOUT (QSR): the product leaves in FP4 (rounded stochastically) instead.
template <int FMT, int TI, int TJ, int RING, int WM, bool BF16OUT, bool QOUT = false, bool QSR = false>
__device__ __forceinline__ void gemm_tile(const GemmArgs &g, uint8_t *smem, uint32_t tm, uint32_t tn)
{
    constexpr bool F8 = FMT == kFmtMxfp8;
    constexpr int TM = 64 * TI, TN = 64 * TJ, kRows = TM + TN;
    constexpr int kWords = 128 * kRows;                         // byte offset of the scale words in a stage
    constexpr int WU = F8 ? 1 : 2;                              // scale words per row and stage
    constexpr int kStage = kWords + (WM ? 4 * WU * kRows : 4 * 256);
    constexpr int CODES = kRows / 32, WORDS = WM ? WU : 1;      // this wave's loads per stage
    constexpr int LOADS = CODES + WORDS, H1 = (LOADS + 1) / 2;  // the first H1 in the second unit
    static_assert(WM || !F8, "MXFP8 has one word per row");
    static_assert(kRows == 256, "each wave loads the words of 64 rows");
    static_assert(RING * kStage == tile_lds_bytes<FMT, TI, TJ, RING, WM>(), "the caller's LDS");

    const int64_t m0 = (int64_t)tm * TM, n0 = (int64_t)tn * TN;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1, half = lane >> 5;
    const uint32_t nu = (uint32_t)(g.K / Fmt<FMT>::kStepK);     // units (MXFP8: an even number)
    const uint32_t ns = (nu + 1) / 2;                           // stages

    // operand row of the stage's row t: A rows, then B rows (clamped into the operand)
    auto row_of = [&](int t) __attribute__((always_inline)) -> int64_t {
        const int tb = t - TM;
        const int64_t r = t < TM ? m0 + t : n0 + (BF16OUT ? interleaved_row(tb) : tb);
        const int64_t lim = t < TM ? g.M : g.N;
        return r < lim ? r : lim - 1;
    };
    const uint8_t *pc[CODES], *pw;
#pragma unroll
    for (int k = 0; k < CODES; ++k) {
        const int t = 32 * k + 8 * wave + (lane >> 3), c16 = ((lane & 7) ^ swz128(t)) * 16;
        pc[k] = (32 * k < TM ? g.a + row_of(t) * g.lda : g.b + row_of(t) * g.ldb) + c16;
    }
    // the last stage of an odd number of units: its second half does not exist (rows
    // t and t + 32 k have the same swizzle, so this holds for every load)
    const int back = ((lane & 7) ^ swz128(8 * wave + (lane >> 3))) >= 4 ? 64 : 0;
    int64_t wstep = 4;                                          // bytes per unit (MXFP8: per stage)
    if constexpr (WM == 0) {
        // lane: unit lane / 32, block row lane % 32 of the wave's TI + TJ (clamped)
        const int x = (lane & 31) < TI + TJ ? (lane & 31) : TI + TJ - 1;
        const bool is_a = x < TI;
        int64_t r = is_a ? m0 + wm * 32 * TI + 32 * x : n0 + wn * 32 * TJ + 32 * (x - TI);
        const int64_t lim = is_a ? g.M : g.N;
        r = r < lim ? r : lim - 1;
        pw = (is_a ? g.sa : g.sb) + (r >> 5) * (is_a ? g.ldsa : g.ldsb) + 4 * half;
    } else {
        // rows 64 wave + lane, of one operand
        const bool is_a = wave < TI;
        const bool oned = is_a ? g.a1d : g.b1d;
        const int64_t ld = is_a ? g.ldsa : g.ldsb;
        if (!F8 && oned) wstep = ld;
        pw = (is_a ? g.sa : g.sb) + word_row<FMT>(row_of(64 * wave + lane), ld, oned);
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)&smem[0];
    // load k of stage s: codes, then scale words (past the last stage: that one
    // again, into a slot that is not read any more)
    auto load = [&](uint32_t s, uint32_t slot, int k) __attribute__((always_inline)) {
        const uint32_t stage = lds0 + slot * kStage;
        const uint32_t t = s < ns ? s : ns - 1;
        const bool cut = !F8 && 2 * t + 1 >= nu;                // only the first unit exists
        if (k < CODES) {
            const uint8_t *p = pc[k < CODES ? k : 0] + (uint64_t)t * 128;
            lds_dma16(cut ? p - back : p, stage + (4 * k + wave) * 1024);
        } else if (WM == 0) {
            const uint8_t *p = pw + (uint64_t)t * 8;
            lds_dma4(cut && half ? p - 4 : p, stage + kWords + wave * 256);
        } else {
            const int u = k - CODES;
            const uint32_t ut = F8 ? t : (cut ? 2 * t : 2 * t + u);
            lds_dma4(pw + ut * wstep, stage + kWords + u * (4 * kRows) + wave * 256);
        }
    };

    v16f acc[TI][TJ];
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

    Frag fa0[TI], fb0[TJ], fa1[TI], fb1[TJ];
    const int sw = swz128(lane & 31);
    // fragment k of unit u of the stage in `slot` (MXFP8: the scale words come with unit 0)
    auto read = [&](auto uc, uint32_t slot, int k, Frag (&fa)[TI], Frag (&fb)[TJ]) __attribute__((always_inline)) {
        constexpr int u = decltype(uc)::value;
        const uint8_t *st = smem + slot * kStage;
        const int r = (k < TI ? (wm * TI + k) * 32 : TM + (wn * TJ + k - TI) * 32) + (lane & 31);
        Frag &f = k < TI ? fa[k < TI ? k : 0] : fb[k < TI ? 0 : k - TI];
        f.q0 = *reinterpret_cast<const uint4 *>(st + r * 128 + (((4 * u + half) ^ sw) * 16));
        f.q1 = *reinterpret_cast<const uint4 *>(st + r * 128 + (((4 * u + 2 + half) ^ sw) * 16));
        if constexpr (WM == 0) {
            // bf16: the interleaved B rows of lanes 0..15 and 16..31 lie in different blocks
            const int x = k < TI ? k : TI + (BF16OUT ? 2 * ((k - TI) >> 1) + ((lane & 31) >> 4) : k - TI);
            f.w = *reinterpret_cast<const uint32_t *>(st + kWords + wave * 256 + u * 128 + 4 * x);
        } else if constexpr (!F8 || u == 0) {
            f.w = *reinterpret_cast<const uint32_t *>(st + kWords + (F8 ? 0 : u) * (4 * kRows) + 4 * r);
        }
    };

    // stages 0 .. RING - 2 and the first part of stage RING - 1
#pragma unroll
    for (uint32_t t = 0; t < RING; ++t)
#pragma unroll
        for (int k = 0; k < (t + 1 < RING ? LOADS : H1); ++k) load(t, t, k);
    wait_vmcnt<(RING - 2) * LOADS + H1>();
    block_barrier();
#pragma unroll
    for (int k = 0; k < TI + TJ; ++k) read(std::integral_constant<int, 0>{}, 0, k, fa0, fb0);
    // the second unit's fragments of the stage in `slot` (MXFP8: the first's words)
    auto read1 = [&](uint32_t slot, int k) __attribute__((always_inline)) {
        read(std::integral_constant<int, 1>{}, slot, k, fa1, fb1);
        if constexpr (F8) {
            if (k < TI) fa1[k < TI ? k : 0].w = fa0[k < TI ? k : 0].w;
            else fb1[k < TI ? 0 : k - TI].w = fb0[k < TI ? 0 : k - TI].w;
        }
    };

    uint32_t slot = 0, prev = RING - 1;                         // s % RING, (s - 1) % RING
    for (uint32_t s = 0; s + 1 < ns; ++s) {
        const uint32_t next = slot + 1 == RING ? 0 : slot + 1;
        // ---- unit 0; the second part of the loads of stage s - 1 + RING
        wait_lgkm();
        stage_products<FMT, 0, TI, TJ, LOADS - H1>(
            acc, fa0, fb0, half, [&](auto k) __attribute__((always_inline)) { read1(slot, k); },
            [&](auto k) __attribute__((always_inline)) { load(s - 1 + RING, prev, H1 + k); });
        wait_lgkm();                                    // this wave has read stage s
        wait_vmcnt<(RING - 2) * LOADS>();               // its loads of stage s + 1 have landed
        block_barrier();
        // ---- unit 1; the first part of the loads of stage s + RING
        stage_products<FMT, 1, TI, TJ, H1>(
            acc, fa1, fb1, half,
            [&](auto k) __attribute__((always_inline)) { read(std::integral_constant<int, 0>{}, next, k, fa0, fb0); },
            [&](auto k) __attribute__((always_inline)) { load(s + RING, slot, k); });
        prev = slot;
        slot = next;
    }
    // ---- the last stage: one or two units
    wait_lgkm();
    stage_products<FMT, 0, TI, TJ, 0>(acc, fa0, fb0, half, [&](auto k) __attribute__((always_inline)) { read1(slot, k); },
                                      [](auto) {});
    if (F8 || (nu & 1) == 0) {
        wait_lgkm();
        stage_products<FMT, 1, TI, TJ, 0>(acc, fa1, fb1, half, [](auto) {}, [](auto) {});
    }
    wait_vmcnt<0>();                                    // nothing lands in LDS from here on

    // a lane holds column lane % 32 (bf16: a pair) and rows 8 q + 4 half + 0..3 of
    // every MFMA tile
    const int64_t r0 = m0 + wm * 32 * TI, c0 = n0 + wn * 32 * TJ;
    if constexpr (QOUT) {
        static_assert(4 * (q_strip(TJ) + kPTab) <= RING * kStage, "strips and draw tables fit the ring");
        __syncthreads();                                // every wave has read its last stage
        uint8_t *strip = smem + wave * (q_strip(TJ) + kPTab), *ptab = strip + q_strip(TJ);
        if (m0 + TM <= g.M && n0 + TN <= g.N)
            store_qblock<false, QSR, TI, TJ, false>(acc, g, strip, ptab, (int)r0, (int)c0, 32 * TI, 32 * TJ);
        else
            store_qblock<true, QSR, TI, TJ, false>(acc, g, strip, ptab, (int)r0, (int)c0, (int)(g.M - r0), (int)(g.N - c0));
        return;
    }
    if (m0 + TM <= g.M && n0 + TN <= g.N && !g.accumulate && (!BF16OUT || pair_stores(g))) {
        uint8_t *p = reinterpret_cast<uint8_t *>(g.c) + ((r0 + 4 * half) * g.ldc + c0) * (BF16OUT ? 2 : 4) + 4 * (lane & 31);
        const int64_t pitch = g.ldc * (BF16OUT ? 2 : 4);
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
#pragma unroll
                for (int j = 0; j < TJ; j += BF16OUT ? 2 : 1) {
                    if constexpr (BF16OUT)
                        *reinterpret_cast<bf2_t *>(p + j * 64) = bf2_t{(__bf16)acc[i][j][r], (__bf16)acc[i][j + 1][r]};
                    else
                        *reinterpret_cast<float *>(p + j * 128) = acc[i][j][r];
                }
                p += (r & 3) == 3 ? 5 * pitch : pitch;
            }
        return;
    }
    // edge tiles, accumulation, unaligned pairs: 32-row strips through LDS, one
    // element per lane and store, in a rolled loop
    constexpr int kPitch = 32 * TJ + 8;                         // floats; a wave's strip is 32 x (32 TJ)
    static_assert(4 * 32 * kPitch * 4 <= RING * kStage, "the strips fit the ring");
    __syncthreads();                                            // every wave has read its last stage
    float *strip = reinterpret_cast<float *>(smem) + wave * 32 * kPitch;
#pragma unroll
    for (int i = 0; i < TI; ++i) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
#pragma unroll
            for (int j = 0; j < TJ; ++j) {
                const int col = BF16OUT ? 64 * (j >> 1) + 2 * (lane & 31) + (j & 1) : 32 * j + (lane & 31);
                strip[(8 * (r >> 2) + 4 * half + (r & 3)) * kPitch + col] = acc[i][j][r];
            }
        __builtin_amdgcn_wave_barrier();
        // 64 columns of a row per step, TJ / 2 steps a row
        const int64_t left = g.M - (r0 + 32 * i);
        const int rows = left < 32 ? (left < 0 ? 0 : (int)left) : 32;
        for (int cc = lane; cc < 32 * TJ; cc += 64) {
            if (c0 + cc >= g.N) continue;
#pragma unroll 8
            for (int rr = 0; rr < rows; ++rr) store_one<BF16OUT>(g, r0 + 32 * i + rr, c0 + cc, strip[rr * kPitch + cc]);
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// (32 TI) x (32 TJ) tiles, TI = TJ, K split over the four waves in whole units of 128.
template <int TI, int TJ>
constexpr int ksplit_lds_bytes()
{
    const int rows = 32 * (TI + TJ), waves = kThreads / 64;
    const int ring = waves * kRing * (rows * 64 + (rows + 63) / 64 * 256), red = waves * TI * TJ * 4 * 64 * 16;
    return ring > red ? ring : red;
}

template <int FMT, int TI, int TJ, bool BF16OUT>
__device__ __forceinline__ void gemm_ksplit(const GemmArgs &g, uint8_t *smem, uint32_t block, uint32_t tiles_m,
                                            uint32_t tiles_n)
{
    constexpr int kWaves = kThreads / 64;
    constexpr int kRows = 32 * (TI + TJ);
    constexpr int CODES = kRows / 16, WORDS = (kRows + 63) / 64;        // loads per wave and stage
    constexpr int kStage = kRows * 64 + WORDS * 256;            // per wave
    constexpr bool PAIR = BF16OUT && TJ == 2;                   // interleaved output columns
    static_assert(kWaves * kRing * kStage <= ksplit_lds_bytes<TI, TJ>() &&
                  kWaves * TI * TJ * 4 * 64 * 16 <= ksplit_lds_bytes<TI, TJ>(), "rings, then partial tiles");

    uint32_t tm, tn;
    tile_coords_of(block, tiles_m, tiles_n, 8u, tm, tn);
    const int64_t m0 = (int64_t)tm * 32 * TI, n0 = (int64_t)tn * 32 * TJ;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int half = lane >> 5;

    // this wave's stages [s0, s0 + n): units of 128 values over the active waves
    // (an MXFP8 unit is two stages, so every wave starts on an even one)
    const uint32_t units = (uint32_t)(g.K / 128), per_unit = 128 / Fmt<FMT>::kStepK;
    const uint32_t active = units < (uint32_t)kWaves ? units : (uint32_t)kWaves;
    const uint32_t u0 = (uint32_t)((uint64_t)units * wave / active), u1 = (uint32_t)((uint64_t)units * (wave + 1) / active);
    const uint32_t s0 = u0 * per_unit, n = (uint32_t)wave < active ? (u1 - u0) * per_unit : 0;

    // row t of the stage: A rows, then B rows
    auto row_of = [&](int t, bool &is_a) __attribute__((always_inline)) -> int64_t {
        is_a = t < 32 * TI;
        const int tb = t - 32 * TI;
        const int64_t r = is_a ? m0 + t : n0 + (PAIR ? interleaved_row(tb) : tb);
        const int64_t lim = is_a ? g.M : g.N;
        return r < lim ? r : lim - 1;
    };
    const uint8_t *pc[CODES], *pw[WORDS];
    int64_t wstep[WORDS];                                       // bytes per stage (MXFP8: per two stages)
#pragma unroll
    for (int c = 0; c < CODES; ++c) {
        const int t = 16 * c + (lane >> 2), c16 = ((lane & 3) ^ swz(t)) * 16;
        bool is_a;
        const int64_t r = row_of(t, is_a);
        pc[c] = (is_a ? g.a + r * g.lda : g.b + r * g.ldb) + c16 + (uint64_t)s0 * 64;
    }
#pragma unroll
    for (int c = 0; c < WORDS; ++c) {
        int t = 64 * c + lane; t = t < kRows ? t : kRows - 1;
        bool is_a;
        const int64_t r = row_of(t, is_a);
        const bool oned = is_a ? g.a1d : g.b1d;
        const int64_t ld = is_a ? g.ldsa : g.ldsb;
        wstep[c] = FMT != kFmtMxfp8 && oned ? ld : 4;
        pw[c] = (is_a ? g.sa : g.sb) + word_row<FMT>(r, ld, oned) + (FMT == kFmtMxfp8 ? s0 >> 1 : s0) * wstep[c];
    }
    uint8_t *ring = smem + wave * (kRing * kStage);
    const uint32_t lds0 = (uint32_t)(uintptr_t)ring;
    auto load = [&](uint32_t s, bool words) __attribute__((always_inline)) {
        const uint32_t stage = lds0 + (s % kRing) * kStage;
#pragma unroll
        for (int k = 0; k < CODES; ++k) lds_dma16(pc[k] + (uint64_t)s * 64, stage + k * 1024);
        if (words) {
#pragma unroll
            for (int k = 0; k < WORDS; ++k)
                lds_dma4(pw[k] + (FMT == kFmtMxfp8 ? s >> 1 : s) * wstep[k], stage + kRows * 64 + k * 256);
        }
    };

    v16f acc[TI][TJ];
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

    Frag fa0[TI], fb0[TJ], fa1[TI], fb1[TJ];
    auto read = [&](auto word, uint32_t s, int k, Frag (&fa)[TI], Frag (&fb)[TJ]) __attribute__((always_inline)) {
        const uint8_t *st = ring + (s % kRing) * kStage;
        read_frag<decltype(word)::value>(k < TI ? fa[k] : fb[k - TI], st, st + kRows * 64, 32 * k + (lane & 31), half);
    };
    auto body = [&](auto par, uint32_t s, Frag (&fa)[TI], Frag (&fb)[TJ], Frag (&na)[TI], Frag (&nb)[TJ])
                    __attribute__((always_inline)) {
        constexpr int PAR = decltype(par)::value;
        constexpr bool F8 = FMT == kFmtMxfp8;
        wait_lgkm();                                    // stage s is in registers, its slot free
        wait_next<FMT, PAR, CODES, WORDS>(n - 1 - s);
        stage_products<FMT, PAR, TI, TJ, 1>(
            acc, fa, fb, half,
            [&](auto k) __attribute__((always_inline)) {
                // past the last stage the slot's bytes are read and never used
                if constexpr (F8 && PAR == 0) {         // an odd stage's words are the even one's
                    read(std::false_type{}, s + 1, k, na, nb);
                    if (k < TI) na[k < TI ? k : 0].w = fa[k < TI ? k : 0].w;
                    else nb[k < TI ? 0 : k - TI].w = fb[k < TI ? 0 : k - TI].w;
                } else {
                    read(std::true_type{}, s + 1, k, na, nb);
                }
            },
            [&](auto) __attribute__((always_inline)) { if (s + kRing < n) load(s + kRing, !F8 || PAR == 0); });
    };

    if (n > 0) {
        for (uint32_t s = 0; s < kRing && s < n; ++s) load(s, FMT != kFmtMxfp8 || (s & 1) == 0);
        wait_first<FMT, CODES, WORDS>(n);
#pragma unroll
        for (int k = 0; k < TI + TJ; ++k) read(std::true_type{}, 0, k, fa0, fb0);
        uint32_t s = 0;
        for (; s + 1 < n; s += 2) {
            body(std::integral_constant<int, 0>{}, s, fa0, fb0, fa1, fb1);
            body(std::integral_constant<int, 1>{}, s + 1, fa1, fb1, fa0, fb0);
        }
        if (FMT == kFmtFp4Block2D && s < n) body(std::integral_constant<int, 0>{}, s, fa0, fb0, fa1, fb1);
    }

    // partial tiles to LDS (the rings are drained): four accumulators of a lane
    // as one 16-byte piece, pieces of a quad (i, q, j) lane by lane
    __syncthreads();
    uint4 *red = reinterpret_cast<uint4 *>(smem);
    if (n > 0) {
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int j = 0; j < TJ; ++j)
                    red[((wave * TI * 4 + i * 4 + q) * TJ + j) * 64 + lane] =
                        make_uint4(f_bits(acc[i][j][4 * q]), f_bits(acc[i][j][4 * q + 1]), f_bits(acc[i][j][4 * q + 2]),
                                   f_bits(acc[i][j][4 * q + 3]));
    }
    __syncthreads();
    // wave q sums and writes row quads q of every 32-row strip: a lane has four
    // consecutive rows of a column (PAIR: of two neighbouring ones)
    const bool pairs = PAIR && n0 + 64 <= g.N && !g.accumulate && pair_stores(g);
    const int q = wave;
#pragma unroll
    for (int i = 0; i < TI; ++i) {
        float v[TJ][4];
#pragma unroll
        for (int j = 0; j < TJ; ++j) {
#pragma unroll
            for (int r = 0; r < 4; ++r) v[j][r] = 0.0f;
            for (uint32_t w = 0; w < active; ++w) {
                const uint4 p = red[((w * TI * 4 + i * 4 + q) * TJ + j) * 64 + lane];
                v[j][0] += bits_f(p.x); v[j][1] += bits_f(p.y); v[j][2] += bits_f(p.z); v[j][3] += bits_f(p.w);
            }
        }
        const int64_t row = m0 + i * 32 + 8 * q + 4 * half;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (row + r >= g.M) continue;
            if (PAIR && pairs) {
                *reinterpret_cast<bf2_t *>(reinterpret_cast<__bf16 *>(g.c) + (row + r) * g.ldc + n0 + 2 * (lane & 31)) =
                    bf2_t{(__bf16)v[0][r], (__bf16)v[TJ - 1][r]};
            } else {
#pragma unroll
                for (int j = 0; j < TJ; ++j) {
                    const int64_t col = n0 + (PAIR ? 2 * (lane & 31) + j : 32 * j + (lane & 31));
                    if (col < g.N) store_one<BF16OUT>(g, row + r, col, v[j][r]);
                }
            }
        }
    }
}

// The tiles of one product, or of two in one grid (workgroups from `first` on belong
// to the second).  BF0, BF1: bf16 outputs.
struct Pair {
    GemmArgs g[2];
    uint32_t first;
    uint32_t tiles_m[2], tiles_n[2];
};

template <int FMT, int TI, int TJ, int RING, int WM, bool BF0, bool BF1>
__global__ __launch_bounds__(kThreads, RING == 2 ? 2 : 1) void gemm_tile_kernel(const Pair p)
{
    __shared__ __attribute__((aligned(1024))) uint8_t smem[tile_lds_bytes<FMT, TI, TJ, RING, WM>()];
    const bool second = blockIdx.x >= p.first;
    const int i = second ? 1 : 0;
    uint32_t tm, tn;
    tile_coords_of(blockIdx.x - (second ? p.first : 0u), p.tiles_m[i], p.tiles_n[i], 8u, tm, tn);
    if (BF0 == BF1 || !second) gemm_tile<FMT, TI, TJ, RING, WM, BF0>(p.g[BF0 == BF1 ? i : 0], smem, tm, tn);
    else gemm_tile<FMT, TI, TJ, RING, WM, BF1>(p.g[1], smem, tm, tn);
}

// Ragged-M grouped (MoE) product on 128 x 128 tiles, two workgroups a CU, each
// walking row tiles of all experts x column tiles.
template <bool BF16OUT>
__global__ __launch_bounds__(kThreads, 2) void gemm_tile_grouped_kernel(const GemmArgs g, const GroupedArgs gr,
                                                                       uint32_t tiles_n)
{
    __shared__ __attribute__((aligned(1024))) uint8_t smem[tile_lds_bytes<kFmtFp4Block2D, 2, 2, 2, 0>()];
    __shared__ int32_t seg_start[kMaxSegs + 1], pad_start[kMaxSegs + 1], tile_start[kMaxSegs + 1];
    if ((threadIdx.x >> 6) == 0) {
        wave_offsets(gr.nseg, gr.seg_offsets, gr.total_rows, seg_start);
        __builtin_amdgcn_wave_barrier();
        const int32_t *off = seg_start;
        wave_prefix(gr.nseg, [&](int i) { return (off[i + 1] - off[i] + 127) / 128 * 128; }, pad_start);
        wave_prefix(gr.nseg, [&](int i) { return (off[i + 1] - off[i] + 127) / 128; }, tile_start);
    }
    __syncthreads();
    const uint32_t total = (uint32_t)__builtin_amdgcn_readfirstlane(tile_start[gr.nseg]) * tiles_n;
    for (uint32_t u = blockIdx.x; u < total; u += gridDim.x) {
        // as in the persistent kernel: a multiple of 8 column tiles already gives each
        // XCD one column band; otherwise a contiguous range of the order
        uint32_t tt = u;
        if (tiles_n % kXcds != 0) {
            const uint32_t xcd = u % kXcds, local = u / kXcds, per = total / kXcds, rem = total % kXcds;
            tt = xcd * per + (xcd < rem ? xcd : rem) + local;
        }
        const uint32_t rt = tt / tiles_n, tn = tt - rt * tiles_n;
        const int e = __builtin_amdgcn_readfirstlane(seg_search(tile_start, gr.nseg, (int32_t)rt));
        const uint32_t tm = rt - (uint32_t)__builtin_amdgcn_readfirstlane(tile_start[e]);
        const int64_t p_e = __builtin_amdgcn_readfirstlane(pad_start[e]);
        const int64_t o0 = __builtin_amdgcn_readfirstlane(seg_start[e]);
        GemmArgs t = g;
        t.M = __builtin_amdgcn_readfirstlane(seg_start[e + 1]) - o0;
        t.a += p_e * g.lda;
        t.sa += (p_e / 32) * g.ldsa;
        t.c = reinterpret_cast<uint8_t *>(t.c) + o0 * g.ldc * (BF16OUT ? 2 : 4);
        if (gr.b_group_rows) {
            t.b += (int64_t)e * gr.b_group_rows * g.ldb;
            t.sb += ((int64_t)e * gr.b_group_rows / 32) * g.ldsb;
        } else {
            t.b += (int64_t)e * gr.b_group_k / 2;
            t.sb += (int64_t)e * gr.b_group_k / 32;
        }
        gemm_tile<kFmtFp4Block2D, 2, 2, 2, 0, BF16OUT>(t, smem, tm, tn);
        __syncthreads();                                // the tile's LDS is the next one's
    }
}

template <int RING, int WM, bool QSR>
__global__ __launch_bounds__(kThreads, RING == 2 ? 2 : 1) void gemm_tile_quant_kernel(const GemmArgs g, uint32_t tiles_m,
                                                                                     uint32_t tiles_n)
{
    __shared__ __attribute__((aligned(1024))) uint8_t smem[tile_lds_bytes<kFmtFp4Block2D, 2, 2, RING, WM>()];
    uint32_t tm, tn;
    tile_coords_of(blockIdx.x, tiles_m, tiles_n, 8u, tm, tn);
    gemm_tile<kFmtFp4Block2D, 2, 2, RING, WM, false, true, QSR>(g, smem, tm, tn);
}

template <int FMT, int TI, int TJ, bool BF0, bool BF1>
__global__ __launch_bounds__(kThreads, 1) void gemm_ksplit_kernel(const Pair p)
{
    __shared__ __attribute__((aligned(1024))) uint8_t smem[ksplit_lds_bytes<TI, TJ>()];
    const bool second = blockIdx.x >= p.first;
    if constexpr (BF0 == BF1) {
        const int i = second ? 1 : 0;
        gemm_ksplit<FMT, TI, TJ, BF0>(p.g[i], smem, blockIdx.x - (second ? p.first : 0u), p.tiles_m[i], p.tiles_n[i]);
    } else {
        if (!second) gemm_ksplit<FMT, TI, TJ, BF0>(p.g[0], smem, blockIdx.x, p.tiles_m[0], p.tiles_n[0]);
        else gemm_ksplit<FMT, TI, TJ, BF1>(p.g[1], smem, blockIdx.x - p.first, p.tiles_m[1], p.tiles_n[1]);
    }
}

constexpr struct { int32_t tm, tn, per_cu; } kTiles[] = {{32, 32, 2}, {64, 64, 1}, {128, 128, 1}, {128, 128, 2}, {256, 256, 1}};

int64_t tiles_of(const GemmArgs &g, int tile)
{
    return ((g.M + kTiles[tile].tm - 1) / kTiles[tile].tm) * ((g.N + kTiles[tile].tn - 1) / kTiles[tile].tn);
}

template <int FMT, bool BF0, bool BF1>
hipError_t launch_t(const GemmArgs &a, const GemmArgs *b, int tile, hipStream_t s)
{
    Pair p;
    p.g[0] = a;
    p.g[1] = b ? *b : a;
    p.first = (uint32_t)tiles_of(a, tile);
    for (int i = 0; i < 2; ++i) {
        p.tiles_m[i] = (uint32_t)((p.g[i].M + kTiles[tile].tm - 1) / kTiles[tile].tm);
        p.tiles_n[i] = (uint32_t)((p.g[i].N + kTiles[tile].tn - 1) / kTiles[tile].tn);
    }
    const dim3 grid((unsigned)(tiles_of(a, tile) + (b ? tiles_of(*b, tile) : 0))), block(kThreads);
    const bool rowwise = FMT == kFmtMxfp8 || a.a1d || a.b1d || (b && (b->a1d || b->b1d));
    switch (tile) {
    case kTile32: hipLaunchKernelGGL((gemm_ksplit_kernel<FMT, 1, 1, BF0, BF1>), grid, block, 0, s, p); break;
    case kTile64: hipLaunchKernelGGL((gemm_ksplit_kernel<FMT, 2, 2, BF0, BF1>), grid, block, 0, s, p); break;
    case kTile128:
        if (rowwise) hipLaunchKernelGGL((gemm_tile_kernel<FMT, 2, 2, 3, 1, BF0, BF1>), grid, block, 0, s, p);
        else if constexpr (FMT != kFmtMxfp8) hipLaunchKernelGGL((gemm_tile_kernel<FMT, 2, 2, 3, 0, BF0, BF1>), grid, block, 0, s, p);
        break;
    default:
        if (rowwise) hipLaunchKernelGGL((gemm_tile_kernel<FMT, 2, 2, 2, 1, BF0, BF1>), grid, block, 0, s, p);
        else if constexpr (FMT != kFmtMxfp8) hipLaunchKernelGGL((gemm_tile_kernel<FMT, 2, 2, 2, 0, BF0, BF1>), grid, block, 0, s, p);
    }
    return hipGetLastError();
}

// Modelled microseconds of `tiles` tiles with `units` 128-value units of K each (see
// pick_tile), without the launch itself.  epi: what the epilogue writes (0 values, 1
// FP4 rounded to nearest, 2 FP4 rounded stochastically).
float cost_of(int tile, int64_t tiles, float units, int fmt, int epi)
{
    static const struct { float once, round[3], unit[2]; } cost[] = {{0.0f, {1.0f, 0.0f, 0.0f}, {0.14f, 0.22f}},    // unit: FP4, MXFP8
                                                                     {0.0f, {2.0f, 0.0f, 0.0f}, {0.21f, 0.375f}},
                                                                     {0.0f, {3.0f, 4.5f, 6.5f}, {0.29f, 0.55f}},
                                                                     {0.0f, {2.6f, 4.0f, 6.7f}, {0.57f, 1.10f}},
                                                                     {4.0f, {5.0f, 11.5f, 18.5f}, {0.82f, 1.55f}}};
    const int64_t slots = (int64_t)cu_count() * kTiles[tile].per_cu;
    return cost[tile].once +
           (float)((tiles + slots - 1) / slots) * (cost[tile].round[epi] + units * cost[tile].unit[fmt == kFmtMxfp8]);
}

}  // namespace

// The tile with the smallest modelled time: rounds of workgroups over the chip
// (kTiles: how many a CU holds), each a fixed part (address setup, first loads,
// epilogue) plus a part per 128 values of K; the 256 x 256 kernels pay some of the
// fixed part once.  Microseconds fitted to timings on one MI355X with a launch's
// own 2.5 us taken off (FP4, bf16 output).  Measured with 32 / 64 / 128 / 128 two a
// CU / 256: 600 x 700 x 128 3.1 / 4.5 / 5.7 / - / 12.2 us; 128 x 4096 x 4096 7.8 /
// 9.2 / 11.0 / - / 30.4; 512 x 4096 x 4096 21.0 / 18.6 / 11.9 / 16.0 / 26.6; 2048 x
// 4096 x 4096 72 / 65 / 26.7 / 23.7 / 28.9; 16384 x 2048 x 768 - / - / 35.7 / 26.4 /
// 26.1; 4096 x 4096 x 4096 139 / 125 / 49 / 44 / 38.  (256 x 128 tiles, one a CU: 45 us
// for the last, 42.3 against 37.8 for 16384 x 1536 x 2048.)
// FP4 outputs (128 / 128 two a CU / 256, nearest): 500 x 1024 x 1024 10.1 / 9.7 / 20.9;
// 4096 x 4096 x 512 23.2 / 15.3 / 19.3; 4096 x 4096 x 4096 54 / 47 / 45; stochastic: 12.0 /
// 11.7 / 28.3; 30.4 / 20.6 / 26.3; 62 / 52 / 52 -- the epilogue's arithmetic leaves the
// matrix cores idle where a CU holds one workgroup.
// `large`: the 256 x 256 kernels can take the problem.
SmallTile pick_tile(const GemmArgs &g, int fmt, bool large, float *time)
{
    const int epi = g.qc ? (g.qsr ? 2 : 1) : 0, last = epi ? kTile128 : kTile32;
    const int top = large ? kTile256 : kTile128x2;
    int best = top;
    float least = 0.0f;
    for (int k = top; k >= last; --k) {
        const float t = cost_of(k, tiles_of(g, k), (float)(g.K / 128), fmt, epi);
        if (k == top || t < least) { best = k; least = t; }
    }
    if (time) *time = least;
    return (SmallTile)best;
}

hipError_t launch_gemm_small(const GemmArgs &g, int fmt, int c_is_bf16, SmallTile tile, hipStream_t stream)
{
    if (fmt == kFmtFp4Block2D)
        return c_is_bf16 ? launch_t<kFmtFp4Block2D, true, true>(g, nullptr, tile, stream)
                         : launch_t<kFmtFp4Block2D, false, false>(g, nullptr, tile, stream);
    return c_is_bf16 ? launch_t<kFmtMxfp8, true, true>(g, nullptr, tile, stream)
                     : launch_t<kFmtMxfp8, false, false>(g, nullptr, tile, stream);
}

hipError_t launch_quantized_small(const GemmArgs &g, SmallTile tile, hipStream_t stream)
{
    const uint32_t tm = (uint32_t)((g.M + 127) / 128), tn = (uint32_t)((g.N + 127) / 128);
    const dim3 grid(tm * tn), block(kThreads);
    const bool rowwise = g.a1d || g.b1d, two = tile == kTile128x2;
    switch ((two ? 4 : 0) | (rowwise ? 2 : 0) | (g.qsr ? 1 : 0)) {
    case 0: hipLaunchKernelGGL((gemm_tile_quant_kernel<3, 0, false>), grid, block, 0, stream, g, tm, tn); break;
    case 1: hipLaunchKernelGGL((gemm_tile_quant_kernel<3, 0, true>), grid, block, 0, stream, g, tm, tn); break;
    case 2: hipLaunchKernelGGL((gemm_tile_quant_kernel<3, 1, false>), grid, block, 0, stream, g, tm, tn); break;
    case 3: hipLaunchKernelGGL((gemm_tile_quant_kernel<3, 1, true>), grid, block, 0, stream, g, tm, tn); break;
    case 4: hipLaunchKernelGGL((gemm_tile_quant_kernel<2, 0, false>), grid, block, 0, stream, g, tm, tn); break;
    case 5: hipLaunchKernelGGL((gemm_tile_quant_kernel<2, 0, true>), grid, block, 0, stream, g, tm, tn); break;
    case 6: hipLaunchKernelGGL((gemm_tile_quant_kernel<2, 1, false>), grid, block, 0, stream, g, tm, tn); break;
    default: hipLaunchKernelGGL((gemm_tile_quant_kernel<2, 1, true>), grid, block, 0, stream, g, tm, tn);
    }
    return hipGetLastError();
}

hipError_t launch_grouped_small(const GemmArgs &g, const GroupedArgs &gr, int c_is_bf16, hipStream_t stream)
{
    const uint32_t tn = (uint32_t)((g.N + 127) / 128);
    const int64_t tiles = ((gr.total_rows + 127) / 128 + gr.nseg) * (int64_t)tn;       // at most
    int64_t grid = 2 * (int64_t)cu_count();
    grid = grid < tiles ? grid : tiles;
    grid = (grid + kXcds - 1) / kXcds * kXcds;
    if (c_is_bf16)
        hipLaunchKernelGGL((gemm_tile_grouped_kernel<true>), dim3((unsigned)grid), dim3(kThreads), 0, stream, g, gr, tn);
    else
        hipLaunchKernelGGL((gemm_tile_grouped_kernel<false>), dim3((unsigned)grid), dim3(kThreads), 0, stream, g, gr, tn);
    return hipGetLastError();
}

// Two FP4 products in one grid of small tiles, where the model finds that no slower
// than a launch each: the launch (2.5 us of the device, 3 of the host) is saved and
// the second product fills the CUs that the first one's last round leaves.  One
// round lasts as long as its longest K; over several rounds K averages out.
// hipErrorNotSupported: not taken.
hipError_t launch_gemm_pair(const GemmArgs &g, int c_is_bf16, bool large, hipStream_t stream)
{
    const GemmArgs &h = *g.also;
    if (g.also_bf16 && !c_is_bf16) return hipErrorNotSupported;        // (no kernel for that order)
    float t0 = 0.0f, t1 = 0.0f;
    pick_tile(g, kFmtFp4Block2D, large, &t0);
    pick_tile(h, kFmtFp4Block2D, large, &t1);
    int best = -1;
    float least = t0 + t1 + 2.5f;
    for (int k = kTile128x2; k >= 0; --k) {
        const int64_t n0 = tiles_of(g, k), n1 = tiles_of(h, k), slots = (int64_t)cu_count() * kTiles[k].per_cu;
        const float u0 = (float)(g.K / 128), u1 = (float)(h.K / 128);
        const float units = n0 + n1 <= slots ? (u0 > u1 ? u0 : u1) : ((float)n0 * u0 + (float)n1 * u1) / (float)(n0 + n1);
        const float t = cost_of(k, n0 + n1, units, kFmtFp4Block2D, 0);
        if (t < least) { best = k; least = t; }
    }
    if (best < 0) return hipErrorNotSupported;
    GemmArgs a = g, b = h;
    a.also = b.also = nullptr;
    if (c_is_bf16) return g.also_bf16 ? launch_t<kFmtFp4Block2D, true, true>(a, &b, best, stream)
                                      : launch_t<kFmtFp4Block2D, true, false>(a, &b, best, stream);
    return launch_t<kFmtFp4Block2D, false, false>(a, &b, best, stream);
}

}  // namespace q2d
