// Block-causal temporal convolution of the Mix-FFN with shortcut (Sec. 3.3.1, "Block Causal
// Mix-FFN"; Mix-FFN paragraph of Sec. 3.2) as one implicit GEMM on the matrix cores.
//
//   y[g][o] = x[g][o] + sum_tap sum_i W[tap][o][i] * src_tap(g)[i]
//
// for token rows g = (b, t, p) of a block of T frames x HW positions, where src_tap(g) is the row
// of the same position in frame t + tap - 1: a row of x, the cached last frame of the previous
// block for frame -1 (zeros without a cache), zeros for frame T.  So the A operand of the GEMM
// is x read three times with its rows shifted by -HW, 0, +HW tokens, the contraction runs over
// 3*D, and nothing is materialised.  Rows that are zero (frame -1 without a cache, frame T,
// token and channel tails, the K tail when D is not a multiple of the K-step) are read from a
// row of zeros in device memory, so the loader has no special cases.
//
// Tiling: a workgroup of four waves (one per SIMD) owns a BM-token x BN-channel tile of y (TcTile); wave (wm, wn) owns a
// quadrant of BM/2 x BN/2 as 16 x 16 accumulators of v_mfma_f32_16x16x32_bf16.  Both operands are K-contiguous
// ([token][channel] and [out][in]), so a K-step of 32 is a [BM][32] and a [BN][32] bf16 tile, and LDS holds a ring of
// four such stages.  Large tiles are bound by the power the matrix cores may draw: with random operands, 1 152
// workgroups of nothing but MFMAs take 604 us with 32 x 32 x 16 instructions and 544 with 16 x 16 x 32 (the
// same products; 469 and 475 with zeros, where the clock holds).  Taps whose rows are all zero are left out where a whole
// tile sees only such rows (tiles inside the last frame: no third tap).  With both, and the schedule below, the 480p clip at 2 240
// channels went from 855 to 796 us (1.12 to 1.20 PFLOP/s of useful products), a block of three frames from 142 to 138.
//
// Pipeline: operand tiles go from global memory straight into LDS (global_load_lds_dwordx4: a
// wave's 64 lanes fill 1 KB of consecutive LDS, no staging registers, completion counted by
// vmcnt).  With one wave per SIMD nothing but the wave itself can fill the time the matrix core
// works, so every memory instruction sits between two MFMAs.  Step s (stage s & 3):
//   barrier      after waiting for this wave's loads of step s+1 and its own reads of stage s
//   MFMAs        on the operand registers of step s, between them: the operands of step s+1 from stage s+1 into the
//                other register set; the loads of step s+4 into stage s (every wave has read it: the
//                barrier has passed)
// so a tile is requested three steps before its first use.  Steps past the end read the row of zeros: the loop body has no
// conditions.
//
// LDS rows are 64 bytes; the 16-byte chunk c of row r sits at chunk slot c ^ f(r); the lane that fills slot (r, c') therefore loads chunk
// c' ^ f(r) of row r.  For operands of 16 rows (four chunk columns) f = tc_swizzle16, for operands of 32 rows tc_swizzle: each leaves
// the 16-byte reads free of bank conflicts (2 to 6 % of LDS-active cycles; the 16-row kernels had them on half with the
// other one: the clip 819 -> 793 us, one block 157 -> 148).
#pragma once

#include <type_traits>

#include "common.hpp"
#include "tconv_tiles.hpp"

namespace sv {

constexpr int kTcBK = 32;                                     // K-step
constexpr int kTcStages = 4;
constexpr int kTcMaxD = 32768;                                // length of the row of zeros

// Tile shape and what follows from it.
template <int BM_, int BN_> struct TcTile {
    static constexpr int BM = BM_, BN = BN_;
    static constexpr int MB = BM / 32, NB = BN / 32;          // 16-row and 16-column blocks of a wave's quadrant
    static constexpr int MP = BM / 64, NP = (BN + 63) / 64;   // loads per lane and step: 64 rows each
    static constexpr int LOADS = MP + NP;
    static constexpr int kTileA = BM * kTcBK * 2, kStage = kTileA + NP * 64 * kTcBK * 2;
    // epilogue: 16 rows of a wave's quadrant in fp32 through LDS; CL lanes of eight channels make a row
    static constexpr int CL = BN > 128 ? 16 : BN / 16, ROWS = 64 / CL, ITERS = 16 / ROWS;
    static constexpr int kEpiPitch = BN / 2 * 4 + 32;
    static constexpr int kLdsBytes = kTcStages * kStage > 4 * 16 * kEpiPitch ? kTcStages * kStage : 4 * 16 * kEpiPitch;
    static_assert(BM % 64 == 0 && BN % 32 == 0 && BN / 16 <= 16 && (BN > 128 || (BN & (BN - 1)) == 0), "tile shape");
};

// A row of zeros for operand rows that do not exist.  Never written.
static __device__ __align__(16) uint16_t tc_zero_row[kTcMaxD];

struct TconvArgs {
    const uint16_t *x, *W, *cache;     // cache may be null
    uint16_t *y;
    int B, T, HW, D;
    int tiles_m, tiles_n;              // token tiles, channel tiles
};

__device__ __forceinline__ uint32_t tc_swizzle(int r) { return (uint32_t)(((r >> 1) & 3) ^ ((r >> 3) & 1)); }

// The same for operands of 16 rows (16 x 16 x 32 instructions): 16 lanes at a time, {0-3, 12-15, 20-27} and {4-11, 16-19, 28-31} of each half
// wave, read 256 bytes.
__device__ __forceinline__ uint32_t tc_swizzle16(int r)
{
    const int g = (r >> 2) & 3;
    return (uint32_t)((((g ^ (g >> 1)) & 1) << 1) | (g >> 1));
}

// 16 bytes per lane from global memory to LDS: lane l of the wave writes lds_wave_base + 16 l.
__device__ __forceinline__ void tc_load_to_lds(const uint16_t *src, unsigned char *lds_wave_base)
{
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src,
                                     (__attribute__((address_space(3))) void *)lds_wave_base, 16, 0, 0);
}

// acc += a * b with the accumulator in the accumulation registers.  As a statement in assembly because the builtin leaves the choice of the
// register file to the compiler, which then moved accumulators to the other file and back in every pass of the loop (256 x 128:
// 192 moves for 64 MFMAs; tconv_frames: 150 for 240).  What the compiler does not see to in return: operands come from LDS
// reads only (their waits it does insert), an accumulator is used again no sooner than four MFMAs later, and
// tc_mfma_done() stands before the first other use.  What register allocation adds at a loop's end, copies of accumulators, comes before
// tc_mfma_done(): a loop whose last instructions are products ends with tc_mfma_settle().  test_host_mfma_hazards.py reads the generated code for
// all of this.
__device__ __forceinline__ void tc_mfma(f32x4 &acc, bf16x8 a, bf16x8 b)
{
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
// Eight wait states, what a 16 x 16 x 32 product needs before anything but a product of the same accumulator reads what it wrote.
__device__ __forceinline__ void tc_mfma_settle() { asm volatile("s_nop 7" ::: "memory"); }
template <int M, int N> __device__ __forceinline__ void tc_mfma_done(f32x4 (&acc)[M][N])
{
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
    for (int i = 0; i < M; ++i)
#pragma unroll
        for (int j = 0; j < N; ++j) asm volatile("" : "+a"(acc[i][j]));
}

// SKIP: measurement variants (sv_measure_tconv_variant; the library's own calls use 0): bit 0 leaves the
// loads into LDS out of the tile loop, bit 1 the operand reads from LDS.  Such a launch touches the same
// memory and writes every element of y, but what it writes is not the convolution.
template <class P, int SKIP = 0>
__global__ __launch_bounds__(kThreads) void tconv_mfma(TconvArgs a)
{
    constexpr int MB = P::MB, NB = P::NB, MP = P::MP, NP = P::NP, LOADS = P::LOADS;
    extern __shared__ __align__(16) unsigned char lds[];
    int tm, tn;
    if (!tc_tile_of(a.tiles_m, a.tiles_n, (int)blockIdx.x, tm, tn)) return;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave & 1, wn = wave >> 1;
    const int M = a.B * a.T * a.HW, D = a.D;
    const int m0 = tm * P::BM, n0 = tn * P::BN;
    const int KC = (D + kTcBK - 1) / kTcBK;

    // the taps that some row of the tile needs (tc_taps): frame -1 without a cache and frame T are zero
    int tap_lo, tap_hi;
    tc_taps(m0, tc_last_row(m0, P::BM, M), a.HW, a.T, a.cache != nullptr, tap_lo, tap_hi);
    const int steps = (tap_hi - tap_lo) * KC;

    // ---- loader role: one 16-byte chunk of rows r0 + 64 i of both operand tiles ------------------
    const int r0 = tid >> 2, c4 = (tid & 3) ^ (int)tc_swizzle16(r0);   // c4: the chunk whose slot is this lane's
    const uint16_t *srcA[MP], *srcB[NP]; // the lane's chunk of each row at K-step 0 of the current tap
    uint32_t kinds = 0;                  // of row r0 + 64 i: bit 2 i, a token of the block; bit 2 i + 1, of its last frame
    // Sources of tap 1 or 2: the row itself or the one a frame behind it.
    auto set_tap = [&](int tap) __attribute__((always_inline)) {
        const uint32_t take = tap == 1 ? kinds & 0x55555555u : kinds & ~(kinds >> 1) & 0x55555555u;
#pragma unroll
        for (int i = 0; i < MP; ++i) {
            const uint16_t *in_x = a.x + ((int64_t)(m0 + r0 + 64 * i) + (int64_t)(tap - 1) * a.HW) * D;
            srcA[i] = (take >> (2 * i) & 1u ? in_x : tc_zero_row) + c4 * 8;
        }
    };
    auto set_weights = [&](int tap) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int n = r0 + 64 * i;
            srcB[i] = (n >= P::BN || n0 + n >= D ? tc_zero_row : a.W + ((int64_t)tap * D + n0 + n) * D) + c4 * 8;
        }
    };
    // Sources of the tile's first tap.  Tap 0 reads the frame in front: x, or for the first frame the cache (or zeros).
#pragma unroll
    for (int i = 0; i < MP; ++i) {
        const int g = m0 + r0 + 64 * i, gc = g < M ? g : M - 1;
        const int thw = a.T * a.HW, b = gc / thw, rem = gc - b * thw, t = rem / a.HW;
        const uint16_t *in_x = a.x + ((int64_t)g - a.HW) * D, *in_c = a.cache + (int64_t)(b * a.HW + (rem - t * a.HW)) * D;
        kinds |= (g < M ? 1u : 0u) << (2 * i) | (t == a.T - 1 ? 2u : 0u) << (2 * i);
        srcA[i] = (g >= M || (t == 0 && !a.cache) ? tc_zero_row : t == 0 ? in_c : in_x) + c4 * 8;
    }
    if (tap_lo == 1) set_tap(1);
    set_weights(tap_lo);
    int tap_n = tap_lo, kc_n = 0;      // the step to request next
    // The last K-step of a tap, when D is not a multiple of the step: lanes whose chunk lies past the row read zeros.  (The
    // pointers are set anew for the next tap.)
    auto clip_tail = [&]() __attribute__((always_inline)) {
        if (kc_n == KC - 1 && kc_n * kTcBK + c4 * 8 >= D) {
#pragma unroll
            for (int i = 0; i < MP; ++i) srcA[i] = tc_zero_row + (c4 * 8 - kc_n * kTcBK);
#pragma unroll
            for (int i = 0; i < NP; ++i) srcB[i] = tc_zero_row + (c4 * 8 - kc_n * kTcBK);
        }
    };
    clip_tail();
    auto advance = [&]() {
        if (kc_n + 1 < KC) {
            ++kc_n;
        } else if (tap_n + 1 < tap_hi) {
            kc_n = 0;
            ++tap_n;
            set_tap(tap_n);
            set_weights(tap_n);
        } else {                       // past the last step: zeros
            kc_n = 0;
#pragma unroll
            for (int i = 0; i < MP; ++i) srcA[i] = tc_zero_row + c4 * 8;
#pragma unroll
            for (int i = 0; i < NP; ++i) srcB[i] = tc_zero_row + c4 * 8;
        }
        clip_tail();
    };
    // Requests load m (m < MP: A row pass m, else B row pass m - MP) of the step to request next.
    auto request_one = [&](int stage, int m, bool leave_out = false) __attribute__((always_inline)) {
        const uint16_t *p = (m < MP ? srcA[m < MP ? m : 0] : srcB[m < MP ? 0 : m - MP]) + kc_n * kTcBK;
        if (leave_out) {               // the address all the same: without it the compiler lays out another loop
            asm volatile("" ::"v"(p));
            return;
        }
        tc_load_to_lds(p, lds + stage * P::kStage + (m < MP ? m * 4096 : P::kTileA + (m - MP) * 4096) + wave * 1024);
    };

    // ---- consumer role: lane l holds chunk l / 16 of row l % 16 of a 16-row block ----------------------
    const uint32_t in_block = (uint32_t)(lane & 15) * 64u + ((((uint32_t)lane >> 4) ^ tc_swizzle16(lane & 15)) << 4);
    const uint32_t rdA = (uint32_t)(wm * (P::BM / 2)) * 64u + in_block;
    const uint32_t rdB = (uint32_t)P::kTileA + (uint32_t)(wn * (P::BN / 2)) * 64u + in_block;
    // operand m of a step: A row block m (m < MB) or B row block m - MB
    auto operand = [&](int stage, int m) -> bf16x8 {
        return *reinterpret_cast<const bf16x8 *>(lds + stage * P::kStage + (m < MB ? rdA + m * 1024 : rdB + (m - MB) * 1024));
    };

    f32x4 acc[MB][NB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    bf16x8 op[2][MB + NB];             // two register sets: the step's operands and the next step's

    // ---- prologue: steps 0..3 requested, step 0 arrived ---------------------------------------------
#pragma unroll
    for (int st = 0; st < kTcStages; ++st) {
#pragma unroll
        for (int m = 0; m < LOADS; ++m) request_one(st, m);
        advance();
    }
    if (SKIP & 1) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // no loads in the loop: the ring is read over and over
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(3 * LOADS) : "memory");
#pragma unroll
    for (int m = 0; m < MB + NB; ++m) op[0][m] = operand(0, m);
    if (SKIP & 2) {
#pragma unroll
        for (int m = 0; m < MB + NB; ++m) op[1][m] = operand(1, m);
    }

    // One step: the MFMAs on register set `cur`, and between them the operand reads, spread over three quarters of them (one
    // after every MFMA asks twice what LDS delivers and holds up the wave), and, evenly spread, the loads.
    auto step = [&](int s, auto cur_c) __attribute__((always_inline)) {
        constexpr int cur = decltype(cur_c)::value, READS = MB + NB, MFMAS = MB * NB;
        const int stage = s & 3, next = (s + 1) & 3;
        // this wave's loads of step s+1 have landed (those of steps s+2 and s+3 may be in flight) and its reads
        // of stage s are done; then so have everybody's
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(2 * LOADS) : "memory");
#pragma unroll
        for (int m = 0; m < MFMAS; ++m) {
            tc_mfma(acc[m / NB][m % NB], op[cur][m / NB], op[cur][MB + m % NB]);
            if (!(SKIP & 2)) {
#pragma unroll
                for (int k = 0; k < READS; ++k)
                    if (m == k * (MFMAS * 3 / 4) / READS) op[cur ^ 1][k] = operand(next, k);
            }
#pragma unroll
            for (int l = 0; l < LOADS; ++l)
                if (m == l * MFMAS / LOADS) request_one(stage, l, SKIP & 1);
            __builtin_amdgcn_sched_barrier(0);
        }
        advance();
    };
    for (int s = 0; s < steps; s += 2) {   // an odd number of steps ends with one of zeros
        step(s, std::integral_constant<int, 0>{});
        step(s + 1, std::integral_constant<int, 1>{});
    }
    tc_mfma_done(acc);
    // ---- epilogue: y = bf16(x + acc), 16 token rows of the wave's quadrant at a time through LDS ----
    // (nobody reads the operand ring any more; each wave uses its own region).  The shortcut's x rows
    // are requested one row group ahead, so their latency is paid once per tile, not once per row.
    constexpr int CL = P::CL, ROWS = P::ROWS, ITERS = P::ITERS;
    unsigned char *epi = lds + wave * (16 * P::kEpiPitch);
    const int er = lane / CL, ec = lane % CL;                 // reader: row in a group of ROWS, 8-channel chunk
    const int n = n0 + wn * (P::BN / 2) + ec * 8;
    const bool col_ok = ec * 8 < P::BN / 2 && n < D;
    const int n_ld = col_ok ? n : 0;                          // lanes past the last channel load a valid address
    u32x4 xin[2][ITERS];
    auto load_x = [&](int buf, int i) {
#pragma unroll
        for (int it = 0; it < ITERS; ++it) {
            const int64_t g = (int64_t)m0 + wm * (P::BM / 2) + i * 16 + it * ROWS + er;
            xin[buf][it] = *reinterpret_cast<const u32x4 *>(a.x + (g < M ? g : (int64_t)M - 1) * D + n_ld);
        }
    };
    load_x(0, 0);
    // the loads past the last step must not land on the epilogue's staging
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
    for (int i = 0; i < MB; ++i) {
        if (i + 1 < MB) load_x((i + 1) & 1, i + 1);
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                *reinterpret_cast<float *>(epi + ((lane >> 4) * 4 + r) * P::kEpiPitch + (j * 16 + (lane & 15)) * 4) = acc[i][j][r];
        wave_lds_fence();
#pragma unroll
        for (int it = 0; it < ITERS; ++it) {
            const int row = it * ROWS + er;
            const int64_t g = (int64_t)m0 + wm * (P::BM / 2) + i * 16 + row;
            const int at = row * P::kEpiPitch + (col_ok ? ec : 0) * 32;
            const f32x4 lo = *reinterpret_cast<const f32x4 *>(epi + at);
            const f32x4 hi = *reinterpret_cast<const f32x4 *>(epi + at + 16);
            if (g < M && col_ok) {
                const u32x4 x4 = xin[i & 1][it];
                u32x4 out;
                out.x = pack_bf16x2(bf16_lo(x4.x) + lo.x, bf16_hi(x4.x) + lo.y);
                out.y = pack_bf16x2(bf16_lo(x4.y) + lo.z, bf16_hi(x4.y) + lo.w);
                out.z = pack_bf16x2(bf16_lo(x4.z) + hi.x, bf16_hi(x4.z) + hi.y);
                out.w = pack_bf16x2(bf16_lo(x4.w) + hi.z, bf16_hi(x4.w) + hi.w);
                *reinterpret_cast<u32x4 *>(a.y + g * D + n) = out;
            }
        }
        wave_lds_fence();
    }
}

// The same convolution with 32 x 32 x 16 MFMAs on tiles of 256 x 256: a wave's quadrant is 4 x 4 accumulators, an instruction runs
// twice as long and hides a memory instruction beside it, which makes the step shorter (0.56 against 0.62 us) while the matrix
// cores' power is no limit: with up to two thirds of the compute units at work (tconv_form).  Step s:
//   first half   16 MFMAs on operand registers of K-chunk 0; reads K-chunk 1 of stage s; requests the B rows of step s+3
//   barrier      after waiting for this wave's loads of step s+1 and its own LDS reads
//   second half  16 MFMAs on K-chunk 1; reads K-chunk 0 of stage s+1; requests the A rows of step s+4 into stage s
// Steps past the end repeat the last one into stages nobody reads.  KTAIL: D is not a multiple of the K-step, the last K-step of
// a tap has chunks past the row end.
constexpr int kTcBM = 256, kTcBN = 256;
constexpr int kTcTileBytes = kTcBM * kTcBK * 2;               // one operand tile of one K-step
constexpr int kTcStageBytes = 2 * kTcTileBytes;               // A and B
constexpr int kTcLdsBytes = kTcStages * kTcStageBytes;
constexpr int kTcEpiPitch = 128 * 4 + 32;                     // fp32 row of a wave's quadrant in the epilogue
static_assert(4 * 32 * kTcEpiPitch <= kTcLdsBytes, "epilogue staging fits in the operand ring");
template <bool KTAIL>
__global__ __launch_bounds__(kThreads) void tconv_mfma32(TconvArgs a)
{
    extern __shared__ __align__(16) unsigned char lds[];
    int tm, tn;
    if (!tc_tile_of(a.tiles_m, a.tiles_n, (int)blockIdx.x, tm, tn)) return;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave & 1, wn = wave >> 1;
    const int M = a.B * a.T * a.HW, D = a.D;
    const int m0 = tm * kTcBM, n0 = tn * kTcBN;
    const int KC = (D + kTcBK - 1) / kTcBK;
    int tap_lo, tap_hi;                // the taps that some row of the tile needs
    tc_taps(m0, tc_last_row(m0, kTcBM, M), a.HW, a.T, a.cache != nullptr, tap_lo, tap_hi);
    const int steps = (tap_hi - tap_lo) * KC;

    // ---- loader role: one 16-byte chunk of rows r0 + 64 i of both operand tiles ------------------
    const int r0 = tid >> 2, c4 = (tid & 3) ^ (int)tc_swizzle(r0);   // c4: the chunk whose slot is this lane's
    int row_t[4], row_c[4];            // frame of the row (or a large value past M), cache row index
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int g = m0 + r0 + 64 * i, gc = g < M ? g : M - 1;
        const int thw = a.T * a.HW, b = gc / thw, rem = gc - b * thw, t = rem / a.HW;
        row_t[i] = g < M ? t : 1 << 20;      // rows past the last token: every tap sees them as past the block
        row_c[i] = b * a.HW + (rem - t * a.HW);
    }
    const uint16_t *srcA[4], *srcB[4]; // the lane's chunk of each row at K-step 0 of the current tap
    auto set_tap = [&](int tap) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int ts = row_t[i] + tap - 1;
            const bool front = ts < 0, zero = ts >= a.T || (front && !a.cache);
            const uint16_t *in_x = a.x + ((int64_t)(m0 + r0 + 64 * i) + (int64_t)(tap - 1) * a.HW) * D;
            const uint16_t *in_c = a.cache + (int64_t)row_c[i] * D;
            srcA[i] = (zero ? tc_zero_row : (front ? in_c : in_x)) + c4 * 8;
            const int n = n0 + r0 + 64 * i;
            srcB[i] = (n >= D ? tc_zero_row : a.W + ((int64_t)tap * D + n) * D) + c4 * 8;
        }
    };
    int tap_n = tap_lo, kc_n = 0;           // the step to request next
    auto advance = [&]() {
        if (kc_n + 1 < KC) {
            ++kc_n;
        } else if (tap_n + 1 < tap_hi) {
            kc_n = 0;
            set_tap(++tap_n);
        }                              // else: stay on the last step
    };
    // Source of load m (m < 4: A row pass m, else B row pass m - 4) of the step to request next.
    auto source = [&](int m) -> const uint16_t * {
        const uint16_t *p = (m < 4 ? srcA[m] : srcB[m - 4]) + kc_n * kTcBK;
        if (KTAIL && kc_n * kTcBK + c4 * 8 >= D) p = tc_zero_row;
        return p;
    };
    auto request_one = [&](int stage, int m) {
        unsigned char *dst = lds + stage * kTcStageBytes + (m < 4 ? 0 : kTcTileBytes) + ((m & 3) * 64 + wave * 16) * 64;
        tc_load_to_lds(source(m), dst);
    };

    // ---- consumer role ------------------------------------------------------------------------------
    uint32_t ko[2];                    // byte offset of K-chunk pair kk inside the lane's operand row
    {
        const uint32_t g = (uint32_t)(lane >> 5) ^ tc_swizzle(lane & 31);
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) ko[kk] = (((uint32_t)kk << 1) ^ g) << 4;
    }
    const uint32_t rdA = (uint32_t)(wm * 128 + (lane & 31)) * 64u;
    const uint32_t rdB = (uint32_t)kTcTileBytes + (uint32_t)(wn * 128 + (lane & 31)) * 64u;
    // operand m of a set: A row block m (m < 4) or B row block m - 4
    auto operand = [&](int stage, int kk, int m) -> bf16x8 {
        const unsigned char *base = lds + stage * kTcStageBytes + (m < 4 ? rdA : rdB) + (m & 3) * 2048 + ko[kk];
        return *reinterpret_cast<const bf16x8 *>(base);
    };

    f32x16 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    bf16x8 op[2][8];                   // op[kk][0..3] = A row blocks, op[kk][4..7] = B row blocks

    // ---- prologue: steps 0..2 and the A half of step 3 requested, step 0 arrived --------------------
    set_tap(tap_lo);
#pragma unroll
    for (int st = 0; st < kTcStages - 1; ++st) {
#pragma unroll
        for (int m = 0; m < 8; ++m) request_one(st, m);
        advance();
    }
#pragma unroll
    for (int m = 0; m < 4; ++m) request_one(kTcStages - 1, m);
    asm volatile("s_waitcnt vmcnt(20)\n\ts_barrier" ::: "memory");
#pragma unroll
    for (int m = 0; m < 8; ++m) op[0][m] = operand(0, 0, m);

    // A load instruction keeps the wave from issuing for longer than one MFMA runs, so the eight
    // loads of a step are spread out: one after every second MFMA of the second half of one step
    // (A rows) and of the first half of the next (B rows).
    for (int s = 0; s < steps; ++s) {
        const int cur = s & 3, nxt = (s + 1) & 3, prv = (s + 3) & 3;
#pragma unroll
        for (int m = 0; m < 16; ++m) {
            acc[m >> 2][m & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op[0][m >> 2], op[0][4 + (m & 3)],
                                                                          acc[m >> 2][m & 3], 0, 0, 0);
            if (m < 8) op[1][m] = operand(cur, 1, m);
            if (m >= 8 && (m & 1)) request_one(prv, 4 + ((m - 8) >> 1));     // B rows of step s+3
            __builtin_amdgcn_sched_barrier(0);
        }
        advance();
        // this wave's loads of step s+1 have landed (those of steps s+2 and s+3 may be in flight) and its reads
        // of stage s are done; then so have everybody's
        asm volatile("s_waitcnt vmcnt(16) lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
        for (int m = 0; m < 16; ++m) {
            acc[m >> 2][m & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op[1][m >> 2], op[1][4 + (m & 3)],
                                                                          acc[m >> 2][m & 3], 0, 0, 0);
            if (m < 8) op[0][m] = operand(nxt, 0, m);
            if (m >= 8 && (m & 1)) request_one(cur, (m - 8) >> 1);           // A rows of step s+4
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // ---- epilogue: y = bf16(x + acc), 32 token rows of the wave's quadrant at a time through LDS ----
    // (nobody reads the operand ring any more; each wave uses its own region).  The shortcut's x rows
    // are requested one 32-row group ahead, so their latency is paid once per tile, not once per row.
    unsigned char *epi = lds + wave * (32 * kTcEpiPitch);
    const int er = lane >> 4, ec = lane & 15;                 // reader: row in a group of four, 8-channel chunk
    const int n = n0 + wn * 128 + ec * 8;
    const bool col_ok = n < D;
    const int n_ld = col_ok ? n : 0;                          // lanes past the last channel load a valid address
    u32x4 xin[2][8];
    auto load_x = [&](int buf, int i) {
#pragma unroll
        for (int it = 0; it < 8; ++it) {
            const int64_t g = (int64_t)m0 + wm * 128 + i * 32 + it * 4 + er;
            xin[buf][it] = *reinterpret_cast<const u32x4 *>(a.x + (g < M ? g : (int64_t)M - 1) * D + n_ld);
        }
    };
    load_x(0, 0);
    // the repeated loads of the last steps must not land on the epilogue's staging
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (i + 1 < 4) load_x((i + 1) & 1, i + 1);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3), col = j * 32 + (lane & 31);
                *reinterpret_cast<float *>(epi + row * kTcEpiPitch + col * 4) = acc[i][j][r];
            }
        wave_lds_fence();
#pragma unroll
        for (int it = 0; it < 8; ++it) {
            const int row = it * 4 + er;
            const int64_t g = (int64_t)m0 + wm * 128 + i * 32 + row;
            const f32x4 lo = *reinterpret_cast<const f32x4 *>(epi + row * kTcEpiPitch + ec * 32);
            const f32x4 hi = *reinterpret_cast<const f32x4 *>(epi + row * kTcEpiPitch + ec * 32 + 16);
            if (g < M && col_ok) {
                const u32x4 x4 = xin[i & 1][it];
                u32x4 out;
                out.x = pack_bf16x2(bf16_lo(x4.x) + lo.x, bf16_hi(x4.x) + lo.y);
                out.y = pack_bf16x2(bf16_lo(x4.y) + lo.z, bf16_hi(x4.y) + lo.w);
                out.z = pack_bf16x2(bf16_lo(x4.z) + hi.x, bf16_hi(x4.z) + hi.y);
                out.w = pack_bf16x2(bf16_lo(x4.w) + hi.z, bf16_hi(x4.w) + hi.w);
                *reinterpret_cast<u32x4 *>(a.y + g * D + n) = out;
            }
        }
        wave_lds_fence();
    }
}

// New cache = last input frame of the block: cache[b][p][:] = x[b][T-1][p][:], 16 bytes per thread.
__global__ __launch_bounds__(kThreads) void tconv_cache_store(const uint16_t *x, uint16_t *cache, int B, int T, int HW, int D)
{
    const int64_t per_batch = (int64_t)HW * D / 8, total = per_batch * B;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t b = e / per_batch, r = e - b * per_batch;
        const u32x4 v = reinterpret_cast<const u32x4 *>(x + ((b * T + (T - 1)) * (int64_t)HW) * D)[r];
        reinterpret_cast<u32x4 *>(cache + b * (int64_t)HW * D)[r] = v;
    }
}

}  // namespace sv
