// Block-causal temporal convolution of the Mix-FFN (see tconv_mfma.hpp for the definition) on tiles of frames x positions.
//
// tconv_mfma takes a tile of consecutive token rows through the taps one after the other and fetches the rows anew for each, shifted by
// a frame.  Here a tile is F frames x P positions (token rows) x BN channels: the same source rows, frames -1 to F (or F - 1)
// of the tile's positions, serve all three taps, frame f taking tap t from source frame f + t - 1.  The loop runs over
// K-steps of 32 channels with three sub-steps, one per tap: a K-step brings (F + 1 or 2) P rows of x and 3 BN rows of W into LDS, where
// the row tiles bring 3 (BM + BN).  That is what large calls are bound by: the path from the L2 into LDS delivers
// 11 to 12 TB/s with all compute units loading.  And taps that meet a zero frame (behind the last one, in front of the first without a
// cache) are left out for every frame, where a row tile had to lie in that frame as a whole.
//
// A workgroup of four waves; wave w owns 16 NB channels of all the tile's rows as 16 x 16 accumulators.  Per K-step a wave reads each
// source block (16 positions of a frame) once from LDS into registers and uses it for three taps x NB channel blocks.
//
// Pipeline, sub-step s = 3 k + t (K-step k, tap t):
//   barrier   after waiting for this wave's loads of W(s + 1) and, at t = 0, x(k + 1), and for its own LDS reads
//   MFMAs     on the operand registers of the sub-step; between them: W operands of s + 1 and a third of the x operands of k + 1 from
//             LDS into the other register set; the loads of W(s + 6) into the slot of W(s) and a third of x(k + 3) into the slot
//             of x(k), which every wave has read
// LDS rows, swizzle and the loads straight into LDS are those of tconv_mfma.  Channels are a multiple of 32.  With an odd number of K-steps
// the last pass takes one more, of zeros on both sides.
#pragma once

#include "tconv_mfma.hpp"

namespace sv {

// FRONT, BACK: there is a frame in front of the tile (the cache) and one behind it.  Both false or true at compile time, so that the
// products they leave out are no branch; a call of several groups of frames takes both and multiplies with the zero frames at its ends.
template <int F_, int PB_, int NB_, bool FRONT_, bool BACK_> struct FrameTile {
    static constexpr int F = F_, PB = PB_, NB = NB_;
    static constexpr bool FRONT = FRONT_, BACK = BACK_;
    static constexpr int P = 16 * PB, BN = 64 * NB, J = F + 1 + (BACK ? 1 : 0);   // source frames
    static constexpr int LA = (J * P + 63) / 64, LW = NB;     // loads per lane of an x tile and a W tile: 64 rows each
    static constexpr int kA = LA * 4096, kW = LW * 4096, NA = 3, NW = 6, kWOffset = NA * kA;
    static constexpr int kEpiPitch = NB * 64 + 32;
    static constexpr int kLdsBytes = NA * kA + NW * kW;
    static_assert(4 * 16 * kEpiPitch <= kLdsBytes && kLdsBytes <= 160 * 1024, "LDS");
    // loads of an x tile and reads of its operands that sub-step t issues
    static constexpr int load_lo(int t) { return LA * t / 3; }
    static constexpr int read_lo(int t) { return J * PB * t / 3; }
    static constexpr int loads(int t) { return LW + load_lo(t + 1) - load_lo(t); }
};

// grid = tc_grid_size(tiles_m * tiles_n), block = 256; token tile tm = (batch, group of F frames, group of P positions)
template <class S>
__global__ __launch_bounds__(kThreads) void tconv_frames(TconvArgs a)
{
    constexpr int F = S::F, PB = S::PB, NB = S::NB, J = S::J, P = S::P, LA = S::LA, LW = S::LW, NW = S::NW;
    extern __shared__ __align__(16) unsigned char lds[];
    int tm, tn;
    if (!tc_tile_of(a.tiles_m, a.tiles_n, (int)blockIdx.x, tm, tn)) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int D = a.D, KC = D / kTcBK;
    const int pos_tiles = (a.HW + P - 1) / P, groups = (a.T + F - 1) / F;
    const int b = tm / (groups * pos_tiles), rest = tm - b * groups * pos_tiles, f0 = rest / pos_tiles * F, p0 = (rest - rest / pos_tiles * pos_tiles) * P;
    const int n0 = tn * S::BN;

    // ---- loader role: one 16-byte chunk of rows r0 + 64 i of both operand tiles.  Positions and channels past the end take the last
    // one's (their products are never stored), frames that do not exist the row of zeros.
    const int r0 = tid >> 2, c4 = (tid & 3) ^ (int)tc_swizzle16(r0);
    const uint16_t *srcA[LA];
    uint32_t offW[LW];                                        // bytes into a tap's matrix; 3 D D < 2^31
#pragma unroll
    for (int i = 0; i < LA; ++i) {
        const int r = r0 + 64 * i, j = r / P, f = f0 - 1 + j;
        int p = p0 + r - j * P;
        p = p < a.HW ? p : a.HW - 1;
        const uint16_t *in_x = a.x + (((int64_t)b * a.T + f) * a.HW + p) * D, *in_c = a.cache + ((int64_t)b * a.HW + p) * D;
        srcA[i] = (j >= J || f >= a.T || (f < 0 && !a.cache) ? tc_zero_row : f < 0 ? in_c : in_x) + c4 * 8;
    }
#pragma unroll
    for (int i = 0; i < LW; ++i) {
        const int n = n0 + r0 + 64 * i;
        offW[i] = ((uint32_t)(n < D ? n : D - 1) * (uint32_t)D + (uint32_t)c4 * 8u) * 2u;
    }
    const uint16_t *zero = tc_zero_row + c4 * 8;
    auto load_a = [&](int k, int slot, int i) __attribute__((always_inline)) {
        tc_load_to_lds(k < KC ? srcA[i] + k * kTcBK : zero, lds + slot * S::kA + i * 4096 + wave * 1024);
    };
    auto load_w = [&](int k, int t, int slot, int i) __attribute__((always_inline)) {
        const uint16_t *base = k < KC ? a.W + ((int64_t)t * D * D + k * kTcBK) : tc_zero_row;
        const uint32_t off = k < KC ? offW[i] : (uint32_t)c4 * 16u;
        tc_load_to_lds(reinterpret_cast<const uint16_t *>(reinterpret_cast<const unsigned char *>(base) + off),
                       lds + S::kWOffset + slot * S::kW + i * 4096 + wave * 1024);
    };

    // ---- consumer role: lane l holds chunk l / 16 of row l % 16 of a 16-row block ----------------------
    const uint32_t in_block = (uint32_t)(lane & 15) * 64u + ((((uint32_t)lane >> 4) ^ tc_swizzle16(lane & 15)) << 4);
    auto read_a = [&](int slot, int m) -> bf16x8 {            // m = source frame * PB + block
        return *reinterpret_cast<const bf16x8 *>(lds + slot * S::kA + m * 1024 + in_block);
    };
    auto read_w = [&](int slot, int nb) -> bf16x8 {
        return *reinterpret_cast<const bf16x8 *>(lds + S::kWOffset + slot * S::kW + (wave * NB + nb) * 1024 + in_block);
    };
    f32x4 acc[F * PB][NB];
#pragma unroll
    for (int i = 0; i < F * PB; ++i)
#pragma unroll
        for (int n = 0; n < NB; ++n) acc[i][n] = f32x4{0.f, 0.f, 0.f, 0.f};
    bf16x8 opA[2][J * PB], opW[2][NB];                        // the operands in use and the next ones

    // ---- prologue: x(0..2) and W(0..5) requested, x(0) and W(0) arrived -----------------------------
    // (in an order in which the loop's waits, which count the loads behind the one they need, hold from the first sub-step on)
    auto all_a = [&](int k) {
#pragma unroll
        for (int i = 0; i < LA; ++i) load_a(k, k, i);
    };
    auto all_w = [&](int s) {
#pragma unroll
        for (int i = 0; i < LW; ++i) load_w(s / 3, s % 3, s, i);
    };
    all_a(0); all_w(0); all_w(1); all_a(1); all_w(2); all_w(3); all_a(2); all_w(4); all_w(5);
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(2 * LA + 5 * LW) : "memory");
#pragma unroll
    for (int m = 0; m < J * PB; ++m) opA[0][m] = read_a(0, m);
#pragma unroll
    for (int n = 0; n < NB; ++n) opW[0][n] = read_w(0, n);

    int slot = 0;                                             // of x(k)
    // sub-step u = 0 .. 5 of K-steps k and k + 1
    auto substep = [&](int k, auto u_c) __attribute__((always_inline)) {
        constexpr int u = decltype(u_c)::value, t = u % 3, kk = u / 3, cur = u & 1;
        constexpr int next_slot_w = (u + 1) % NW;
        const int s1 = slot + 1 >= 3 ? slot - 2 : slot + 1;   // of x(k + kk + 1)
        // loads of W(s + 1) and x(k + 1) have landed: what may be in flight are those of the last four sub-steps, at t = 0 three
        constexpr int in_flight = t == 0 ? S::loads(0) + S::loads(1) + S::loads(2)
                                         : S::loads(0) + S::loads(1) + S::loads(2) + S::loads((t + 2) % 3);
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(in_flight) : "memory");
        constexpr int f_lo = t == 0 && !S::FRONT ? 1 : 0, f_hi = t == 2 && !S::BACK ? F - 1 : F;   // frames whose source is not zero
        auto mfma = [&](int f, int pb, int nb) __attribute__((always_inline)) {
            tc_mfma(acc[f * PB + pb][nb], opA[kk][(f + t) * PB + pb], opW[cur][nb]);
        };
        constexpr int READS_A = S::read_lo(t + 1) - S::read_lo(t), READS = NB + READS_A, LOADS = S::loads(t);
        constexpr int MFMAS = (f_hi - f_lo) * PB * NB;
#pragma unroll
        for (int f = f_lo; f < f_hi; ++f)
#pragma unroll
            for (int pb = 0; pb < PB; ++pb)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    const int m = ((f - f_lo) * PB + pb) * NB + nb;
                    mfma(f, pb, nb);
#pragma unroll
                    for (int i = 0; i < READS; ++i)
                        if (m == i * (MFMAS * 3 / 4) / READS) {
                            if (i < NB) opW[cur ^ 1][i] = read_w(next_slot_w, i);
                            else opA[kk ^ 1][S::read_lo(t) + i - NB] = read_a(s1, S::read_lo(t) + i - NB);
                        }
#pragma unroll
                    for (int l = 0; l < LOADS; ++l)
                        if (m == l * MFMAS / LOADS) {
                            if (l < LW) load_w(k + kk + 2, t, u, l);
                            else load_a(k + kk + 3, slot, S::load_lo(t) + l - LW);
                        }
                    __builtin_amdgcn_sched_barrier(0);
                }
        if (t == 2) slot = s1;
    };
    for (int k = 0; k < KC; k += 2) {
        substep(k, std::integral_constant<int, 0>{});
        substep(k, std::integral_constant<int, 1>{});
        substep(k, std::integral_constant<int, 2>{});
        substep(k, std::integral_constant<int, 3>{});
        substep(k, std::integral_constant<int, 4>{});
        substep(k, std::integral_constant<int, 5>{});
        tc_mfma_settle();
    }

    tc_mfma_done(acc);
    // ---- epilogue: y = bf16(x + acc), a block of 16 positions at a time through the wave's own LDS; eight lanes of eight channels
    // make a row.  The shortcut's x rows are requested one block ahead.
    unsigned char *epi = lds + wave * (16 * S::kEpiPitch);
    const int er = lane >> 3, ec = lane & 7;
    const int n = n0 + wave * 16 * NB + ec * 8;
    const bool col_ok = ec < 2 * NB && n < D;
    const int n_ld = col_ok ? n : 0;
    u32x4 xin[2][2];
    auto row_of = [&](int i, int it) -> int64_t {             // row of x and y, or -1
        const int f = f0 + i / PB, p = p0 + (i % PB) * 16 + it * 8 + er;
        return f < a.T && p < a.HW ? ((int64_t)b * a.T + f) * a.HW + p : -1;
    };
    auto load_x = [&](int buf, int i) {
#pragma unroll
        for (int it = 0; it < 2; ++it) {
            const int64_t g = row_of(i, it);
            xin[buf][it] = *reinterpret_cast<const u32x4 *>(a.x + (g < 0 ? 0 : g) * D + n_ld);
        }
    };
    load_x(0, 0);
    // the loads past the last K-step must not land on the epilogue's staging
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
    for (int i = 0; i < F * PB; ++i) {
        if (i + 1 < F * PB) load_x((i + 1) & 1, i + 1);
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                *reinterpret_cast<float *>(epi + ((lane >> 4) * 4 + r) * S::kEpiPitch + (j * 16 + (lane & 15)) * 4) = acc[i][j][r];
        wave_lds_fence();
#pragma unroll
        for (int it = 0; it < 2; ++it) {
            const int64_t g = row_of(i, it);
            const int at = (it * 8 + er) * S::kEpiPitch + (col_ok ? ec : 0) * 32;
            const f32x4 lo = *reinterpret_cast<const f32x4 *>(epi + at), hi = *reinterpret_cast<const f32x4 *>(epi + at + 16);
            if (g >= 0 && col_ok) {
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

}  // namespace sv
