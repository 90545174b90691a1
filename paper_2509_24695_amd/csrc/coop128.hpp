// Apply for d = 112 and 128 (DP = 128): the waves of a workgroup work on the same tile
// together (the state kernel is in wide_state.hpp).
//
// With 64 features a wave can keep a whole 64 x 64 state (or a 64-column panel of it) to itself
// and never talks to its neighbours.  With 128 the state is four such quadrants and the apply
// needs several panels, so every token row is needed by more than one wave.  Letting all of them
// fetch it costs far more than the extra instructions: half rows of 224 or 256 bytes split cache
// lines between waves and the non-temporal streams fetch them twice (measured: 2.4 TB/s instead of
// 5.4).  Here each wave loads whole rows that nobody else loads, the tile is assembled in
// workgroup-shared LDS, and barriers hand it to the waves that compute:
//
//   apply: wave w loads rows 8w .. 8w+8 of a 32-token Q tile, computes 32 of the 128 output
//          features of the whole tile (its 128 x 32 panel of S stays in registers) into a shared
//          output tile, then stores whole rows 8w .. 8w+8 of O; two barriers per tile, two or
//          three workgroups per compute unit (see sv_linattn.hip; the stream and the loop are written for other splits of
//          the tile among the waves as well, see CoopApplyStream).
//
// Barriers are bare s_barrier instructions behind an LDS-only wait, so the global loads of later
// tiles and the stores of earlier ones stay in flight across them.  For d = 112 the features past
// 112 are addressed out of range: they read as zeros and their stores are dropped.
#pragma once

#include "apply_mfma.hpp"
#include "state_mfma.hpp"

namespace sv {

constexpr int kCoopRow = 128 * 2 + 16;           // LDS row: 128 bf16 features + padding
constexpr int kCoopTile = 32 * kCoopRow;         // one 32-token tile in LDS

// ---- apply ---------------------------------------------------------------------------------------

// One wave's share of the workgroup's Q/O stream, both for the loads of Q and for the stores of O.
// A wave computes NB blocks of 32 output features, so 4/NB waves work on one 32-token tile and a
// workgroup of WAVES waves takes WAVES*NB/4 tiles per step; its rows are dealt evenly to the waves:
//   WAVES = 4, NB = 1   one tile, 8 rows per wave, few enough registers for two waves per SIMD (in use)
//   WAVES = 4, NB = 2   a pair of tiles per step, 16 rows per wave
//   WAVES = 2, NB = 2   one tile, 16 rows per wave
template <int DEPTH, int ROPE, int WAVES, int NB, bool NT>
struct CoopApplyStream {
    static constexpr int STEP = 8 * WAVES * NB;   // tokens per workgroup step
    static constexpr int ROWS = STEP / WAVES;     // rows per wave
    static constexpr int NLD = ROWS / 4;          // 4 rows per load instruction
    rsrc_t rQ, rO;
    uint32_t row_bytes, lane_off;
    bool valid;
    TileWalk walk;                       // the workgroup's steps (units of STEP tokens)
    u32x4 q[DEPTH][NLD];
    Rotator<ROPE, NLD, DEPTH> rot;

    __device__ __forceinline__ CoopApplyStream(const uint16_t *Qh, uint16_t *Oh, const RopeArg &rope,
                                               const unsigned char *lds_tab, int64_t stride_n, int t1, int d, int wave,
                                               int lane, const TileWalk &w)
        : rQ(make_rsrc(Qh, (uint32_t)t1 * (uint32_t)stride_n * 2u)),
          rO(make_rsrc(Oh, (uint32_t)t1 * (uint32_t)stride_n * 2u)), row_bytes((uint32_t)stride_n * 2u),
          lane_off((uint32_t)(ROWS * wave + (lane >> 4)) * (uint32_t)stride_n * 2u + (uint32_t)(lane & 15) * 16u),
          valid((lane & 15) * 8 < d), walk(w),
          rot(rope, t1, d, ROWS * wave + (lane >> 4), 4, 4 * (lane & 15), 1, lds_tab) {}

    __device__ __forceinline__ void request(int s, int i)
    {
        const uint32_t base = valid ? walk.offset<STEP>(i, row_bytes) : kOutOfRange;
#pragma unroll
        for (int j = 0; j < NLD; ++j) q[s][j] = load_stream16<NT>(rQ, base + lane_off + (uint32_t)j * 4u * row_bytes);
        rot.request(s, i < walk.count, walk.token<STEP>(i));
    }
};

template <int FROM, int TO, int DEPTH, int ROPE, int WAVES, int NB, bool NT>
__device__ __forceinline__ void coop_apply_prefetch(CoopApplyStream<DEPTH, ROPE, WAVES, NB, NT> &st)
{
#pragma unroll
    for (int s = FROM; s < TO; ++s) {
        st.request(s, s);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// LDS of the apply phase: the Q tiles of a step (as the MFMAs want them: rotated with ROPE), its
// O tiles and the denominators of its tokens.
template <int WAVES, int NB> __host__ __device__ constexpr int coop_apply_lds_bytes() {
    return 2 * (WAVES * NB / 4) * kCoopTile + 8 * WAVES * NB * 4;
}

// The lane's part of phi(Q_i) . z: eight features of a row and the matching key sums.
__device__ __forceinline__ float key_sum_products(u32x4 pq, const float (&zr)[8])
{
    float dot = bf16_lo(pq.x) * zr[0];
    dot = __builtin_fmaf(bf16_hi(pq.x), zr[1], dot);
    dot = __builtin_fmaf(bf16_lo(pq.y), zr[2], dot);
    dot = __builtin_fmaf(bf16_hi(pq.y), zr[3], dot);
    dot = __builtin_fmaf(bf16_lo(pq.z), zr[4], dot);
    dot = __builtin_fmaf(bf16_hi(pq.z), zr[5], dot);
    dot = __builtin_fmaf(bf16_lo(pq.w), zr[6], dot);
    return __builtin_fmaf(bf16_hi(pq.w), zr[7], dot);
}
// Sixteen numerators of a row, times the row's reciprocal, as bf16 into an O tile.
__device__ __forceinline__ void store_scaled(unsigned char *row, const f32x16 &a, float inv)
{
    u32x4 lo4, hi4;
    lo4.x = pack_bf16x2(a[0] * inv, a[1] * inv);
    lo4.y = pack_bf16x2(a[2] * inv, a[3] * inv);
    lo4.z = pack_bf16x2(a[4] * inv, a[5] * inv);
    lo4.w = pack_bf16x2(a[6] * inv, a[7] * inv);
    hi4.x = pack_bf16x2(a[8] * inv, a[9] * inv);
    hi4.y = pack_bf16x2(a[10] * inv, a[11] * inv);
    hi4.z = pack_bf16x2(a[12] * inv, a[13] * inv);
    hi4.w = pack_bf16x2(a[14] * inv, a[15] * inv);
    *reinterpret_cast<u32x4 *>(row) = lo4;
    *reinterpret_cast<u32x4 *>(row + 16) = hi4;
}

// Applies the state panel in `A` (value block wave % (4/NB)) to tile wave / (4/NB) of every step
// of the workgroup's share.  Must be called by all waves of the workgroup.
//
// Denominators phi(Q_i) . z + eps: the wave that loads a row also takes its dot product with z on
// the vector ALU (a lane holds eight features of the row and the matching eight of z, `zr`; 16
// lanes share a row and add up by row permutations: as four shuffles through LDS the sums took 3 to 6 % of the kernel, 18.0 -> 17.4 us for
// 20 heads of 112, 4 680 tokens, 62.7 -> 60.4 at 32 760; without DPP_SUM the shuffles, see apply_mfma_d128) and leaves it in LDS beside the tile.
// The products are exact in fp32, the unrotated phi(Q) is at hand there even with ROPE, and the matrix core is left with the numerator.
template <bool HILO, bool DPP_SUM, int DEPTH, int ROPE, int WAVES, int NB, bool NT>
__device__ __forceinline__ void apply_tiles_coop(CoopApplyStream<DEPTH, ROPE, WAVES, NB, NT> &st, unsigned char *lds,
                                                 int wave, int lane, const ApplyOperands<128, HILO, NB, false> &A,
                                                 const float (&zr)[8], float eps)
{
    constexpr int NS = HILO ? 2 : 1;
    constexpr int STEP = 8 * WAVES * NB, TILES = WAVES * NB / 4, ROWS = STEP / WAVES, NLD = ROWS / 4, WT = 4 / NB;
    const int t = wave / WT, vb = wave % WT;
    const int n = lane & 31, g = lane >> 5;
    unsigned char *bufQ = lds, *bufO = lds + TILES * kCoopTile;
    float *den = reinterpret_cast<float *>(lds + 2 * TILES * kCoopTile);            // [STEP]
    const int my_row = ROWS * wave + (lane >> 4);                                   // + 4 j: the rows this lane loads
    const int wr_off = my_row * kCoopRow + (lane & 15) * 16;
    const unsigned char *brow = bufQ + (32 * t + n) * kCoopRow;
    unsigned char *orow = bufO + (32 * t + n) * kCoopRow + (32 * NB * vb + 16 * NB * g) * 2;

    auto round = [&](int i0) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < DEPTH; ++s) {
            __builtin_amdgcn_sched_barrier(0);   // stages stay in program order
            const bool valid = i0 + s < st.walk.count;
            const uint32_t out_off = st.valid ? st.walk.template offset<STEP>(i0 + s, st.row_bytes) : kOutOfRange;
            if (valid) {
                st.rot.template begin_tile<STEP>(st.walk, i0 + s);
                // the table lookups of the step go out first; ReLU and denominators fill their latency
                f32x2 cs[NLD][4];
#pragma unroll
                for (int j = 0; j < NLD; ++j) st.rot.fetch(s, j, cs[j]);
#pragma unroll
                for (int j = 0; j < NLD; ++j) {
                    const u32x4 pq = relu_bf16x8(st.q[s][j]);                          // phi(Q)
                    float dot = key_sum_products(pq, zr);
                    if (DPP_SUM) dot = row16_sum(dot);                                  // the 16 lanes of the row
                    else
#pragma unroll
                        for (int m = 1; m < 16; m *= 2) dot += __shfl_xor(dot, m);
                    if ((lane & 15) == 0) den[my_row + 4 * j] = dot;
                    *reinterpret_cast<u32x4 *>(bufQ + wr_off + 4 * j * kCoopRow) = st.rot.rotate_with(pq, cs[j]);
                }
            }
            st.request(s, i0 + s + DEPTH);   // refill this stage: DEPTH steps ahead
            __builtin_amdgcn_sched_barrier(0);
            u32x4 o[NLD] = {};
            if (valid) {
                // Q tiles and denominators complete.  They are overwritten in the next round, by waves
                // that have passed the second barrier below, which every wave reaches after its reads.
                lds_barrier();
                f32x16 acc[NB];
#pragma unroll
                for (int i = 0; i < 16; ++i)
#pragma unroll
                    for (int rb = 0; rb < NB; ++rb) acc[rb][i] = 0.f;
                const float inv = 1.0f / (den[32 * t + n] + eps);
#pragma unroll
                for (int ks = 0; ks < 8; ++ks) {
                    const bf16x8 bq = *reinterpret_cast<const bf16x8 *>(brow + (16 * ks + 8 * g) * 2);
#pragma unroll
                    for (int p = NS - 1; p >= 0; --p) {      // small (lo) terms first
#pragma unroll
                        for (int rb = 0; rb < NB; ++rb)
                            acc[rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A.s[p][rb][ks], bq, acc[rb], 0, 0, 0);
                    }
                }
#pragma unroll
                for (int rb = 0; rb < NB; ++rb) store_scaled(orow + 32 * rb, acc[rb], inv);
                // O tiles complete after this barrier; they are overwritten after the first
                // barrier of the next round, which every wave reaches after the reads below.
                lds_barrier();
#pragma unroll
                for (int j = 0; j < NLD; ++j) o[j] = *reinterpret_cast<const u32x4 *>(bufO + wr_off + 4 * j * kCoopRow);
            }
#pragma unroll
            for (int j = 0; j < NLD; ++j)
                store_stream16<NT>(st.rO, out_off + st.lane_off + (uint32_t)j * 4u * st.row_bytes, o[j]);
        }
    };
    // first round apart: the loop is entered in its own steady state of outstanding loads and stores
    if (st.walk.count > 0) round(0);
    for (int i0 = DEPTH; i0 < st.walk.count; i0 += DEPTH) round(i0);
}

// The same for eight waves with NB = 1, two tiles a step, pipelined over two Q and two O tiles of each in LDS, with one barrier per step: between two barriers a
// wave multiplies step i, prepares step i + 1 (ReLU, denominators, rotation) and stores step i - 1, so that vector and matrix
// instructions of one wave can overlap, and a step is one meeting of the waves instead of two.  The tiles are 64 tokens of one head (WAVES = 8, the one-launch block
// step) or 32 tokens each of two heads (WAVES = 4, apply_mfma_d128 with two heads to a workgroup); `wave` counts the workgroup's
// eight.  The stream's rotation is at the first step (begin_tile).
constexpr int kStepTileBytes = 2 * kCoopTile;    // a step's 64 rows
constexpr int step_apply_lds_bytes() { return 4 * kStepTileBytes + 2 * 64 * 4; }
template <int DEPTH, int ROPE, int WAVES, bool NT>
__device__ __forceinline__ void apply_tiles_steps(CoopApplyStream<DEPTH, ROPE, WAVES, 1, NT> &st, unsigned char *lds, int wave, int lane,
                                                  const ApplyOperands<128, true, 1, false> &A, const float (&zr)[8], float eps)
{
    static_assert(DEPTH % 2 == 0, "a stage's tile lies in the same buffer every round");
    constexpr int NLD = 2, STEP = CoopApplyStream<DEPTH, ROPE, WAVES, 1, NT>::STEP;
    const int t = wave >> 2, vb = wave & 3, n = lane & 31, g = lane >> 5;
    const int my_row = 8 * wave + (lane >> 4);                                      // + 4 j: the rows this lane loads and stores
    const int wr_off = my_row * kCoopRow + (lane & 15) * 16;
    const int b_off = (32 * t + n) * kCoopRow + 16 * g, o_off = (32 * t + n) * kCoopRow + (32 * vb + 16 * g) * 2;
    auto q_tile = [&](int p) __attribute__((always_inline)) { return lds + p * kStepTileBytes; };
    auto o_tile = [&](int p) __attribute__((always_inline)) { return lds + (2 + p) * kStepTileBytes; };
    auto dens = [&](int p) __attribute__((always_inline)) { return reinterpret_cast<float *>(lds + 4 * kStepTileBytes) + p * 64; };

    auto prepare = [&](int i, int s) __attribute__((always_inline)) {
        f32x2 cs[NLD][4];
#pragma unroll
        for (int j = 0; j < NLD; ++j) st.rot.fetch(s, j, cs[j]);
#pragma unroll
        for (int j = 0; j < NLD; ++j) {
            const u32x4 pq = relu_bf16x8(st.q[s][j]);                          // phi(Q)
            float dot = key_sum_products(pq, zr);
            dot = row16_sum(dot);
            dens(s & 1)[my_row + 4 * j] = dot;                                 // the same value from the row's sixteen lanes
            *reinterpret_cast<u32x4 *>(q_tile(s & 1) + wr_off + 4 * j * kCoopRow) = st.rot.rotate_with(pq, cs[j]);
        }
    };
    uint32_t out_prev = kOutOfRange;
    auto store = [&](int p) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < NLD; ++j)
            store_stream16<NT>(st.rO, out_prev + st.lane_off + (uint32_t)j * 4u * st.row_bytes,
                               *reinterpret_cast<const u32x4 *>(o_tile(p) + wr_off + 4 * j * kCoopRow));
    };
    if (st.walk.count == 0) return;
    prepare(0, 0);
    lds_barrier();
    for (int i0 = 0; i0 < st.walk.count; i0 += DEPTH) {
#pragma unroll
        for (int s = 0; s < DEPTH; ++s) {
            if (i0 + s >= st.walk.count) break;
            __builtin_amdgcn_sched_barrier(0);
            st.request(s, i0 + s + DEPTH);           // the stage was prepared one step ago
            st.rot.template begin_tile<STEP>(st.walk, i0 + s + 1);     // past the share: zeros
            __builtin_amdgcn_sched_barrier(0);
            const float den = dens(s & 1)[32 * t + n];
            bf16x8 bq[8];
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) bq[ks] = *reinterpret_cast<const bf16x8 *>(q_tile(s & 1) + b_off + 32 * ks);
            f32x16 acc = {};
#pragma unroll
            for (int ks = 0; ks < 8; ++ks)
#pragma unroll
                for (int p = 1; p >= 0; --p)         // small (lo) terms first
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A.s[p][0][ks], bq[ks], acc, 0, 0, 0);
            store((s & 1) ^ 1);
            prepare(i0 + s + 1, (s + 1) % DEPTH);
            const float inv = 1.0f / (den + eps);
            store_scaled(o_tile(s & 1) + o_off, acc, inv);
            out_prev = st.valid ? st.walk.template offset<STEP>(i0 + s, st.row_bytes) : kOutOfRange;
            lds_barrier();
        }
    }
    store((st.walk.count - 1) & 1);
}

// ---- kernels ---------------------------------------------------------------------------------------

// Apply for d = 112 or 128.  grid = (C, B*H), block = 64 * WAVES; workgroup c owns the steps
// c + C*i of the ceil((t1-t0)/STEP) steps of STEP = 8*WAVES*NB tokens (see CoopApplyStream).
// With NB = 1 a wave keeps one 128 x 32 panel of S and fits in half a SIMD's registers: two
// workgroups (eight waves) share a compute unit, and while one wave waits at a barrier or works on
// the vector ALU (ReLU, rotation, scaling) the other wave of its SIMD feeds the matrix core.
//
// HEADS = 2, where neighbouring heads share cache lines (224-byte rows side by side): grid = (C, B*H / 2), block = 128 * WAVES, the first
// half of the waves on head 2 y, the other on 2 y + 1.  As workgroups of their own the two drift apart within a few tiles; here
// each tile's barriers hold them together, so that a line is read twice by one compute unit and its two parts are written at nearly the
// same time.  Apply, 40 heads of 112, 32 760 tokens: 149 -> 119 us (586 MB, 4.9 TB/s), factored tables 176 -> 150, full table 175 -> 168.
// One head to a workgroup (odd H, see pairs_heads): the slower sums by shuffles, whose pace keeps the heads more in step
// (state and apply 271 us, with row permutations 288 to 302; factored tables 293 and 306).
// Three workgroups to a compute unit leave a wave 168 registers; with factored tables the compiler takes 177 if it may.
template <bool HILO, int DEPTH, int ROPE, int WAVES, int NB, bool NT, int HEADS, bool STEPS>
__global__ __launch_bounds__(64 * WAVES * HEADS, NB != 1 ? 1 : ROPE == kRope3D && HEADS == 1 ? 3 : 2) void apply_mfma_d128(
    const uint16_t *__restrict__ Q, uint16_t *__restrict__ O, RopeArg rope, TokStrides st, int H,
    int d, int t0, int t1, int C, const float *__restrict__ S, const float *__restrict__ z, float eps, int order)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1), wg_wave = __builtin_amdgcn_readfirstlane(tid >> 6), wave = wg_wave % WAVES, half = wg_wave / WAVES;
    const WgRole role(C, order);
    const int c = role.c, bh = HEADS * role.bh + half;
    const int b = bh / H, h = bh % H;
    const uint16_t *Qh = Q + b * st.b + h * st.h;
    uint16_t *Oh = O + b * st.b + h * st.h;
    constexpr int STEP = 8 * WAVES * NB;
    constexpr int kTiles = coop_apply_lds_bytes<WAVES, NB>(), kTabs = STEPS ? step_apply_lds_bytes() : HEADS * kTiles;
    const int n_steps = (t1 - t0 + STEP - 1) / STEP;

    CoopApplyStream<DEPTH, ROPE, WAVES, NB, NT> stream(Qh, Oh, rope, lds + kTabs, st.n, t1, d,
                                                    wave, lane, TileWalk(t0, c, C, n_steps, role.phase(b, order)));
    Rope3dFill tabs;
    if (ROPE == kRope3D) rope3d_lds_fill_begin(rope.r3, tabs);   // the first loads of the kernel
    coop_apply_prefetch<0, DEPTH>(stream);   // in flight while S is fetched
    if (ROPE == kRope3D) {
        rope3d_lds_fill_end(lds + kTabs, rope.r3, tabs);
        wg_barrier();
    }
    ApplyOperands<128, HILO, NB, false> A;
    A.template load<false>(S + (size_t)bh * d * d, z + (size_t)bh * d, d, wave % (4 / NB), lane);
    float zr[8];                                   // the key sums of the eight features this lane loads of a row
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int k = 8 * (lane & 15) + e;
        const float x = z[(size_t)bh * d + (k < d ? k : 0)];   // loaded by every lane: a load under a condition is a branch
        zr[e] = k < d ? x : 0.f;
    }
    if constexpr (STEPS) {
        stream.rot.template begin_tile<STEP>(stream.walk, 0);
        apply_tiles_steps(stream, lds, wg_wave, lane, A, zr, eps);
        return;
    }
    apply_tiles_coop<HILO, NT || HEADS == 2>(stream, lds + half * kTiles, wave, lane, A, zr, eps);
}

}  // namespace sv
