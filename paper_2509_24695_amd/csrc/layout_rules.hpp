// What a call's sizes and a token tensor's strides mean for the kernels: whether 32-bit offsets reach its heads, in which order workgroups
// are dealt to it, how many it gets and which kernel serves it.  Plain C++ (no device code), shared by the launcher and host-side tests.
#pragma once

#include <stdint.h>

#include "tile_walk.hpp"

namespace sv {

constexpr int kMaxChunks = 32;       // upper bound on token chunks per head (workspace sizing)

// Token chunks (workgroups) per head: about one workgroup per compute unit over
// the whole grid, never more than kMaxChunks (which sizes the workspace) or
// than there are tiles.
inline int plan_chunks(int BH, int n_tokens, int tokens_per_wg_step, int num_cu)
{
    if (n_tokens <= 0) return 0;
    const int steps = (n_tokens + tokens_per_wg_step - 1) / tokens_per_wg_step;
    int chunks = num_cu / BH;
    if (chunks > kMaxChunks) chunks = kMaxChunks;
    if (chunks > steps) chunks = steps;
    if (chunks < 1) chunks = 1;
    return chunks;
}

// The matrix-core kernels address a head's tokens with 32-bit byte offsets below 2^31: what a head spans, and what one tile of 64 rows
// spans (rows past the end are reached by address before they are dropped).
inline bool head_offsets_fit(int64_t N, int64_t stride_n, int elem_bytes)
{
    constexpr int64_t kLimit = int64_t(1) << 31;
    const int64_t rows = N > 64 ? N : 64;
    return stride_n <= (kLimit - 1) / (rows * elem_bytes);   // rows * stride_n * elem_bytes < kLimit, without overflow
}

// How a grid's workgroups are dealt to (chunk, head) and the heads' walks staggered (kernel argument `order`):
constexpr int kOrderChunkMajor = 1;   // chunk_major_role instead of (blockIdx.x, blockIdx.y)
constexpr int kOrderLockstep = 2;     // all heads of a batch walk in phase: they read pieces of the same rows

// A token tensor as the rules below see it; strides in elements.
struct TokenLayout {
    int BH, H, d, elem_bytes;
    int64_t stride_h, stride_n;
    // Token rows of all heads side by side: [B][N][H][d], what a projection leaves behind.
    bool token_major() const { return H > 1 && stride_h < stride_n; }
    // ... and neighbouring heads have pieces of the same 128-byte cache lines (d = 112: 224-byte pieces)?  Then the bf16 kernels
    // go without the non-temporal hint, which makes a head's pieces of a line leave the L2 before the neighbour's accesses: the
    // apply kernel alone 64 against 104 us (32 760 tokens, 20 heads), both kernels 158 against 174.
    bool shares_lines() const { return token_major() && (stride_h * elem_bytes) % 128 != 0; }
    // 256-byte granules of memory hold pieces of several heads?
    bool shares_granules() const { return token_major() && (stride_h * elem_bytes) % 256 != 0; }
};

// Token-major tensors: all heads of a batch walk in phase, so that together they read whole runs of consecutive rows
// (bf16, state and apply, against staggered walks: 1.00-0.90 for every number of heads from 2 to 128).
//
// The heads of a chunk on one die as well:
//   d != 64, shared granules   both kernels (40 heads of 112, 32 760 tokens, rotated, layer: 290 us, 319 in phase only).
//   d = 64, state              up to 12 heads in all (2 heads, 4 680 tokens 9.7 against 10.2 us; 12 with a full table 0.92 against 0.98
//                              of the staggered time); with more it costs up to 9 % (8 x 16 heads, 32 760 tokens: 214 against 196 us).
//   d = 64, apply, full table  always: the heads share the chunk's table rows (level to 0.95).
//   d = 64, apply, plain       rows of 32 heads, 4 KB and its multiples, and long ranges, where walking in phase alone is slow:
//                              32 heads, 20 000 tokens 40.6 against 45.5 us, 32 760 tokens 59.0 against 77.8; level at 12 480;
//                              9 360 tokens 28.3 against 25.6.  With 128 heads and more it is level or loses (128 heads, 20 000
//                              tokens: 202 against 148), with any other number of heads it loses (2 x 5 heads, 32 760 tokens: 29.0 against 23.6;
//                              20, 14 040: 25.9 against 22.6; 40, 14 040: 42.2 against 36.1).
//   d = 64, apply, factored    never (level to 1.23).
// d = 112 and 128 with a full table, any layout, state: always; die c's L2 then serves the heads their chunk's table rows (20 heads of 112,
// 32 760 tokens, layer: 142.9 against 145.5 us; d = 64, with half the table per token, 500 against 482).
inline int state_order(const TokenLayout &t, bool full_table)
{
    int order = 0;
    if (t.token_major()) {
        order = kOrderLockstep;
        const bool d64 = t.d == 64 && t.elem_bytes == 2;
        if (t.shares_granules() && (!d64 || t.BH <= 12)) order |= kOrderChunkMajor;
    }
    if (full_table && t.d > 64 && t.elem_bytes == 2) order |= kOrderChunkMajor;
    return order;
}
inline int apply_order(const TokenLayout &t, bool full_table, bool factored_tables, int n_tokens)
{
    if (!t.token_major()) return 0;
    if (!t.shares_granules()) return kOrderLockstep;
    const bool d64 = t.d == 64 && t.elem_bytes == 2;
    const bool runs_of_32 = !factored_tables && t.H % 32 == 0 && t.BH < 128 && n_tokens >= 12288;
    return !d64 || full_table || runs_of_32 ? kOrderLockstep | kOrderChunkMajor : kOrderLockstep;
}

// d = 112 and 128, apply without a full table: workgroups per compute unit, three or two (layers, state and apply in turn, three -> two).
//   shared lines, plain    two, also where they go in pairs (pairs_heads): the heads of a chunk, which read and write pieces of the same lines, stay closer together (20 heads of 112, 32 760
//                          tokens 155 -> 150 us, 40 heads 312 -> 266, 64 heads, 14 040 tokens 228 -> 195; with factored tables 299 -> 286 on
//                          one device and 286 -> 290 on another, so not there).
//   d = 128, plain         two (64 heads, 14 040 tokens 190 -> 187 us, token-major 40 heads, 32 760 tokens 258 -> 249, 20 heads 140 -> 137; at
//                          d = 112 level, with a rotation up to 9 % more).
//   a poor fit             two, where three would leave a tenth of the places empty, that is some compute units with a third less work to share
//                          (160 heads of 128, 1 560 tokens 68.0 -> 65.8 us, 4 680 tokens 170.6 -> 160.3; of 112 62.4 -> 58.2, 143.7 -> 139.1).
inline int wide_apply_wgs_per_cu(const TokenLayout &t, bool rotated, int num_cu)
{
    if (!rotated && (t.shares_lines() || t.d == 128)) return 2;
    const int c3 = 3 * num_cu / t.BH, c2 = 2 * num_cu / t.BH;
    return 10 * c3 * t.BH < 27 * num_cu && 3 * c2 > 2 * c3 ? 2 : 3;
}

// d = 112, shared lines, apply: two neighbouring heads to a workgroup (apply_mfma_d128, HEADS = 2), of which one fits on a compute unit.  State +
// apply, one / two heads to a workgroup:
//   plain            20 heads, 4 680 tokens 37.8 / 37.1, 14 040 71.2 / 68.6, 32 760 149 / 140; 40 heads, 9 360 88.6 / 85.6, 32 760 274 / 253;
//                    160 heads, 6 240 238 / 219
//   rotated          with one barrier per step from 65 536 head-tokens on, below it is level.  Layers: factored tables 20 heads, 4 680 tokens 35.9 / 35.3, 9 360 74.4 / 70.2, 80 heads, 4 680 tokens 99.1 / 93.8, 160 heads, 1 560 75.0 / 71.9; full table 20
//                    heads, 9 360 63.3 / 62.1, 17 160 100.5 / 95.6, 32 760 173 / 165, 160 heads, 1 560 84.7 / 81.5
inline bool pairs_heads(const TokenLayout &t, bool rotated, int n_tokens)
{
    return t.shares_lines() && t.H % 2 == 0 && (!rotated || (int64_t)t.BH * n_tokens >= 1 << 16);
}
// ... their steps with one barrier instead of two (apply_tiles_steps): rotated calls always, 5 to 6 % less (40 heads, 32 760 tokens, factored tables 284 / 269 us, full
// table 324 / 307; 16 heads, 75 600, factored 258 / 249); plain ones (252 / 241) unless the token rows are multiples of 1 KB (32 heads: 7 KB), where it costs
// 2 to 5 %: 64 heads, 32 760 tokens 405 / 427, 14 040 189 / 193, 32 heads, 32 760 214 / 220.
inline bool pipelines_plain_pairs(const TokenLayout &t) { return t.stride_n * t.elem_bytes % 1024 != 0; }

// d = 112 and 128 without a full table, state: shared tiles (coop_state.hpp) instead of a state in every wave (wide_state.hpp) up to 2 048
// tokens per workgroup: there the end, which the sum over the waves makes longer, counts.  State + apply, us, a state per wave / shared tiles:
//   360 to 1 560 tokens each  20 heads of 112, 4 680: 32.5 / 30.3, factored tables 37.3 / 35.5; 20 heads of 128, 14 040, factored tables 72.4 / 70.1;
//                             64 heads of 112, 6 240, factored tables 87.2 / 84.2; 256 heads, 1 560: 85.1 / 79.6, factored tables 91.7 / 87.8
//   5 070 to 6 300            plain 64 heads, 20 280: 245 / 242, 160 heads, 6 240: 174 / 187; factored tables 20 heads, 75 600: 271 / 291,
//                             40 heads, 32 760: 239 / 260, 160 heads, 6 240: 206 / 225
// With a full table nothing is gained: 20 heads of 112, 9 360, 14 040 and 20 280 tokens 57.8 / 55.9, 75.1 / 75.3, 99.8 / 101.0; of 128 60.8 / 61.1,
// 81.7 / 82.7, 110.1 / 108.6.
// Shared lines, where the apply takes heads in pairs: always, the state alone gains little at full length, the two together 2 to 4 %
// (40 heads, 32 760 tokens 263 -> 253, factored tables 294 -> 283; 160 heads, 6 240 tokens 225 -> 219).
inline bool coop_state_pays(int n_tokens, int C) { return n_tokens <= 2048 * C; }

// d = 112 and 128, state: the kernel of quadrants (quad_state.hpp) instead of whole rows, for ranges whose exchange among workgroups takes
// longer than their tokens.  Both read in step with the number of head-tokens, the quadrants slower, and what the quadrants save depends on how
// many chunks C a head has: all of the exchange with one, little with two, whose quadrants fetch as many partials as twice as many workgroups
// of whole rows.  The lines, in thousands of head-tokens, are where layers (state, apply) on one kernel and on the other meet; quadrants over rows:
//   d = 112, plain      C = 1: 64 heads 0.93 to 61, 0.96 at 76, 48 heads 1.00 at 69; C = 2: 1.00 at 20, 1.02 at 30, 1.05 at 40; C = 3: 0.97 at 20, 0.99
//                       at 30, 1.00 to 1.01 from 40 to 60, 1.03 at 70; C = 4 to 10: 0.95 to 0.99 at 60, 0.99 to 1.02 at 70; 4 and 5 heads: 1.01 to 1.08
//                       from 40 on; 2 heads: 0.93 to 0.98
//   d = 112, factored   C = 1: 0.94 to 1.01 at 70; C = 2: 0.98 at 20, 0.99 at 30, 1.00 at 40, 1.03 at 60; C = 3: 0.98 at 50, 1.00 at 60 and 70, 1.02 at 80;
//                       from 4 on: 0.96 to 1.00 at 70, 0.94 to 1.01 at 79
//   d = 112, full table 24 heads 0.99, others 0.86 to 0.96 at 40
//   d = 128, plain      0.91 to 1.00 at 100
//   d = 128, factored   C = 1: 0.95 to 1.01 at 99; C = 2: 0.99 at 70, 1.00 at 80, 1.01 at 90 (24 heads 1.03); C = 3: 0.99 at 80 to 100; from 4 on: 0.93 to
//                       0.99 at 99
//   d = 128, full table 0.84 to 0.97 at 68
// (C = 2 and 3: averages over 17 to 32 heads and both layouts, four devices, single calls up to 4 % to either side.)
// Four workgroups per chunk have to fill most of the device (40 heads of 112, 1 560 tokens, 160 workgroups: 15.5 / 13.5 us).
inline bool quad_state_pays(int BH, int d, int n_tokens, bool full_table, bool factored_tables, int num_cu)
{
    const int C = num_cu / (4 * BH);
    if (16 * BH * C < 3 * num_cu) return false;
    constexpr int kThousands[2][3][4] = {{{76, 22, 60, 70}, {76, 38, 70, 76}, {40, 40, 40, 40}},            // d = 112: plain, factored, full table
                                         {{100, 100, 100, 100}, {100, 80, 100, 100}, {66, 66, 66, 66}}};    // d = 128
    if (d == 112 && !full_table && !factored_tables && C > 10 && BH >= 4) return false;
    return (int64_t)BH * n_tokens <= 1000 * kThousands[d == 128][full_table ? 2 : factored_tables ? 1 : 0][C < 4 ? C - 1 : 3];
}

// Chunks per head of a call on the kernel of quadrants, 0: whole rows serve it.
constexpr int kQuadMaxChunks = 16;                            // flags: [quadrant][chunk] in the head's 2 x kMaxChunks words
constexpr int quad_wg_tokens(bool rotated) { return 8 * (rotated ? 16 : 32); }   // a round of a workgroup's waves
inline int quad_state_chunks(int BH, int d, int n_tokens, bool full_table, bool factored_tables, int num_cu)
{
    if (!quad_state_pays(BH, d, n_tokens, full_table, factored_tables, num_cu)) return 0;
    const int round = quad_wg_tokens(full_table || factored_tables), steps = (n_tokens + round - 1) / round, C = num_cu / (4 * BH);
    const int most = steps < kQuadMaxChunks ? steps : kQuadMaxChunks;
    return C < most ? C : most;
}
// Whole rows, C chunks per head: shared tiles instead of a state in every wave?
inline bool coop_state_serves(const TokenLayout &t, int n_tokens, int C, bool full_table, bool factored_tables)
{
    return !full_table && (coop_state_pays(n_tokens, C) || pairs_heads(t, factored_tables, n_tokens));
}
constexpr int kWideWgTokens = 64;                             // of whole rows: tokens of a workgroup's step

// fp32-arithmetic state: tokens up to which one workgroup sums a head in one launch, instead of several and a second launch for
// their sum.  The lines lie where a host that enqueues layers (state, apply) back to back sees the two meet; one / several, us, two devices:
//   d = 32 (sixteen waves), fp32, plain   2 heads, 1 024 tokens 1.2 less, 1 152 0.5 less, 1 280 0.1 more; 16 heads, 768 1.1 less, 896 0.7 less, 1 024 0.6
//            more, 1 152 1.7 more; 6 and 12 heads 832 0.3 more; 32 heads, 640 0.6 less, 768 0.1 more, 896 1.2 more; 64 heads, 640 0.9 less; 128, 768 2.3 less;
//            rotated   2 heads, 768 0.9 less to 0.2 more; 16, 640 0.6 less to 0.6 more, 1 024 3.4 to 3.8 more; 32, 512 0.2 less to 0.3 more, 896 2.7 more;
//            bf16, plain   16 heads, 1 152 0.5 more, 1 280 1.2 more; rotated   16, 896 0.2 more to 1.1 less, 1 280 2.3 to 4.0 more; 32, 704 level; 64, 640 level;
//   d = 64   8 heads, 192 tokens 0.7 less, 256 0.6 more; 12 heads, 256 0.3 less; rotated 16 heads, 192 0.7 more, 256 1.7 more; 64 heads, 192 1.2 less.
// of 12 to 18 us a layer.  In a captured graph, where a launch costs no host time, they meet earlier: d = 32, fp32 at 512 tokens for up to
// 32 heads, 1 152 tokens are 3 to 5 us slower there on one workgroup; d = 64 at 160.
// Both forms of the rotation have the same lines, so that they give the same bits.
// d = 112 and 128 end at 48 tokens, of which no running sum takes more than 16 (two groups of waves, tiles of 8, two sums each): a longer one is further from the exact sum than those of
// several workgroups (64 heads of 112, 128 tokens: S 9.4e-8 against 7.3e-8), although with many heads it would be the faster one up to 128 tokens
// (8 heads, 64 tokens 16.0 / 16.7 us, 128 heads, 64 tokens 24 / 32, 128 tokens 31 / 36).  Adding the sums to a total after every round of tiles
// would keep them short, but neither in registers nor in LDS does the compiler get by without spilling.
constexpr int kF32WideSoleTokens = 48, kF32WideSumTokens = 16;
inline int f32_sole_tokens(int d, int BH, int elem_bytes, bool rotated)
{
    if (d > 64) return kF32WideSoleTokens;
    if (d == 64) return BH <= 16 && !rotated ? 256 : 192;
    constexpr int kTokens[2][2][5] = {{{1152, 832, 640, 640, 768}, {832, 640, 512, 512, 768}},         // fp32: plain, rotated
                                      {{1280, 1152, 1024, 896, 896}, {960, 896, 704, 640, 896}}};      // bf16
    return kTokens[elem_bytes == 2][rotated][BH <= 2 ? 0 : BH <= 16 ? 1 : BH <= 32 ? 2 : BH <= 64 ? 3 : 4];
}

// fp32 arithmetic, state of a head that C workgroups share: the last of them adds the partial states up (LastFold) instead of a second launch.  One
// compute unit then reads C partials, which costs what the launch did at 130 KB.  Layers, us, second launch / last workgroup: d = 32
// (4 KB each), bf16 128 heads, 4 096 tokens, C = 2 34.6 / 33.4, 32 heads, C = 8 16.9 / 16.2, 20 heads, 1 560 tokens, C = 12 11.6 / 11.0; fp32 32 heads, 4 680 tokens 26.5 / 25.9;
// C = 32 15.5 / 15.8; d = 64 (17 KB), 64 heads, 2 000 tokens, C = 4 39.8 / 38.7, 32 heads, 4 680, C = 8 44.3 / 44.3, 16 heads, 1 560, C = 16 20.1 / 21.5.
// Where few heads share little more than f32_sole_tokens the kernels alone are as long either way or the launch a little shorter, but a host that enqueues call by call is what
// paces such a layer, and a launch costs it more.  d = 64, rotated, from the host / in a captured graph: 1 head, 240 tokens 16.1 / 13.3 with the launch, 14.9 / 14.1 with the last workgroup, 8, 220
// 16.0 / 13.7 and 15.2 / 14.4, 20, 200 16.3 / 14.7 and 15.6 / 15.3, 32, 256 17.0 / 16.1 and 16.1 / 16.0; plain, 16, 260 16.0 / 13.1 and 15.3 / 13.1.  (From a faster host 1 head 13.9 and 14.7, 48, 200 16.6
// and 16.4.  d = 32, up to 16 heads: in a graph 1 to 3 % longer, from the host up to 13 % shorter.)
inline bool f32_last_folds(int d, int C) { return d == 32 ? C <= 16 : d == 64 && C <= 4; }

// d = 112 and 128, block step: one launch (block_step_wide.hpp) or two (a state kernel, the apply kernel).  Streams of three look-ahead passes and a
// committing one, us per block, two launches / one:
//   plain           20 heads of 112, 4 680 tokens 32.9 / 29.0, 32 760 114 / 104, 98 280 309 / 294; 64 heads, 32 760 333 / 311; 8 heads, 131 040 178 / 158; of
//                   128: 20 heads, 9 360 50 / 46, 98 280 354 / 332; 64 heads, 32 760 394 / 395; 9 to 15 heads, whose worst-off have ten workgroups, 1 040 tokens 0.90 to
//                   0.98 of two launches', 1 560 0.95 to 1.07, 3 120 0.96 to 1.05, 4 680 0.93 to 1.02, 5 460 0.93 to 0.99
//   factored        20 heads, 4 680 37.7 / 32.1, 49 920 175 / 162, 98 280 341 / 346; 16 heads, 65 520 186 / 181; 68 heads, 10 920 147 / 146, 12 480 160 / 161
//   two workgroups  of 128, plain: 128 heads, 9 360 243 / 225, 16 380 396 / 370, 100 heads, 9 360 189 / 184, 16 380 306 / 301, 87 heads, 9 360 168 / 167, 12 480 223 / 217,
//   per head        15 600 266 / 271.  (Of 112 and with factored tables the line could lie further out: 128 heads, 4 680 111 / 98, factored 119 / 112, 7 800
//                   196 / 175; 87 heads, factored, 7 800 154 / 149, 9 360 163 / 168.)
//   full table      20 heads, 4 680 38.6 / 35.9, 9 360 53 / 52; 64 heads, 3 000 55 / 53; 100 heads of 128, 2 048 69 / 66; few heads of 128, all spread: 8, 4 680
//                   26.4 / 30.0, 6 240 28.9 / 32.6, 7 800 33.0 / 32.9, 10, 3 120 24.7 / 27.5, 15, 3 120 27.6 / 29.0, 4 680 39.0 / 35.2; 16, 2 070 25.5 / 27.5, 3 120 30.3 / 31.7, 3 780 33.9 / 32.5; 18, 2 756
//                   30.4 / 31.9, 3 120 33.2 / 32.5; 20, 2 340 28.6 / 30.6, 2 756 32.5 / 31.1; 22, 2 070 32.9 / 28.3
//   shared lines    plain 20 heads, 4 680 36 / 34, 7 800 45.5 / 45.8, 9 360 52 / 53, 40 heads, 3 120 42 / 41, 4 680 52 / 53, 16 heads, 9 360 44.7 / 44.7; factored tables 40 heads,
//                   4 680 58 / 56, 20 heads, 9 360 58 / 56
//   few heads       a head on all dies.  Of 112: 5 heads, 2 028 tokens 19.7 / 18.0, 6, 1 560 18.1 / 17.9, 2 028 18.4 / 18.7, 7, 1 560 18.2 / 19.0, factored tables 20.8 / 21.1, full
//                   table, 2 028 20.4 / 20.4, shared lines 19.2 / 19.2.  Of 128: 3 heads, 1 560 16.2 / 16.1, 2 028 16.5 / 17.4, 5, 1 040 16.3 / 15.8, 1 560 16.9 / 17.9, factored tables
//                   20.0 / 20.1, 7, 1 040 19.6 / 19.7, full table 18.9 / 18.9, 5, 2 028 20.9 / 20.6
// A workgroup per head, by how much of the device the heads fill:
//   plain           130 of 112: 2 560 75 / 72; 146: 3 900 113 / 107, 4 680 123 / 126; 160: 4 680 129 / 129; 192: 14 040 433 / 427, 18 720 563 / 559, 32 760 994 / 1 026; 200:
//                   32 760 1 102 / 1 038; of 128, 130: 4 680 137 / 136; 192: 32 760 1 189 / 1 144; 256: 18 720 and 32 760 of 112 754 / 739 and 1 309 / 1 282, of 128 14 040 671 / 629,
//                   32 760 1 551 / 1 585
//   factored        130: 1 248 53 / 52, 1 560 61 / 62; 150: 1 560 62 / 62, 2 560 91 / 93; 160: 2 560 94 / 94, 3 120 109 / 112; 180: 3 120 117 / 114; 192: 3 900 155 / 150
//   full table      130: 780 45 / 44; 160: 600 40 / 36; 185: 780 52 / 45
//   more heads      than compute units: a second round, nearly empty at first, which the state kernel of two launches has too, its apply not.  257 of 112: 1 560
//                   148 / 110, 4 680 310 / 288, 7 800 473 / 474, 9 360 551 / 559, 18 720 1 050 / 1 109; 320: 9 360 591 / 569, 18 720 1 107 / 1 128; 350: 14 040 889 / 878, 18 720
//                   1 155 / 1 151; 400: 18 720 1 278 / 1 192; factored tables 257: 4 680 342 / 338, 5 460 396 / 397, 9 360 624 / 660; 350: 9 360 691 / 688, 10 920 790 / 791; 400:
//                   9 360 794 / 731; full table 257: 1 560 184 / 146; shared lines 257: 960 129 / 83; of 128 the lines lie further out: 257: 9 360 625 / 623
//   shared lines    160 heads, 600 76 / 69, 4 680 334 / 398 (factored 376 / 411)
inline bool wide_step_serves(const TokenLayout &t, int n_tokens, int C, bool full_table, bool factored_tables, int num_cu)
{
    const int64_t head_tokens = (int64_t)t.BH * n_tokens;
    const bool plain = !full_table && !factored_tables;
    if (C > 1) {
        if (t.BH < 8) {
            if (t.d == 112) return n_tokens <= 2048 && (full_table || t.shares_lines() || head_tokens <= 10240);
            return n_tokens <= 2048 && head_tokens <= (plain ? 5200 : factored_tables ? 8192 : 10240);
        }
        if (full_table && t.d == 128 && n_tokens > 2048 && (t.BH < 16 ? n_tokens < 7000 : t.BH <= 20 && head_tokens < 54000)) return false;
        if (full_table || t.shares_lines()) return head_tokens <= (plain ? 150000 : 200000);
        if (plain && t.d == 128 && t.BH > 8 && t.BH < 16 && n_tokens > 1250 && n_tokens < 5000) return false;
        if (C == 2 && (t.d == 112 || factored_tables)) return n_tokens <= 3072;
        if (C == 2 && 4 * C * t.BH < 3 * num_cu) return n_tokens <= 12288;
        return n_tokens <= (factored_tables ? 4096 : 8192) * C;
    }
    if (t.shares_lines()) return n_tokens <= 1024;
    const int fill = 100 * t.BH / num_cu;
    if (t.BH > num_cu) return n_tokens <= (full_table ? 2048 : fill <= 125 ? (factored_tables ? 5120 : 8192) : factored_tables ? 10240 : 18720);
    if (full_table) return n_tokens <= 768;
    if (factored_tables) return n_tokens <= (fill < 60 ? 1280 : fill < 70 ? 2560 : fill < 75 ? 3120 : 4096);
    if (fill < 57 && t.d == 112) return n_tokens <= 2560;
    if (fill < 75) return n_tokens <= (fill < 60 && t.d == 112 ? 4096 : 4680);
    return n_tokens <= (fill < 78 ? 18720 : 32760);
}

// ... its workgroups: as many heads as fill the dies evenly live on one die each, where its workgroups exchange their sums through that die's L2, the
// others are spread over all dies; of the splits of a die's compute units between the two, the one whose worst-off head has the most
// workgroups, a spread head counted for eight tenths: its exchange takes 2 to 3 us longer.  (20 heads, 4 680 tokens, plain and factored tables, all spread: 32.0
// and 38.0 us a block; 16 local heads of 13 workgroups and 4 spread of 12: 28.8 and 34.3, of 12 and 16: 27.8 and 33.0.)  Not where heads share cache lines,
// which then lie on different dies; with a full table, whose rows every die fetches then, up to 2 048 tokens (20 heads, 1 560 tokens 74.8 -> 69.5
// us per stream, 4 680 level, 18 000 258 -> 291).
// `flags_at`: address of the workspace's flags (see wide_flag_word; 9 heads of 112, the only ones with more than 24 workgroups beside spread heads, lose none
// to it where the workspace starts a line).
inline WideRoles wide_roles(const TokenLayout &t, int n_tokens, int n_steps, bool full_table, int num_cu, int dies, uint64_t flags_at = 0)
{
    WideRoles best{0, 0, 0, 0, t.BH};
    if (dies <= 0 || t.BH < dies || t.BH * 2 > num_cu || t.shares_lines() || (full_table && n_tokens > 2048)) return best;
    const int cus = num_cu / dies, per_die = t.BH / dies, spread = t.BH % dies, most = n_steps < kMaxChunks ? n_steps : kMaxChunks;
    const int beside = spread ? wide_most_beside_spread((int)(flags_at % 128), kMaxChunks) : kMaxChunks, most_local = most < beside ? most : beside;
    int worst = 0;
    for (int C = cus / per_die < most_local ? cus / per_die : most_local; C >= 1; --C) {
        int Cs = spread ? dies * (cus - per_die * C) / spread : C;
        Cs = Cs < most ? Cs : most;
        const int score = 10 * C < 8 * Cs || !spread ? 10 * C : 8 * Cs;
        if (score <= worst) continue;
        worst = score;
        best = WideRoles{dies, per_die, C, Cs, t.BH};
    }
    return best;
}

}  // namespace sv
