// What a token tensor's strides mean for the kernels: whether 32-bit offsets reach its heads, and in which order workgroups
// are dealt to it.  Plain C++ (no device code), shared by the launcher and a host-side test.
#pragma once

#include <stdint.h>

namespace sv {

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

}  // namespace sv
