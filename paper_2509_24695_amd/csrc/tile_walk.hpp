// Which token tiles a wave visits, and in which order.  Plain C++ (no device code): shared by the
// kernels and a host-side coverage test.
#pragma once

#include <stdint.h>

#ifndef SV_HOST_DEVICE
#if defined(__HIPCC__)
#define SV_HOST_DEVICE __host__ __device__
#else
#define SV_HOST_DEVICE
#endif
#endif

namespace sv {

constexpr uint32_t kOutOfRange = 0x80000000u;   // a byte offset no buffer resource built by the kernels covers

// Byte offset of the first row of the tile that starts at token `tok0`, or kOutOfRange.
SV_HOST_DEVICE inline uint32_t tile_offset(bool valid, int tok0, uint32_t row_bytes) {
    return valid ? (uint32_t)tok0 * row_bytes : kOutOfRange;
}

// A wave's share of the tiles that cover the token range [t0, t1): tiles
// first + j*step for j = 0 .. count-1 (all values wave-uniform), visited in the
// cyclic order j = rot, rot+1, .., count-1, 0, .., rot-1.  Heads start at
// different phases of their shares, head bh at (bh mod 16)/16: when all heads
// march through memory in lockstep, some sequence lengths put their streams on
// the same DRAM resources at the same time (N = 75 600, 64 heads: apply 290 us
// in lockstep, 246 us staggered; no length measured got slower).
struct TileWalk {
    int t0, first, step, count, rot;
    SV_HOST_DEVICE inline TileWalk(int t0_, int first_, int step_, int n_tiles, int bh)
        : t0(t0_), first(first_), step(step_),
          count(first_ < n_tiles ? (n_tiles - first_ + step_ - 1) / step_ : 0), rot(((bh & 15) * count) >> 4) {}
    // first token of the i-th tile the wave visits (TILE tokens per tile), i < count
    template <int TILE> SV_HOST_DEVICE inline int token(int i) const {
        int j = i + rot;
        j = j >= count ? j - count : j;
        return t0 + (first + j * step) * TILE;
    }
    // its byte offset for rows of row_bytes bytes, kOutOfRange past the share
    template <int TILE> SV_HOST_DEVICE inline uint32_t offset(int i, uint32_t row_bytes) const {
        return tile_offset(i < count, token<TILE>(i), row_bytes);
    }
};

// Slice c of a head's state when C workgroups fold it together: 8-byte units [lo, hi) of the
// d*d/2 + d/2 units that S (d x d floats) and z (d floats) make, per = ceil(units / C) each; late
// slices may be short or empty.
struct StateSlice {
    int s_units, units, lo, hi;
    SV_HOST_DEVICE inline StateSlice(int c, int C, int d) : s_units(d * d / 2), units(d * d / 2 + d / 2), lo(0), hi(0)
    {
        const int per = (units + C - 1) / C;
        lo = c * per < units ? c * per : units;
        hi = lo + per < units ? lo + per : units;
    }
};

// The share of the token tiles that workgroup c of head bh takes in the one-launch block step:
// dealt from a different start in each head (see block_step_mfma).
SV_HOST_DEVICE inline int block_step_share(int c, int bh, int C) { return (c + bh) % C; }

// Which (chunk, head) workgroup `id` of a grid of C chunks x BH heads works on in the chunk-major order: the
// grid's ids go round the `dies` dies one by one, and die e takes the e-th part of the list (chunk 0 of all
// heads, chunk 1 of all heads, ...).  So the heads of one chunk, which read the same rows of a rotation table and,
// in a [B][N][H][d] tensor, neighbouring pieces of the same cache lines, share a die's L2.
SV_HOST_DEVICE inline void chunk_major_role(int id, int C, int BH, int dies, int &c, int &bh)
{
    const int total = C * BH, e = id % dies, left = total % dies;
    const int logical = e * (total / dies) + (e < left ? e : left) + id / dies;
    c = logical / BH;
    bh = logical - c * BH;
}

// Which chunk, head and quadrant of the state workgroup `id` of the quadrant kernel works on: the four quadrants of one (chunk, head), which
// read the same rows, run on one die.  Die e takes groups e, e + dies, ... of the list (head by head, chunk by chunk) or, in the
// chunk-major order, the e-th part of the chunk-major list.  False: the id has no work (the grid is rounded up to whole
// groups on every die).
SV_HOST_DEVICE inline bool quad_role(int id, int C, int BH, int dies, bool chunk_major, int &c, int &bh, int &q)
{
    const int slot = id / dies, group = (slot / 4) * dies + id % dies;
    q = slot & 3;
    if (group >= C * BH) return false;
    if (chunk_major) {
        chunk_major_role(group, C, BH, dies, c, bh);
    } else {
        bh = group / C;
        c = group - bh * C;
    }
    return true;
}
SV_HOST_DEVICE inline int quad_grid(int C, int BH, int dies) { return 4 * dies * ((C * BH + dies - 1) / dies); }

// How the one-launch block step of d = 112 and 128 is dealt to the dies: heads 0 .. dies * per_die - 1 live on one die each, C_local workgroups,
// the others are spread over all of them, C_spread workgroups.  dies = 0: every head is spread, by a grid of (C, BH).
struct WideRoles {
    int dies, per_die, C_local, C_spread, BH;
    SV_HOST_DEVICE inline int grid() const {
        return dies * (per_die * C_local + ((BH - dies * per_die) * C_spread + dies - 1) / dies);
    }
};
// What workgroup `id` of such a grid works on; false: nothing.
SV_HOST_DEVICE inline bool wide_role(int id, const WideRoles &r, int &c, int &C, int &bh, bool &local)
{
    const int die = id % r.dies, slot = id / r.dies, of_heads = r.per_die * r.C_local;
    local = slot < of_heads;
    if (local) {
        C = r.C_local;
        bh = die + r.dies * (slot / C);
        c = slot % C;
        return true;
    }
    C = r.C_spread;
    const int k = (slot - of_heads) * r.dies + die;
    bh = r.dies * r.per_die + k / C;
    c = k % C;
    return bh < r.BH;
}

// The flag words of such a head, of the 2 * kMaxChunks it has in the workspace: the phases side by side, or packed where the head lives on one die.
// Its flags are stored into that die's L2; the next head's, where it is spread, are polled across dies, and the two have to stay off one cache line.  Where
// the flags lie `past_line` bytes past a multiple of 128 (a multiple of 16), a packed head of at most this many workgroups ends a line early enough.
SV_HOST_DEVICE inline int wide_flag_word(bool local, int phase, int c, int C, int max_chunks) { return phase * (local ? C : max_chunks) + c; }
SV_HOST_DEVICE inline int wide_most_beside_spread(int past_line, int max_chunks) { return max_chunks - past_line / 16; }

// Phase key (the `bh` argument of TileWalk) of head bh in the die-local forms of the kernels, where die x
// holds heads x, x + n_dies, ...: keyed by the head index itself, heads of one die would share phases (two
// distinct ones for four heads), so the sixteen phases are dealt die by die, the heads of a die as far apart
// as their number allows.
SV_HOST_DEVICE inline int die_local_phase_key(int bh, int n_dies, int BH)
{
    const int per_die = BH / n_dies > 0 ? BH / n_dies : 1;
    const int stride = per_die < 16 ? 16 / per_die : 1;
    return ((bh / n_dies) * stride + (bh % n_dies) % stride) & 15;
}

}  // namespace sv
