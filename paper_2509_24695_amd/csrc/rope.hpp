// RoPE after ReLU (numerator of the Sec. 3.2 equation): where the (cos, sin)
// entries of a token tile come from.
//
//   kRopeNone   no rotation (the plain entry points);
//   kRopeTable  a caller-made table, fp32 [N][d/2][2], read with the tile: its rows
//               are as long as the token's K and V rows together, and although all
//               heads share them (they come from HBM once) every wave has to pull
//               its rows through the caches;
//   kRope3D     3-D rotary embedding in factored form: pair p is turned by the frame,
//               the row or the column position of the token, so three small tables
//               (frames x n_t, rows x n_h, cols x n_w entries) say everything.  They
//               are copied into LDS once per workgroup and looked up per pair:
//               the token loops then issue no memory instruction for the rotation
//               and the kernel's traffic stays at the four token streams.
//
// All kernels apply the rotation in the coalesced register layout of a freshly
// loaded tile, where a 32-bit word is exactly one feature pair (2p, 2p+1) and a
// lane's 16-byte chunk holds four consecutive pairs of one token.
#pragma once

#include "common.hpp"

namespace sv {

constexpr int kRopeNone = 0, kRopeTable = 1, kRope3D = 2;
// kRope3D whose axes have a multiple of four pairs each: a lane's four pairs, whose first is a multiple of four, lie in one axis side by side, and
// a chunk's entries are one address and two 16-byte LDS reads instead of four and four of 8.  For the d = 64 kernels, chosen by the
// launcher: block steps of 32 heads, 4 680 tokens 27.1 -> 25.4 us, 10 800 tokens 44.2 -> 42.2, layer of 2 x 32 heads, 75 600 tokens 447 -> 444
// (a run-time choice inside the kernel gains nothing: its branch keeps the reads from being moved ahead).
constexpr int kRope3DWhole = 3;
constexpr bool is_rope3d(int mode) { return mode >= kRope3D; }

// Factored 3-D rotary tables (device pointers): [frames][n_t][2], [rows][n_h][2],
// [cols][n_w][2] fp32 (cos, sin).  Token t sits at frame t / (rows*cols), row
// (t / cols) % rows, column t % cols; pairs [0, n_t) follow the frame, pairs
// [n_t, n_t + n_h) the row, the rest the column.
struct Rope3D {
    const float *cs_t, *cs_h, *cs_w;
    int frames, rows, cols, n_t, n_h, n_w;
};

// Kernel argument of every mode.
struct RopeArg {
    const float *table;   // kRopeTable
    Rope3D r3;            // kRope3D
};

constexpr int kRope3dLdsBytes = 32768;   // LDS reserved for the three tables (the host checks that they fit)

__host__ __device__ constexpr int rope3d_entries(int frames, int rows, int cols, int n_t, int n_h, int n_w) {
    return frames * n_t + rows * n_h + cols * n_w;
}

// Copies the three tables to LDS, frame table first, in two parts so that the table reads can be
// the first memory operations of a kernel: _begin issues the loads of the first kRope3dFillBatch
// entries per thread (all of them, for tables of up to 16 KB and 256 threads) without waiting,
// the caller then requests its first token tiles, and _end stores to LDS (and copies whatever
// is left).  Memory operations return in order, so the tables are there before the tiles and the
// copy costs no round trip of its own.  All threads of the workgroup call both; the caller places
// a workgroup barrier between _end and the first lookup.
constexpr int kRope3dFillBatch = 8;
struct Rope3dFill {
    f32x2 v[kRope3dFillBatch];
};
// Entry e (clamped into range) of the three tables laid end to end.
__device__ __forceinline__ f32x2 rope3d_entry_flat(const Rope3D &R, int nt, int nh, int total, int e)
{
    e = e < total ? e : total - 1;
    const f32x2 *src = e < nt ? reinterpret_cast<const f32x2 *>(R.cs_t) + e
                              : (e < nt + nh ? reinterpret_cast<const f32x2 *>(R.cs_h) + (e - nt)
                                             : reinterpret_cast<const f32x2 *>(R.cs_w) + (e - nt - nh));
    return *src;
}
__device__ __forceinline__ void rope3d_lds_fill_begin(const Rope3D &R, Rope3dFill &f)
{
    const int nt = R.frames * R.n_t, nh = R.rows * R.n_h, total = nt + nh + R.cols * R.n_w;
#pragma unroll
    for (int j = 0; j < kRope3dFillBatch; ++j)
        f.v[j] = rope3d_entry_flat(R, nt, nh, total, (int)threadIdx.x + j * (int)blockDim.x);
}
__device__ __forceinline__ void rope3d_lds_fill_end(unsigned char *lds_tab, const Rope3D &R, const Rope3dFill &f)
{
    f32x2 *dst = reinterpret_cast<f32x2 *>(lds_tab);
    const int nt = R.frames * R.n_t, nh = R.rows * R.n_h, total = nt + nh + R.cols * R.n_w;
#pragma unroll
    for (int j = 0; j < kRope3dFillBatch; ++j) {
        const int e = (int)threadIdx.x + j * (int)blockDim.x;
        if (e < total) dst[e] = f.v[j];
    }
    for (int e = (int)threadIdx.x + kRope3dFillBatch * (int)blockDim.x; e < total; e += (int)blockDim.x)
        dst[e] = rope3d_entry_flat(R, nt, nh, total, e);
}

// One (cos, sin) entry straight from global memory (plain-FMA kernels).
__device__ __forceinline__ f32x2 rope3d_entry_global(const Rope3D &R, int tok, int p)
{
    const int rc = R.rows * R.cols;
    const int f = tok / rc, rem = tok - f * rc, r = rem / R.cols, c = rem - r * R.cols;
    if (p < R.n_t) return reinterpret_cast<const f32x2 *>(R.cs_t)[f * R.n_t + p];
    if (p < R.n_t + R.n_h) return reinterpret_cast<const f32x2 *>(R.cs_h)[r * R.n_h + (p - R.n_t)];
    return reinterpret_cast<const f32x2 *>(R.cs_w)[c * R.n_w + (p - R.n_t - R.n_h)];
}

// Rotation source of one wave's token stream.
//   STEPS  16-byte chunks a lane holds per tile (rows row0 + j * rows_per_step, j < STEPS)
//   DEPTH  tiles in flight (kRopeTable keeps their table rows in registers)
template <int MODE, int STEPS, int DEPTH>
struct Rotator;

template <int STEPS, int DEPTH>
struct Rotator<kRopeNone, STEPS, DEPTH> {
    __device__ __forceinline__ Rotator(const RopeArg &, int, int, int, int, int, int, const unsigned char *) {}
    __device__ __forceinline__ void request(int, bool, int) {}
    template <int TILE> __device__ __forceinline__ void begin_tile(const TileWalk &, int) {}
    __device__ __forceinline__ void fetch(int, int, f32x2 (&)[4]) const {}
    __device__ __forceinline__ u32x4 rotate_with(u32x4 w, const f32x2 (&)[4]) const { return w; }
};

template <int STEPS, int DEPTH>
struct Rotator<kRopeTable, STEPS, DEPTH> {
    rsrc_t rT;
    uint32_t table_row_bytes, lane_off, step_bytes;
    f32x4 cs[DEPTH][STEPS][2];

    // t1: end of the token range; d: head dimension; row0, rows_per_step: the lane's rows of a
    // tile; pair0: first of the lane's four consecutive pairs; lane_valid: the pairs exist.
    __device__ __forceinline__ Rotator(const RopeArg &a, int t1, int d, int row0, int rows_per_step, int pair0,
                                       int /*lane_valid*/, const unsigned char *)
        : rT(make_rsrc(a.table, (uint32_t)t1 * (uint32_t)d * 4u)), table_row_bytes((uint32_t)d * 4u),
          lane_off((uint32_t)row0 * (uint32_t)d * 4u + (uint32_t)pair0 * 8u),
          step_bytes((uint32_t)rows_per_step * (uint32_t)d * 4u) {}
    // A new one holds no rows: assigned over another it would take the requested ones with it.
    Rotator &operator=(const Rotator &) = delete;

    // Requests the table rows of the tile that starts at token tok0 into stage s (nothing
    // is read if !valid: out-of-range offsets return zeros).
    __device__ __forceinline__ void request(int s, bool valid, int tok0)
    {
        const uint32_t off0 = tile_offset(valid, tok0, table_row_bytes);
#pragma unroll
        for (int j = 0; j < STEPS; ++j) {
            cs[s][j][0] = load_cached16(rT, off0 + lane_off + (uint32_t)j * step_bytes);
            cs[s][j][1] = load_cached16(rT, off0 + lane_off + (uint32_t)j * step_bytes + 16u);
        }
    }
    template <int TILE> __device__ __forceinline__ void begin_tile(const TileWalk &, int) {}
    __device__ __forceinline__ void fetch(int s, int j, f32x2 (&e)[4]) const
    {
        e[0] = f32x2{cs[s][j][0].x, cs[s][j][0].y};
        e[1] = f32x2{cs[s][j][0].z, cs[s][j][0].w};
        e[2] = f32x2{cs[s][j][1].x, cs[s][j][1].y};
        e[3] = f32x2{cs[s][j][1].z, cs[s][j][1].w};
    }
    __device__ __forceinline__ u32x4 rotate_with(u32x4 w, const f32x2 (&e)[4]) const
    {
        return u32x4{rope_rotate_pair(w.x, e[0].x, e[0].y), rope_rotate_pair(w.y, e[1].x, e[1].y),
                     rope_rotate_pair(w.z, e[2].x, e[2].y), rope_rotate_pair(w.w, e[3].x, e[3].y)};
    }
};

// Where a lane's STEPS rows of the tile in work are on the three axes.  BYTES: positions are byte offsets into the axes' tables, one position
// n pairs * 8 bytes from the next (8 where the axis has no pairs: its offsets are not used); otherwise frame, row and column themselves.
template <int STEPS, bool BYTES>
struct Rope3dPositions {
    int rows, cols, rc, row0, rows_per_step;
    int bytes_t, bytes_h, bytes_w;     // wave-uniform: bytes from one position to the next
    int last_t, end_h, end_w;          // the last frame; past the last row, column
    float inv_rows, inv_cols;
    int st, sh, sw;                    // wave-uniform: one stride of the walk as (frames, rows, columns)
    int t[STEPS], h[STEPS], w[STEPS];

    __device__ __forceinline__ Rope3dPositions(const Rope3D &R, int row0_, int rows_per_step_)
        : rows(R.rows), cols(R.cols), rc(R.rows * R.cols), row0(row0_), rows_per_step(rows_per_step_), bytes_t(8 * (R.n_t ? R.n_t : 1)),
          bytes_h(8 * (R.n_h ? R.n_h : 1)), bytes_w(8 * (R.n_w ? R.n_w : 1)), last_t((R.frames - 1) * step_t()), end_h(R.rows * step_h()),
          end_w(R.cols * step_w()), inv_rows(1.0f / (float)R.rows), inv_cols(1.0f / (float)R.cols), st(0), sh(0), sw(0) {}
    __device__ __forceinline__ int step_t() const { return BYTES ? bytes_t : 1; }
    __device__ __forceinline__ int step_h() const { return BYTES ? bytes_h : 1; }
    __device__ __forceinline__ int step_w() const { return BYTES ? bytes_w : 1; }

    // Positions of the lane's rows of the i-th tile of the walk; call for i = 0, 1, 2, ... in turn.
    // A walk visits tiles a constant stride apart except where its cyclic order wraps around, so
    // normally every row is the same row of the previous tile plus the stride's (frames, rows,
    // columns), with two carries: a dozen integer instructions per row and one scalar comparison.
    // Integer divisions (long instruction sequences on this hardware) are left to the first tile
    // and the wrap; there the rows inside the tile are reached from the tile's own position
    // with small carries done in floating point: (x + 0.5) / n is at least 0.5 / n away from
    // an integer and x stays far below 2^20, so the truncated product with the rounded
    // reciprocal is the exact quotient.  A frame index is capped at the last frame: that
    // happens to rows past the last token only (they hold zeros, any entry will do), and a
    // row past the end stays past the end until the walk wraps.
    template <int TILE> __device__ __forceinline__ void begin_tile(const TileWalk &walk, int i)
    {
        if (i == 0 || i + walk.rot == walk.count) {
            if (i == 0) {                                  // one stride as (frames, rows, columns)
                const int stride = walk.step * TILE, f = stride / rc, srem = stride - f * rc, r = srem / cols;
                st = f * step_t();
                sh = r * step_h();
                sw = (srem - r * cols) * step_w();
            }
            const int tok0 = walk.template token<TILE>(i);
            const int f0 = tok0 / rc, rem = tok0 - f0 * rc, r0 = rem / cols, c0 = rem - r0 * cols;
#pragma unroll
            for (int j = 0; j < STEPS; ++j) {
                const int c1 = c0 + row0 + j * rows_per_step;
                const int dr = (int)(((float)c1 + 0.5f) * inv_cols);
                const int r1 = r0 + dr;
                const int df = (int)(((float)r1 + 0.5f) * inv_rows);
                w[j] = __mul24(c1 - __mul24(dr, cols), step_w());
                h[j] = __mul24(r1 - __mul24(df, rows), step_h());
                const int tt = __mul24(f0 + df, step_t());
                t[j] = tt < last_t ? tt : last_t;
            }
        } else {
#pragma unroll
            for (int j = 0; j < STEPS; ++j) {
                const int cc = w[j] + sw;
                const bool cr = cc >= end_w;
                w[j] = cr ? cc - end_w : cc;
                const int rr = h[j] + sh + (cr ? step_h() : 0);
                const bool cf = rr >= end_h;
                h[j] = cf ? rr - end_h : rr;
                const int tt = t[j] + st + (cf ? step_t() : 0);
                t[j] = tt < last_t ? tt : last_t;
            }
        }
    }

};

template <int STEPS, int DEPTH>
struct Rotator<kRope3D, STEPS, DEPTH> {
    const unsigned char *tab;          // the three tables in LDS
    // Entry of pair q: base + the position on its axis, in bytes.  Which axis a pair follows are two lane masks in scalar registers: two selections and an
    // addition per pair, where position times a stride that is zero on the other axes took four instructions and twelve vector
    // registers (d = 112 layers 1 to 2 % less; what it frees lets the one-launch block step of d = 112 fit).
    uint32_t base[4];
    bool on_t[4], on_h[4];
    Rope3dPositions<STEPS, true> pos;

    __device__ __forceinline__ Rotator(const RopeArg &a, int /*t1*/, int d, int row0, int rows_per_step, int pair0, int /*lane_valid*/,
                                       const unsigned char *lds_tab)
        : tab(lds_tab), pos(a.r3, row0, rows_per_step)
    {
        const Rope3D &R = a.r3;
        const uint32_t off_h = (uint32_t)(R.frames * R.n_t) * 8u, off_w = off_h + (uint32_t)(R.rows * R.n_h) * 8u;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            int p = pair0 + q;
            p = p < d / 2 ? p : d / 2 - 1;        // lanes past d (their features are zero) look at a valid entry
            on_t[q] = p < R.n_t;
            on_h[q] = p < R.n_t + R.n_h;          // looked at where on_t is false
            base[q] = on_t[q] ? (uint32_t)p * 8u : on_h[q] ? off_h + (uint32_t)(p - R.n_t) * 8u : off_w + (uint32_t)(p - R.n_t - R.n_h) * 8u;
        }
    }

    __device__ __forceinline__ void request(int, bool, int) {}
    template <int TILE> __device__ __forceinline__ void begin_tile(const TileWalk &walk, int i) { pos.template begin_tile<TILE>(walk, i); }

    // The (cos, sin) entries of the lane's four pairs of chunk j: four LDS reads.  Split from the
    // arithmetic so that a caller can issue the reads of a whole tile first and do other work
    // while they are in flight.
    __device__ __forceinline__ void fetch(int /*s*/, int j, f32x2 (&e)[4]) const
    {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int t = pos.t[j], h = pos.h[j], w = pos.w[j];   // values: a choice between the array elements would put them into memory
            e[q] = *reinterpret_cast<const f32x2 *>(tab + base[q] + (uint32_t)(on_t[q] ? t : on_h[q] ? h : w));
        }
    }
    __device__ __forceinline__ u32x4 rotate_with(u32x4 w, const f32x2 (&e)[4]) const
    {
        return u32x4{rope_rotate_pair(w.x, e[0].x, e[0].y), rope_rotate_pair(w.y, e[1].x, e[1].y),
                     rope_rotate_pair(w.z, e[2].x, e[2].y), rope_rotate_pair(w.w, e[3].x, e[3].y)};
    }
};

template <int STEPS, int DEPTH>
struct Rotator<kRope3DWhole, STEPS, DEPTH> {
    const unsigned char *tab;          // the three tables in LDS
    // Address of the lane's four entries = base + f * mul_f + r * mul_r + c * mul_c, one of the three not zero.  (With the offsets and lane masks of
    // kRope3D, which this form's single address gains nothing from, block steps of 64 heads and more took 1 % longer.)
    uint32_t base, mul_f, mul_r, mul_c;
    Rope3dPositions<STEPS, false> pos;

    __device__ __forceinline__ Rotator(const RopeArg &a, int /*t1*/, int d, int row0, int rows_per_step, int pair0, int /*lane_valid*/,
                                       const unsigned char *lds_tab)
        : tab(lds_tab), base(0), mul_f(0), mul_r(0), mul_c(0), pos(a.r3, row0, rows_per_step)
    {
        const Rope3D &R = a.r3;
        const uint32_t off_h = (uint32_t)(R.frames * R.n_t) * 8u, off_w = off_h + (uint32_t)(R.rows * R.n_h) * 8u;
        const int p = pair0 < d / 2 ? pair0 : d / 2 - 1;
        if (p < R.n_t) {
            base = (uint32_t)p * 8u;
            mul_f = (uint32_t)R.n_t * 8u;
        } else if (p < R.n_t + R.n_h) {
            base = off_h + (uint32_t)(p - R.n_t) * 8u;
            mul_r = (uint32_t)R.n_h * 8u;
        } else {
            base = off_w + (uint32_t)(p - R.n_t - R.n_h) * 8u;
            mul_c = (uint32_t)R.n_w * 8u;
        }
    }

    __device__ __forceinline__ void request(int, bool, int) {}
    template <int TILE> __device__ __forceinline__ void begin_tile(const TileWalk &walk, int i) { pos.template begin_tile<TILE>(walk, i); }
    __device__ __forceinline__ void fetch(int /*s*/, int j, f32x2 (&e)[4]) const
    {
        // 24-bit multiplies run at full rate (32-bit ones at a quarter); positions and strides are far below 2^24
        const uint32_t addr = base + __umul24((uint32_t)pos.t[j], mul_f) + __umul24((uint32_t)pos.h[j], mul_r) + __umul24((uint32_t)pos.w[j], mul_c);
        const f32x4 a = *reinterpret_cast<const f32x4 *>(tab + addr), b = *reinterpret_cast<const f32x4 *>(tab + addr + 16);
        e[0] = f32x2{a.x, a.y};
        e[1] = f32x2{a.z, a.w};
        e[2] = f32x2{b.x, b.y};
        e[3] = f32x2{b.z, b.w};
    }
    __device__ __forceinline__ u32x4 rotate_with(u32x4 w, const f32x2 (&e)[4]) const
    {
        return u32x4{rope_rotate_pair(w.x, e[0].x, e[0].y), rope_rotate_pair(w.y, e[1].x, e[1].y),
                     rope_rotate_pair(w.z, e[2].x, e[2].y), rope_rotate_pair(w.w, e[3].x, e[3].y)};
    }
};

}  // namespace sv
