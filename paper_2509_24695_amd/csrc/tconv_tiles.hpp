// Tiles of the temporal-convolution kernels: which size a call takes, which tile a workgroup id works on, which taps a tile
// needs.  Plain C++ (no device code), shared by the kernels, the launcher and host-side tests.
#pragma once

#include <stdint.h>

#include <initializer_list>

#ifndef SV_HOST_DEVICE
#if defined(__HIPCC__)
#define SV_HOST_DEVICE __host__ __device__
#else
#define SV_HOST_DEVICE
#endif
#endif

namespace sv {

constexpr int kTcGroupM = 4;   // token tiles per group of the tile order

// Workgroups a grid needs for `tiles` tiles: eight XCD shares, each as long as the longest.
SV_HOST_DEVICE inline int64_t tc_grid_size(int64_t tiles) { return 8 * ((tiles + 7) / 8); }

// Workgroup id -> tile (token tile tm < tiles_m, channel tile tn < tiles_n); false if the id has no
// tile.  Tiles are ordered in groups of kTcGroupM token tiles, token tile fastest inside a group;
// consecutive workgroup ids go to the eight XCDs in turn, each with its own L2, so XCD e takes the
// e-th eighth of that order: the workgroups that run on one XCD at a time share a few token tiles
// and W's current K-slice, and all XCDs get the same number of tiles (to within one) however few
// there are.
SV_HOST_DEVICE inline bool tc_tile_of(int tiles_m, int tiles_n, int wg, int &tm, int &tn)
{
    const int64_t tiles = (int64_t)tiles_m * tiles_n;
    const int xcd = wg & 7, seq = wg >> 3;
    const int64_t begin = (xcd * tiles) >> 3, end = ((xcd + 1) * tiles) >> 3;
    const int64_t t = begin + seq;
    if (t >= end) return false;
    const int per_group = kTcGroupM * tiles_n, g = (int)(t / per_group), in = (int)(t - (int64_t)g * per_group);
    const int left = tiles_m - g * kTcGroupM, rows = left < kTcGroupM ? left : kTcGroupM;   // token tiles in this group
    tn = in / rows;
    tm = g * kTcGroupM + (in - tn * rows);
    return true;
}

// Taps [lo, hi) of the three that some token row of [g0, g1] needs (rows are numbered (batch, frame, position)): a tile whose
// rows all lie in the last frame has no use for the frame behind it, which is zero, one in the first frame without a
// cache none for the frame in front.
SV_HOST_DEVICE inline void tc_taps(int g0, int g1, int HW, int T, bool cache, int &lo, int &hi)
{
    const int f0 = g0 / HW, f1 = g1 / HW;                      // frames counted over batches
    lo = !cache && (T == 1 || (f0 == f1 && f0 % T == 0)) ? 1 : 0;
    hi = T == 1 || (f0 == f1 && f0 % T == T - 1) ? 2 : 3;
}

// The kernels a call may take: tconv_mfma on tiles of four sizes and tconv_mfma32 (256 x 256, 32 x 32 x 16 instructions), on tiles of
// consecutive token rows; tconv_frames on tiles of frames x positions.
enum TconvFormId { kForm256, kForm256x128, kForm128, kForm64, kForm256Long, kFrames3, kFrames5, kFrames7, kTconvForms, kRowForms = kFrames3 };
struct TconvTileSize { int bm, bn; };
constexpr TconvTileSize kTconvTile[kRowForms] = {{256, 256}, {256, 128}, {128, 128}, {64, 64}, {256, 256}};
// `frames` x 16 `blocks` positions x `channels`; back: the frames of a call make several groups, otherwise the call has no more than these.
struct FrameShape { int frames, blocks, channels; bool back; };
constexpr FrameShape kFrameShape[kTconvForms - kFrames3] = {{3, 5, 192, false}, {5, 3, 192, false}, {7, 2, 192, true}};

// Token tiles of a call on kernel `f`: groups of rows, or batches x groups of frames x groups of positions.
inline int64_t tconv_tiles_m(TconvFormId f, int B, int T, int HW)
{
    if (f < kRowForms) return ((int64_t)B * T * HW + kTconvTile[f].bm - 1) / kTconvTile[f].bm;
    const FrameShape &s = kFrameShape[f - kFrames3];
    return (int64_t)B * ((T + s.frames - 1) / s.frames) * (((int64_t)HW + 16 * s.blocks - 1) / (16 * s.blocks));
}
inline int tconv_tiles_n(TconvFormId f, int D)
{
    const int bn = f < kRowForms ? kTconvTile[f].bn : kFrameShape[f - kFrames3].channels;
    return (D + bn - 1) / bn;
}
// May kernel `f` serve the call at all?  Frame tiles take whole K-steps, and not one frame: it would fill a third of a tile
// (and tconv_frames counts positions in 32 bits: of two frames and more there are less than 2^30).
inline bool tconv_fits(TconvFormId f, int T, int D)
{
    if (f < kRowForms) return true;
    return D % 32 == 0 && T > 1 && f == (T <= 3 ? kFrames3 : T <= 5 ? kFrames5 : kFrames7);
}

// Time of a call in us on kernel `f`: a start, more of it per further round of tiles, and a time per K-step of 32 channels (and tap) that
// depends on how many tiles a compute unit gets.  Fitted to 2 878 calls (1 to 8 batches, 1 to 40 frames, 16 to 7 200 positions, 8 to 3 200 channels, with and
// without a cache; eight devices), each on all kernels that may serve it, so that the kernel of the smallest cost is the fastest one: the choice is on
// average 0.2 % slower than the fastest kernel, over 6 % slower for 18 of the calls and 15 % at worst (399 calls of a ninth device that the fit had not seen: 0.1 %, 5 % at worst).  For a kernel
// within 15 % of the fastest the cost itself is 5 to 11 % off.  Fitted before the kernels had their accumulators in one register file and their
// operand reads free of bank conflicts, it chose 0.7 % and up to 42 % slower ones: 2 x 2 286 x 2 016 (4 batches, no cache) 430 us on frame tiles,
// 332 on 256 x 256, 2 x 1 190 rows of 1 728 channels with a cache 63 on 128 x 128, 50 on 256 x 128.
// Where channels are no multiple of 32 rows start inside 64-byte blocks, which costs loads more than products: TAIL.
inline double tconv_cost(TconvFormId f, int B, int T, int HW, int D, bool cache, int num_cu)
{
    const int64_t tiles = tconv_tiles_m(f, B, T, HW) * tconv_tiles_n(f, D);
    const double per_cu = (double)tiles / num_cu, rounds = (double)((tiles + num_cu - 1) / num_cu);
    const int taps = f >= kFrames3 ? 1 : T > 1 ? 3 : cache ? 2 : 1;      // of a row tile that needs most (tc_taps); a frame tile takes all in a K-step
    const double steps = (double)((D + 31) / 32) * taps;
    const bool tail = D % 32 != 0;
    // one tile to a compute unit at a time: per step with up to half of the units busy, with all, and per further round
    struct Large { double start, half, full, more, again; };
    constexpr Large k256[2] = {{15.3, 0.535, 0.678, 0.652, 0.899}, {12.6, 0.706, 0.849, 0.677, 1.479}};
    constexpr Large k256x128[2] = {{9.71, 0.371, 0.481, 0.486, 0.587}, {8.60, 0.557, 0.604, 0.602, 0.629}};
    constexpr Large kLong[2] = {{14.8, 0.506, 0.543, 0.692, 0.934}, {10.7, 0.709, 0.693, 0.845, 0.730}};
    constexpr Large kFrames[kTconvForms - kFrames3] = {{13.3, 0.915, 1.159, 0.962, 2.213}, {14.2, 0.965, 1.206, 1.133, 1.268}, {14.0, 0.975, 1.274, 1.268, 0.947}};
    // two at a time: per step with one tile each (on few units, on all), just above one, with two; then in proportion
    struct Middle { double start, few, one, above, two, each; };
    constexpr Middle k128[2] = {{5.66, 0.211, 0.303, 0.442, 0.631, 0.339}, {4.97, 0.272, 0.401, 0.693, 0.749, 0.445}};
    // five at a time: per step by tiles per unit, half of it rounded up
    struct Small { double start, base, each; };
    constexpr Small k64[2] = {{3.96, -0.011, 0.141}, {3.97, -0.056, 0.185}};

    if (f == kForm64) {
        const double each = 0.5 * (rounds + per_cu);
        return k64[tail].start + steps * (k64[tail].base + k64[tail].each * (each > 1 ? each : 1));
    }
    if (f == kForm128) {
        const Middle &m = k128[tail];
        const double over = m.each * per_cu;
        return m.start + steps * (per_cu <= 1 ? m.few + (m.one - m.few) * per_cu
                                  : per_cu <= 2 ? m.above + (m.two - m.above) * (per_cu - 1) : over > m.two ? over : m.two);
    }
    const Large &l = f >= kFrames3 ? kFrames[f - kFrames3] : f == kForm256 ? k256[tail] : f == kForm256x128 ? k256x128[tail] : kLong[tail];
    const double filled = per_cu <= 0.5 ? 0 : 2 * per_cu - 1;
    return l.start * (1 + l.again * (rounds - 1)) + steps * (rounds <= 1 ? l.half + (l.full - l.half) * filled : rounds * l.more);
}

// Which kernel serves a call on num_cu compute units.
inline TconvFormId tconv_form(int B, int T, int HW, int D, bool cache, int num_cu)
{
    TconvFormId best = kForm256;
    double least = tconv_cost(kForm256, B, T, HW, D, cache, num_cu);
    for (const TconvFormId f : {kForm256x128, kForm128, kForm64, kForm256Long, kFrames3, kFrames5, kFrames7}) {
        if (!tconv_fits(f, T, D)) continue;
        // The long kernel only while its tiles leave a third of the compute units idle.  With more it is level with the 256 x 256 kernel
        // (2 % ahead on average) but draws more power: 171 tiles of 210 steps, six calls in a row take 812, 818, 825, 831, 839 and 846 us on
        // six devices, where the 256 x 256 kernel takes 829 to 834.
        if (f == kForm256Long && 3 * tconv_tiles_m(f, B, T, HW) * tconv_tiles_n(f, D) > 2 * num_cu) continue;
        const double us = tconv_cost(f, B, T, HW, D, cache, num_cu);
        if (us < least) { least = us; best = f; }
    }
    return best;
}

// Last token row of the tile of `bm` rows from m0 on, M tokens in all (m0 < M; m0 + bm may not fit an int).
SV_HOST_DEVICE inline int tc_last_row(int m0, int bm, int M) { return M - m0 > bm ? m0 + bm - 1 : M - 1; }

}  // namespace sv
