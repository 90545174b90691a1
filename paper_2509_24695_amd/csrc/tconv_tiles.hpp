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

// Time of a call in us on the tile kernel `f`, as a fit to what it measures: a start that grows with the tile, and a time per
// K-step of 32 channels that depends on how many tiles a compute unit gets.  From 1 050 calls (1 to 151 200 tokens, 64 to
// 2 240 channels, 1 to 21 frames, with and without a cache; five devices), each on all five kernels: the kernel with the smallest
// fitted time (with the limit in tconv_form) is on average 0.3 % and at worst 14 % slower than the fastest one, and never more than 3.4 % slower than the single
// kernel of 256 x 256 that served every call before.  A rule without the starts, and with one time per step for each kernel, took 4.9 % and up
// to 56 % (short contractions on too large tiles; 3 600 tokens of 1 920 channels 110 us where the long kernel takes 103).
// Where channels are no multiple of 32 rows start inside 64-byte blocks, which costs loads more than products: TAIL.
inline double row_cost(TconvFormId f, int B, int T, int HW, int D, bool cache, int num_cu)
{
    const int64_t tiles = tconv_tiles_m(f, B, T, HW) * tconv_tiles_n(f, D);
    const int taps = T > 1 ? 3 : cache ? 2 : 1;       // of a tile that needs most (tc_taps)
    const double per_cu = (double)tiles / num_cu;
    const double rounds = (double)((tiles + num_cu - 1) / num_cu);
    const double steps = (double)((D + 31) / 32) * taps;
    const bool tail = D % 32 != 0;
    // one tile to a compute unit at a time: per step with up to half of the units busy, with all, and per further round
    struct Large { double start, half, full, more; };
    constexpr Large k256[2] = {{12.5, 0.555, 0.63, 0.66}, {12, 0.70, 0.81, 0.82}};
    constexpr Large k256x128[2] = {{9.5, 0.565, 0.565, 0.62}, {9.5, 0.57, 0.64, 0.64}};
    constexpr Large kLong[2] = {{10.2, 0.535, 0.62, 0.67}, {10, 0.70, 0.82, 0.83}};
    // two at a time: per step with one tile each (on few units, on all), just above one, with two; then in proportion
    struct Middle { double start, few, one, above, two, each; };
    constexpr Middle k128[2] = {{6, 0.36, 0.36, 0.45, 0.66, 0.345}, {6, 0.335, 0.40, 0.62, 0.70, 0.44}};
    // five at a time: per step by tiles per unit, rounded up
    struct Small { double start, base, each; };
    constexpr Small k64[2] = {{4, 0.06, 0.115}, {3.6, 0.01, 0.17}};

    if (f == kForm64) return k64[tail].start + steps * (k64[tail].base + k64[tail].each * rounds);
    if (f == kForm128) {
        const Middle &m = k128[tail];
        const double over = m.each * per_cu;
        return m.start + steps * (per_cu <= 1 ? m.few + (m.one - m.few) * per_cu
                                  : per_cu <= 2 ? m.above + (m.two - m.above) * (per_cu - 1) : over > m.two ? over : m.two);
    }
    const Large &l = f == kForm256 ? k256[tail] : f == kForm256x128 ? k256x128[tail] : kLong[tail];
    const double filled = per_cu <= 0.5 ? 0 : 2 * per_cu - 1;
    return l.start * (1 + 0.4 * (rounds - 1)) + steps * (rounds <= 1 ? l.half + (l.full - l.half) * filled : rounds * l.more);
}

// Time of a call in us on a frame kernel: a start, more of it per further round of tiles, and a time per K-step with up to half of the
// compute units busy, with all, and per round of several.  Fitted to 1 246 calls (1 to 21 frames, 40 to 3 600 positions, 96 to 2 240
// channels), 5 to 7 % off.
inline double frame_cost(TconvFormId f, int B, int T, int HW, int D, int num_cu)
{
    struct Fit { double start, half, full, more, again; };
    constexpr Fit kFit[kTconvForms - kFrames3] = {{11.0, 0.93, 1.24, 1.10, 0.43}, {11.9, 0.98, 1.30, 1.15, 1.48}, {11.8, 1.01, 1.32, 1.21, 1.14}};
    const Fit &fit = kFit[f - kFrames3];
    const int64_t tiles = tconv_tiles_m(f, B, T, HW) * tconv_tiles_n(f, D);
    const double per_cu = (double)tiles / num_cu, rounds = (double)((tiles + num_cu - 1) / num_cu);
    const double filled = per_cu <= 0.5 ? 0 : 2 * per_cu - 1, steps = (double)D / 32;
    return fit.start * (1 + fit.again * (rounds - 1)) + steps * (rounds <= 1 ? fit.half + (fit.full - fit.half) * filled : rounds * fit.more);
}
// Which kernel serves a call on num_cu compute units: the cheapest on row tiles, or one on frame tiles where that is cheaper.  A third of the calls of 32 channels and more, 100 to
// 3 600 positions and 2 frames and more are faster on tiles of frames, by 4 to 50 %: a block of 3 x 1 560 x 2 240 with a cache 131 -> 101 us,
// 2 x 3 x 1 447 x 2 240 264 -> 179, 5 x 752 x 2 240 120 -> 86, a clip of 21 x 1 560 x 2 240 809 -> 758; small calls and few channels are not
// (3 x 449 x 96 7.1 against 15.3).  kNow: what the kernels on row tiles take of what row_cost says since their accumulators stay in one
// register file and their operand reads go without bank conflicts.  Over those calls the choice costs 0.7 % on average against the fastest
// kernel of all, and no call takes more than 3 % longer than on row tiles.
inline TconvFormId tconv_form(int B, int T, int HW, int D, bool cache, int num_cu)
{
    TconvFormId best = kForm256;
    double least = row_cost(kForm256, B, T, HW, D, cache, num_cu);
    // The long kernel only while its tiles leave a third of the compute units idle.  With more it is level with the 256 x 256 kernel
    // (2 % ahead on average) but draws more power: 171 tiles of 210 steps, six calls in a row take 812, 818, 825, 831, 839 and 846 us on
    // six devices, where the 256 x 256 kernel takes 829 to 834.
    const int64_t tiles = tconv_tiles_m(kForm256Long, B, T, HW) * tconv_tiles_n(kForm256Long, D);
    for (const TconvFormId f : {kForm256x128, kForm128, kForm64, kForm256Long}) {
        if (f == kForm256Long && 3 * tiles > 2 * num_cu) continue;
        const double us = row_cost(f, B, T, HW, D, cache, num_cu);
        if (us < least) { least = us; best = f; }
    }
    constexpr double kNow[kRowForms] = {0.99, 0.725, 0.826, 0.99, 1.0};
    least *= kNow[best];
    for (const TconvFormId f : {kFrames3, kFrames5, kFrames7})
        if (tconv_fits(f, T, D) && frame_cost(f, B, T, HW, D, num_cu) < least) return f;
    return best;
}

// Last token row of the tile of `bm` rows from m0 on, M tokens in all (m0 < M; m0 + bm may not fit an int).
SV_HOST_DEVICE inline int tc_last_row(int m0, int bm, int M) { return M - m0 > bm ? m0 + bm - 1 : M - 1; }

}  // namespace sv
