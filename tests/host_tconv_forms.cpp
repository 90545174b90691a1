// Prints, for each "B T HW D cache num_cu" on the command line, the kernel that a temporal convolution takes (tconv_form,
// csrc/tconv_tiles.hpp).  With no arguments: over a range of calls the choice may serve the call, its tiles cover every row, frame tiles have room for a
// call's frames or take them in groups, costs are finite and positive, and of the kernels that may serve the call the choice is the cheapest.
#include <cmath>
#include <cstdio>
#include <cstdlib>

#include "../paper_2509_24695_amd/csrc/tconv_tiles.hpp"

int main(int argc, char **argv)
{
    using namespace sv;
    const char *names[kTconvForms] = {"256x256", "256x128", "128x128", "64x64", "long", "3 frames", "5 frames", "7 frames"};
    for (int i = 1; i + 5 < argc; i += 6)
        printf("%s\n", names[tconv_form(atoi(argv[i]), atoi(argv[i + 1]), atoi(argv[i + 2]), atoi(argv[i + 3]), atoi(argv[i + 4]) != 0, atoi(argv[i + 5]))]);
    if (argc > 1) return 0;
    long cases = 0, on_frames = 0;
    for (int cus : {1, 64, 256, 304})
        for (int B : {1, 2, 7})
            for (int T : {1, 2, 3, 4, 5, 6, 7, 8, 14, 21, 1000})
                for (int HW : {1, 63, 64, 65, 79, 80, 81, 1560, 3600, 100000, (1 << 30) - 1, 2147483600, 2147483647})
                    for (int D = 8; D <= 26000; D = D < 256 ? D + 8 : D * 3 / 2 / 8 * 8)
                        for (int cache = 0; cache < 2; ++cache) {
                            if ((int64_t)B * T * HW >= (int64_t)1 << 31) continue;
                            ++cases;
                            const TconvFormId f = tconv_form(B, T, HW, D, cache != 0, cus);
                            if (f < 0 || f >= kTconvForms || !tconv_fits(f, T, D)) return printf("FAIL form T=%d D=%d\n", T, D), 1;
                            int64_t rows = tconv_tiles_m(f, B, T, HW);
                            if (f >= kFrames3) {
                                const FrameShape &s = kFrameShape[f - kFrames3];
                                ++on_frames;
                                if (D % 32 || T == 1 || (!s.back && T > s.frames)) return printf("FAIL T=%d D=%d\n", T, D), 1;
                                rows *= (int64_t)s.frames * 16 * s.blocks;
                            } else {
                                rows *= kTconvTile[f].bm;
                            }
                            if (rows < (int64_t)B * T * HW) return printf("FAIL cover B=%d T=%d HW=%d\n", B, T, HW), 1;
                            for (int i = 0; i < kTconvForms; ++i) {
                                const TconvFormId g = (TconvFormId)i;
                                const double us = tconv_cost(g, B, T, HW, D, cache != 0, cus);
                                const bool may = tconv_fits(g, T, D) && (g != kForm256Long || 3 * tconv_tiles_m(g, B, T, HW) * tconv_tiles_n(g, D) <= 2 * cus);
                                if (!(us > 0) || !std::isfinite(us) || (!may && f == g) || (may && us < tconv_cost(f, B, T, HW, D, cache != 0, cus)))
                                    return printf("FAIL cost HW=%d D=%d form %d\n", HW, D, g), 1;
                            }
                        }
    // rows of a tile: the last one exists, also where the tile's end does not fit an int
    const int max = 2147483647;
    struct { int m0, bm, M, want; } rows[] = {{0, 256, 1, 0}, {0, 64, 64, 63}, {64, 64, 65, 64}, {max - 255, 256, max, max - 1}, {max - 7, 64, max, max - 1},
                                             {max - 300, 256, max, max - 45}};
    for (auto &r : rows)
        if (tc_last_row(r.m0, r.bm, r.M) != r.want) return printf("FAIL last row %d\n", tc_last_row(r.m0, r.bm, r.M)), 1;
    printf("OK %ld calls, %ld on frames\n", cases, on_frames);
    return on_frames > 0 ? 0 : 1;
}
