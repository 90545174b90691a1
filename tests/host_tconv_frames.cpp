// For each "B T HW D cache num_cu" on the command line, the frames of the tile that the temporal convolution takes, 0 for a kernel on row
// tiles.  With no arguments: a call takes frame tiles only with whole K-steps, a tile with room for its frames or in several groups,
// and where that is fitted to be cheaper than on row tiles; tiles cover every row once.
#include <cmath>
#include <cstdio>
#include <cstdlib>

#include "../paper_2509_24695_amd/csrc/tconv_tiles.hpp"

int main(int argc, char **argv)
{
    using namespace sv;
    for (int i = 1; i + 5 < argc; i += 6) {
        const FrameFormId f = frame_form(atoi(argv[i]), atoi(argv[i + 1]), atoi(argv[i + 2]), atoi(argv[i + 3]), atoi(argv[i + 4]) != 0, atoi(argv[i + 5]));
        printf("%d\n", f == kNoFrames ? 0 : kFrameShape[f].frames);
    }
    if (argc > 1) return 0;
    long cases = 0, taken = 0;
    for (int cus : {1, 64, 256, 304})
        for (int B : {1, 2, 7})
            for (int T : {1, 2, 3, 4, 5, 6, 7, 8, 14, 21, 1000})
                for (int HW : {1, 79, 80, 81, 1560, 3600, 100000, (1 << 30) - 1, 2147483600, 2147483647})
                    for (int D = 8; D <= 26000; D = D < 256 ? D + 8 : D * 3 / 2 / 8 * 8)
                        for (int cache = 0; cache < 2; ++cache) {
                            if ((int64_t)B * T * HW >= (int64_t)1 << 31) continue;
                            ++cases;
                            const FrameFormId f = frame_form(B, T, HW, D, cache != 0, cus);
                            if (f == kNoFrames) continue;
                            ++taken;
                            const FrameShape &s = kFrameShape[f];
                            if (D % 32 || T == 1 || (!s.back && T > s.frames)) return printf("FAIL T=%d D=%d\n", T, D), 1;
                            const int64_t tiles = frame_tiles_m(s, B, T, HW), rows = (int64_t)s.frames * 16 * s.blocks;
                            if (tiles * rows < (int64_t)B * T * HW || !std::isfinite(frame_cost(f, B, T, HW, D, cus))) return printf("FAIL cover\n"), 1;
                        }
    printf("OK %ld calls, %ld on frames\n", cases, taken);
    return taken > 0 ? 0 : 1;
}
