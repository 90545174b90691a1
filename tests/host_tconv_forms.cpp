// Prints, for each "M D T cache num_cu" on the command line, the kernel that tconv_form (csrc/tconv_tiles.hpp) chooses.  With no
// arguments: over a range of calls the choice is one of the kernels, its cost is the smallest of those that may serve the call, and costs are
// finite and positive.
#include <cmath>
#include <cstdio>
#include <cstdlib>

#include "../paper_2509_24695_amd/csrc/tconv_tiles.hpp"

int main(int argc, char **argv)
{
    using namespace sv;
    const char *names[kTconvForms] = {"256x256", "256x128", "128x128", "64x64", "long"};
    for (int i = 1; i + 4 < argc; i += 5)
        printf("%s\n", names[tconv_form(atoll(argv[i]), atoi(argv[i + 1]), atoi(argv[i + 2]), atoi(argv[i + 3]) != 0, atoi(argv[i + 4]))]);
    if (argc > 1) return 0;
    long cases = 0;
    for (int cus : {1, 64, 256, 304})
        for (long M : {1L, 63L, 64L, 65L, 1560L, 4680L, 32760L, 151200L, 2147483647L})
            for (int D = 8; D <= 32768; D = D < 512 ? D + 8 : D * 3 / 2 / 8 * 8)
                for (int T : {1, 2, 21})
                    for (int cache = 0; cache < 2; ++cache) {
                        const TconvFormId f = tconv_form(M, D, T, cache != 0, cus);
                        if (f < 0 || f >= kTconvForms) return printf("FAIL form M=%ld D=%d\n", M, D), 1;
                        const int taps = T > 1 ? 3 : 1 + cache;
                        for (int g = 0; g < kTconvForms; ++g) {
                            const double us = tconv_cost((TconvFormId)g, M, D, taps, cus);
                            const bool may = g != kForm256Long || 3 * ((M + 255) / 256) * ((D + 255) / 256) <= 2 * cus;
                            if (!(us > 0) || !std::isfinite(us) || (may && us < tconv_cost(f, M, D, taps, cus)) || (!may && f == g)) return printf("FAIL cost M=%ld D=%d form %d\n", M, D, g), 1;
                        }
                        ++cases;
                    }
    // rows of a tile: the last one exists, also where the tile's end does not fit an int
    const int max = 2147483647;
    struct { int m0, bm, M, want; } rows[] = {{0, 256, 1, 0}, {0, 64, 64, 63}, {64, 64, 65, 64}, {max - 255, 256, max, max - 1}, {max - 7, 64, max, max - 1},
                                             {max - 300, 256, max, max - 45}};
    for (auto &r : rows)
        if (tc_last_row(r.m0, r.bm, r.M) != r.want) return printf("FAIL last row %d\n", tc_last_row(r.m0, r.bm, r.M)), 1;
    printf("OK %ld calls\n", cases);
    return 0;
}
