// tc_taps (csrc/tconv_tiles.hpp): a tap is left out of a tile only if it is zero for every row of it.
#include <cstdio>
#include <initializer_list>

#include "../paper_2509_24695_amd/csrc/tconv_tiles.hpp"

int main()
{
    long cases = 0;
    for (int B = 1; B <= 3; ++B)
        for (int T = 1; T <= 5; ++T)
            for (int HW : {1, 3, 16, 53, 300})
                for (int bm : {1, 7, 64, 256})
                    for (int cache = 0; cache < 2; ++cache)
                        for (int g0 = 0; g0 < B * T * HW; g0 += bm) {
                            const int M = B * T * HW, g1 = (g0 + bm < M ? g0 + bm : M) - 1;
                            bool need[3] = {false, true, false};
                            for (int g = g0; g <= g1; ++g) {
                                const int t = g / HW % T;
                                need[0] |= t > 0 || cache;
                                need[2] |= t < T - 1;
                            }
                            int lo = -1, hi = -1;
                            sv::tc_taps(g0, g1, HW, T, cache != 0, lo, hi);
                            const bool covers = lo <= (need[0] ? 0 : 1) && hi >= (need[2] ? 3 : 2) && lo >= 0 && lo <= 1 && hi >= 2 && hi <= 3;
                            // tiles inside one frame leave out every tap they can
                            const bool tight = g0 / HW != g1 / HW || (lo == (need[0] ? 0 : 1) && hi == (need[2] ? 3 : 2));
                            if (!covers || !tight) return printf("FAIL T=%d HW=%d [%d, %d] cache=%d: %d %d\n", T, HW, g0, g1, cache, lo, hi), 1;
                            ++cases;
                        }
    printf("OK %ld tiles\n", cases);
    return 0;
}
