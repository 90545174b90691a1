// quad_role (csrc/tile_walk.hpp): every quadrant of every (chunk, head) exactly once, the four of one on one die; and where the rules
// of csrc/layout_rules.hpp put the quadrant kernel, its chunks fill the device and fit its flags.
#include <cstdio>
#include <vector>

#include "../paper_2509_24695_amd/csrc/layout_rules.hpp"
#include "../paper_2509_24695_amd/csrc/tile_walk.hpp"

int main()
{
    long cases = 0;
    for (int dies : {1, 2, 4, 8})
        for (bool major : {false, true})
            for (int C = 1; C <= 16; ++C)
                for (int BH : {1, 2, 3, 5, 7, 8, 13, 20, 32, 40, 64, 129}) {
                    std::vector<int> hits(4 * C * BH, 0), die(C * BH, -1);
                    const int grid = sv::quad_grid(C, BH, dies);
                    if (grid < 4 * C * BH || grid >= 4 * (C * BH + dies)) return printf("FAIL grid\n"), 1;
                    for (int id = 0; id < grid; ++id) {
                        int c = -1, bh = -1, q = -1;
                        if (!sv::quad_role(id, C, BH, dies, major, c, bh, q)) continue;
                        if (c < 0 || c >= C || bh < 0 || bh >= BH || q < 0 || q > 3) return printf("FAIL range\n"), 1;
                        int &e = die[c * BH + bh];
                        if (e >= 0 && e != id % dies) return printf("FAIL die C=%d BH=%d\n", C, BH), 1;
                        e = id % dies;
                        ++hits[4 * (c * BH + bh) + q];
                    }
                    for (int h : hits)
                        if (h != 1) return printf("FAIL cover C=%d BH=%d\n", C, BH), 1;
                    ++cases;
                }
    for (int d : {112, 128})
        for (int mode : {0, 1, 2})
            for (int BH = 1; BH <= 300; ++BH)
                for (int n : {1, 100, 1000, 5000, 40000, 200000}) {
                    if (!sv::quad_state_pays(BH, d, n, mode == 1, 256)) continue;
                    const int C = 256 / (4 * BH);
                    if (C < 1 || 4 * C * BH > 256 || 4 * C * BH < 192) return printf("FAIL fill BH=%d\n", BH), 1;
                    ++cases;
                }
    printf("OK %ld\n", cases);
    return 0;
}
