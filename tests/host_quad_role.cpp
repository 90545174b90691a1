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
                    if (!sv::quad_state_pays(BH, d, n, mode == 1, mode == 2, 256)) continue;
                    const int C = 256 / (4 * BH);
                    if (C < 1 || 4 * C * BH > 256 || 4 * C * BH < 192) return printf("FAIL fill BH=%d\n", BH), 1;
                    ++cases;
                }
    // layers on the quadrants and on whole rows: one's time over the other's (percent, in both of two runs to one side of 100 by 2 and more)
    struct Layer { int d, mode, BH, n, percent; } layers[] = {       // mode 0: plain, 1: full table, 2: factored tables
        {112, 0, 64, 960, 93}, {112, 0, 64, 1080, 94}, {112, 0, 24, 1680, 106}, {112, 0, 32, 2400, 105}, {112, 0, 28, 2520, 105}, {112, 0, 20, 4200, 103},
        {112, 0, 18, 3360, 105}, {112, 0, 12, 4680, 95}, {112, 0, 8, 6840, 97}, {112, 0, 5, 12840, 104}, {112, 0, 4, 9960, 108}, {112, 0, 2, 32040, 94},
        {112, 2, 64, 960, 94}, {112, 2, 24, 2520, 104}, {112, 2, 32, 2640, 105}, {112, 2, 26, 2640, 105}, {112, 2, 20, 2040, 97}, {112, 2, 16, 2520, 95},
        {112, 2, 8, 8760, 97}, {112, 1, 20, 1560, 94}, {112, 1, 24, 2640, 105}, {112, 1, 64, 600, 87}, {128, 0, 24, 2880, 95}, {128, 0, 20, 4560, 96},
        {128, 0, 64, 1440, 91}, {128, 2, 24, 3720, 107}, {128, 2, 21, 3840, 95}, {112, 0, 30, 1320, 105}, {112, 0, 19, 1200, 95}, {112, 2, 28, 840, 98}, {112, 2, 19, 2160, 97}, {128, 2, 16, 4320, 96}, {128, 2, 64, 1440, 95}, {128, 1, 20, 3240, 94}};
    for (const Layer &l : layers) {
        if (sv::quad_state_pays(l.BH, l.d, l.n, l.mode == 1, l.mode == 2, 256) != (l.percent < 100)) return printf("FAIL line d=%d mode=%d BH=%d n=%d\n", l.d, l.mode, l.BH, l.n), 1;
        ++cases;
    }
    printf("OK %ld\n", cases);
    return 0;
}
