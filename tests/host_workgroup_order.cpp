// chunk_major_role (csrc/tile_walk.hpp): every (chunk, head) exactly once, and each die's ids are one run of the list.
#include <cstdio>
#include <vector>

#include "../paper_2509_24695_amd/csrc/tile_walk.hpp"

int main()
{
    long cases = 0;
    for (int dies : {1, 2, 4, 8})
        for (int C = 1; C <= 40; ++C)
            for (int BH : {1, 2, 3, 5, 7, 8, 13, 20, 32, 40, 64, 129, 160}) {
                std::vector<int> hits(C * BH, 0);
                for (int e = 0; e < dies; ++e) {
                    int last = -1;
                    for (int id = e; id < C * BH; id += dies) {
                        int c = -1, bh = -1;
                        sv::chunk_major_role(id, C, BH, dies, c, bh);
                        if (c < 0 || c >= C || bh < 0 || bh >= BH) return printf("FAIL range\n"), 1;
                        const int at = c * BH + bh;
                        if (last >= 0 && at != last + 1) return printf("FAIL run C=%d BH=%d\n", C, BH), 1;
                        last = at;
                        ++hits[at];
                    }
                }
                for (int h : hits)
                    if (h != 1) return printf("FAIL cover C=%d BH=%d\n", C, BH), 1;
                ++cases;
            }
    printf("OK %ld grids\n", cases);
    return 0;
}
