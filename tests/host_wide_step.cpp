// The one-launch block step of d = 112 and 128 (csrc/layout_rules.hpp, csrc/tile_walk.hpp): every (chunk, head) is dealt exactly once, a local head's to
// one die, within the device's compute units and the flags; and for each "d B H tokens rope layout" on the command line which form serves it on 256 compute
// units: "two" launches, a "sole" workgroup per head, "spread" (no head on one die), "local" or "mixed", and the workgroups of a spread and of a local head.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "../paper_2509_24695_amd/csrc/layout_rules.hpp"

static int check()
{
    long cases = 0;
    for (int BH = 8; BH <= 128; ++BH)
        for (int n : {1, 64, 65, 129, 700, 1560, 2048, 4680, 100000})
            for (bool table : {false, true}) {
                const sv::TokenLayout t{BH, BH, 112, 2, (int64_t)n * 112, 112};
                const int steps = (n + 63) / 64, plain = sv::plan_chunks(BH, n, 64, 256);
                const sv::WideRoles r = sv::wide_roles(t, n, steps, table, 256, 8);
                if (!r.dies) {
                    if (!table || n <= 2048) return printf("FAIL none BH=%d n=%d\n", BH, n), 1;
                    continue;
                }
                const int locals = r.dies * r.per_die, grid = r.grid();
                if (grid > 256 || r.C_local < 1 || r.C_spread < 1 || r.C_local > steps || r.C_spread > steps) return printf("FAIL size BH=%d n=%d\n", BH, n), 1;
                if (r.C_local > sv::kMaxChunks || r.C_spread > sv::kMaxChunks || 10 * r.C_local < 8 * plain) return printf("FAIL chunks BH=%d n=%d\n", BH, n), 1;
                std::vector<int> hits(BH * sv::kMaxChunks, 0), die(BH, -1);
                for (int id = 0; id < grid; ++id) {
                    int c = -1, C = -1, bh = -1;
                    bool local = false;
                    if (!sv::wide_role(id, r, c, C, bh, local)) continue;
                    if (bh < 0 || bh >= BH || local != (bh < locals) || C != (local ? r.C_local : r.C_spread) || c < 0 || c >= C) return printf("FAIL role BH=%d\n", BH), 1;
                    if (local && die[bh] >= 0 && die[bh] != id % 8) return printf("FAIL die BH=%d\n", BH), 1;
                    die[bh] = id % 8;
                    ++hits[bh * sv::kMaxChunks + c];
                }
                for (int bh = 0; bh < BH; ++bh)
                    for (int c = 0; c < sv::kMaxChunks; ++c)
                        if (hits[bh * sv::kMaxChunks + c] != (c < (bh < locals ? r.C_local : r.C_spread))) return printf("FAIL cover BH=%d n=%d\n", BH, n), 1;
                ++cases;
            }
    printf("OK %ld\n", cases);
    return 0;
}

int main(int argc, char **argv)
{
    if (argc == 1) return check();
    for (int i = 1; i + 5 < argc; i += 6) {
        const int d = atoi(argv[i]), B = atoi(argv[i + 1]), H = atoi(argv[i + 2]), n = atoi(argv[i + 3]);
        const bool table = !strcmp(argv[i + 4], "table"), axes = !strcmp(argv[i + 4], "axes"), token_major = !strcmp(argv[i + 5], "bnhd");
        const sv::TokenLayout t = token_major ? sv::TokenLayout{B * H, H, d, 2, d, (int64_t)H * d} : sv::TokenLayout{B * H, H, d, 2, (int64_t)n * d, d};
        const int C = sv::plan_chunks(B * H, n, 64, 256);
        const sv::WideRoles r = sv::wide_roles(t, n, (n + 63) / 64, table, 256, C > 1 ? 8 : 0);
        if (!sv::wide_step_serves(t, n, C, table, axes, 256)) printf("two 0 0\n");
        else if (C == 1) printf("sole 1 0\n");
        else if (!r.dies) printf("spread %d 0\n", C);
        else printf("%s %d %d\n", t.BH % 8 ? "mixed" : "local", t.BH % 8 ? r.C_spread : 0, r.C_local);
    }
    return 0;
}
