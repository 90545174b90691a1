// The flags of the one-launch block step of d = 112 and 128 (csrc/tile_walk.hpp, csrc/layout_rules.hpp): heads on one die store theirs into that die's L2, spread
// heads poll theirs across dies; wherever the workspace starts, no 128-byte line holds both, no word has two meanings and none is past the head's own.
#include <algorithm>
#include <cstdio>
#include <map>
#include <set>

#include "../paper_2509_24695_amd/csrc/layout_rules.hpp"

int main()
{
    long mixed = 0;
    for (int d : {112, 128})
        for (int BH = 8; BH <= 128; ++BH)
            for (int n : {65, 700, 1792, 4680, 100000})
                for (uint64_t base = 4096; base < 4096 + 128; base += 16) {
                    const sv::TokenLayout t{BH, BH, d, 2, (int64_t)n * d, d};
                    const sv::WideRoles r = sv::wide_roles(t, n, (n + 63) / 64, false, 256, 8, base);
                    if (!r.dies) return printf("FAIL none BH=%d\n", BH), 1;
                    if (BH % 8 == 0 && r.C_local != std::min({256 / BH, (n + 63) / 64, sv::kMaxChunks})) return printf("FAIL fewer BH=%d n=%d\n", BH, n), 1;
                    const int locals = r.dies * r.per_die;
                    std::map<uint64_t, int> lines;                     // line -> 1: local, 2: spread
                    std::set<uint64_t> words;
                    for (int bh = 0; bh < BH; ++bh) {
                        const bool local = bh < locals;
                        const int C = local ? r.C_local : r.C_spread;
                        for (int phase = 0; phase < 2; ++phase)
                            for (int c = 0; c < C; ++c) {
                                const int w = sv::wide_flag_word(local, phase, c, C, sv::kMaxChunks);
                                if (w < 0 || w >= 2 * sv::kMaxChunks) return printf("FAIL word BH=%d\n", BH), 1;
                                const uint64_t at = base + ((uint64_t)bh * 2 * sv::kMaxChunks + w) * 8;
                                if (!words.insert(at).second) return printf("FAIL twice BH=%d\n", BH), 1;
                                lines[at / 128] |= local ? 1 : 2;
                            }
                    }
                    for (const auto &l : lines)
                        if (l.second == 3) return printf("FAIL line BH=%d d=%d n=%d base=%d C=%d\n", BH, d, n, (int)(base % 128), r.C_local), 1;
                    mixed += locals < BH;
                }
    printf("OK %ld\n", mixed);
    return 0;
}
