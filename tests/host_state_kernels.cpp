// For each "d B H tokens rope layout" on the command line (rope none, table or axes; layout bhnd or bnhd), the bf16 state kernel of d = 112
// and 128 that serves the call on 256 compute units (csrc/layout_rules.hpp) and its chunks per head.
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "../paper_2509_24695_amd/csrc/layout_rules.hpp"

int main(int argc, char **argv)
{
    for (int i = 1; i + 5 < argc; i += 6) {
        const int d = atoi(argv[i]), B = atoi(argv[i + 1]), H = atoi(argv[i + 2]), n = atoi(argv[i + 3]);
        const bool table = !strcmp(argv[i + 4], "table"), axes = !strcmp(argv[i + 4], "axes"), token_major = !strcmp(argv[i + 5], "bnhd");
        const sv::TokenLayout t = token_major ? sv::TokenLayout{B * H, H, d, 2, d, (int64_t)H * d} : sv::TokenLayout{B * H, H, d, 2, (int64_t)n * d, d};
        int C = sv::quad_state_chunks(B * H, d, n, table, axes, 256);
        const char *kernel = "quad";
        if (C == 0) {
            C = sv::plan_chunks(B * H, n, sv::kWideWgTokens, 256);
            kernel = sv::coop_state_serves(t, n, C, table, axes) ? "coop" : "rows";
        }
        printf("%s %d\n", kernel, C);
    }
    return 0;
}
