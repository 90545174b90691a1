// csrc/layout_rules.hpp against the statements it stands for, computed without its arithmetic.
#include <cstdio>
#include <initializer_list>

#include "../paper_2509_24695_amd/csrc/layout_rules.hpp"

int main()
{
    long cases = 0;
    const __int128 limit = (__int128)1 << 31;
    for (int e : {2, 4})
        for (long N : {1L, 63L, 64L, 65L, 1024L, 32760L, 65533L, 65535L, 65536L, 75600L, 1000003L, 33554431L})
            for (long base : {64L, 4096L, 7168L, 16384L, 1L << 22, 1L << 23, 1L << 24, 1L << 25, 1L << 40, (1L << 62) / 64})
                for (long off = -64; off <= 64; off += 8) {
                    long stride = base + off;
                    for (int exact = 0; exact < 2; ++exact) {     // and the strides around the limit itself
                        if (exact) stride = (long)(limit / ((__int128)(N > 64 ? N : 64) * e)) / 8 * 8 + off;
                        if (stride < 32) continue;
                        const bool want = (__int128)(N > 64 ? N : 64) * stride * e < limit;
                        if (sv::head_offsets_fit(N, stride, e) != want) return printf("FAIL fit N=%ld stride=%ld e=%d\n", N, stride, e), 1;
                        ++cases;
                    }
                }
    // the order rules at their lines
    using sv::TokenLayout;
    const int both = sv::kOrderChunkMajor | sv::kOrderLockstep, ls = sv::kOrderLockstep, cm = sv::kOrderChunkMajor;
    auto tm = [](int B, int H, int d, int e) { return TokenLayout{B * H, H, d, e, d, (int64_t)H * d}; };       // [B][N][H][d]
    auto hm = [](int B, int H, int d, int e) { return TokenLayout{B * H, H, d, e, 1000 * d, d}; };              // [B][H][N][d]
    struct Want { TokenLayout t; bool table, factored; int n, state, apply; } want[] = {
        {hm(2, 32, 64, 2), false, false, 20000, 0, 0}, {hm(2, 32, 64, 2), true, false, 20000, 0, 0},
        {hm(2, 20, 112, 2), true, false, 20000, cm, 0}, {hm(2, 20, 128, 4), true, false, 20000, 0, 0},
        {tm(1, 1, 64, 2), false, false, 20000, 0, 0},
        {tm(4, 3, 64, 2), false, false, 20000, both, ls}, {tm(1, 13, 64, 2), false, false, 20000, ls, ls},
        {tm(2, 32, 64, 2), false, false, 12287, ls, ls}, {tm(2, 32, 64, 2), false, false, 12288, ls, both},
        {tm(2, 32, 64, 2), false, true, 20000, ls, ls}, {tm(2, 32, 64, 2), true, false, 5, ls, both},
        {tm(4, 32, 64, 2), false, false, 20000, ls, ls}, {tm(1, 96, 64, 2), false, false, 20000, ls, both},
        {tm(1, 20, 112, 2), false, true, 5, both, both}, {tm(1, 20, 128, 2), false, false, 5, ls, ls},
        {tm(1, 20, 128, 2), true, false, 5, both, ls}, {tm(1, 20, 32, 2), false, false, 5, both, both},
        {tm(1, 20, 64, 4), true, false, 5, ls, ls}, {tm(1, 20, 32, 4), false, false, 5, both, both},
    };
    for (const Want &w : want) {
        const int s = sv::state_order(w.t, w.table), a = sv::apply_order(w.t, w.table, w.factored, w.n);
        if (s != w.state || a != w.apply) return printf("FAIL order BH=%d H=%d d=%d e=%d n=%d: %d %d\n", w.t.BH, w.t.H, w.t.d, w.t.elem_bytes, w.n, s, a), 1;
        ++cases;
    }
    // fp32 states of d = 112 and 128: no running sum of a head's only workgroup takes more than 16 tokens (tiles of 8 tokens dealt to two groups of four
    // waves, a quadrant of the state to each; two sums per wave, taken in turn)
    auto longest = [](int n) {
        const int tiles = (n + 7) / 8, share = (tiles + 1) / 2;
        return 8 * ((share + 1) / 2);
    };
    for (int d : {112, 128})
        for (int BH = 1; BH <= 300; ++BH)
            for (int n = 1; n <= 400; ++n) {
                if (n > sv::f32_sole_tokens(d, BH, 4, false) && n > sv::f32_sole_tokens(d, BH, 4, true)) continue;
                if (longest(n) > 16) return printf("FAIL sole d=%d BH=%d n=%d\n", d, BH, n), 1;
                ++cases;
            }
    // d = 32 and 64: layers on one workgroup per head and on several, one's time less the other's (0.1 us, the slower of two devices where both
    // were measured): the rule takes the faster one
    struct Layer { int d, BH, bytes; bool rotated; int n, tenths; } layers[] = {
        {32, 2, 4, false, 1024, -12}, {32, 2, 4, false, 1536, 14}, {32, 16, 4, false, 768, -11}, {32, 16, 4, false, 1152, 17}, {32, 12, 4, false, 1024, 18},
        {32, 32, 4, false, 512, -22}, {32, 32, 4, false, 896, 12}, {32, 64, 4, false, 512, -7}, {32, 128, 4, false, 768, -23},
        {32, 2, 4, true, 512, -19}, {32, 2, 4, true, 1152, 32}, {32, 16, 4, true, 1024, 38}, {32, 8, 4, true, 512, -4}, {32, 32, 4, true, 384, -12},
        {32, 32, 4, true, 896, 27}, {32, 64, 4, true, 768, 7}, {32, 2, 2, false, 1024, -17}, {32, 16, 2, false, 896, -14}, {32, 16, 2, false, 1280, 12},
        {32, 16, 2, true, 768, -7}, {32, 16, 2, true, 1280, 40}, {32, 32, 2, true, 512, -22}, {32, 32, 2, true, 1024, 22}, {32, 64, 2, true, 896, 18},
        {64, 8, 4, false, 192, -7}, {64, 2, 4, false, 320, 6}, {64, 16, 4, true, 256, 18}, {64, 64, 4, true, 192, -9}};
    for (const Layer &l : layers) {
        if ((l.n <= sv::f32_sole_tokens(l.d, l.BH, l.bytes, l.rotated)) != (l.tenths < 0)) return printf("FAIL line d=%d BH=%d n=%d\n", l.d, l.BH, l.n), 1;
        ++cases;
    }
    // ... of the heads that several workgroups share, layers with their partial states added up by a launch and by the last workgroup, enqueued call by call: the rule takes the faster one
    struct Shared { int d, BH, C; double launch, last; } shared[] = {
        {32, 128, 2, 33.4, 32.4}, {32, 32, 8, 15.9, 15.4}, {32, 16, 16, 12.4, 12.3}, {32, 2, 32, 10.5, 11.3}, {64, 1, 4, 16.1, 14.9}, {64, 8, 4, 16.0, 15.2}, {64, 32, 4, 17.0, 16.1},
        {64, 48, 4, 16.6, 16.4}, {64, 64, 4, 38.9, 37.8}, {64, 128, 2, 63.3, 61.1}, {64, 32, 8, 18.0, 19.5}, {112, 64, 4, 0, 1}, {128, 128, 2, 0, 1}};
    for (const Shared &l : shared) {
        if (sv::f32_last_folds(l.d, l.C) != (l.last < l.launch)) return printf("FAIL fold d=%d BH=%d C=%d\n", l.d, l.BH, l.C), 1;
        ++cases;
    }
    printf("OK %ld\n", cases);
    return 0;
}
