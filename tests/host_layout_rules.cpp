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
    printf("OK %ld\n", cases);
    return 0;
}
