// CPU check of the row tiles a wavefront of the dense layer takes: one or two, by the rounds of the resident wavefronts, but always two where
// the stores decide: short products, a wide result, more than the memory-side cache.  Prints "ok <cases>" or the first failure.
#include <cstdio>
#include <initializer_list>

#include "dense_tiles.h"

using namespace scorch;

#define EXPECT(cond)                                                                                            \
    do {                                                                                                        \
        if (!(cond)) {                                                                                          \
            std::printf("line %d: %s (m=%lld k=%d n=%d)\n", __LINE__, #cond, (long long)m, k, n);               \
            return 1;                                                                                           \
        }                                                                                                       \
    } while (0)

int main() {
    long cases = 0, ones = 0, kept = 0;
    for (int64_t m : {1ll, 15ll, 16ll, 17ll, 2000ll, 65536ll, 65537ll, 169343ll, 291683ll, 350000ll, 565655ll, 600000ll, 1500000ll, 2147483647ll})
        for (int k : {1, 15, 16, 17, 25, 33, 47, 48, 64, 100, 128, 144})
            for (int n : {1, 16, 48, 49, 53, 64, 75, 99, 100, 128, 144, 200, 208, 256, 2147483647})
                for (int64_t resident : {0ll, 8ll, 2048ll, 4096ll}) {
                    const int rt = dense_row_tiles(m, k, n, resident);
                    EXPECT(rt == 1 || rt == 2);
                    if (k >= 16 && k < 48 && n >= (k == 16 ? 49 : 100) && (double)m * ((double)k + n) * 4 > 256.0 * 1048576) {
                        EXPECT(rt == 2);
                        ++kept;
                    } else if (resident > 0) {
                        const int64_t one = ((m + 15) / 16 + resident - 1) / resident, two = ((m + 31) / 32 + resident - 1) / resident * 2;
                        EXPECT((rt == 2) == (two * 100 <= one * 104));
                        ones += rt == 1;
                    }
                    ++cases;
                }
    if (ones == 0 || kept == 0) {
        std::printf("one side of the rule was not met\n");
        return 1;
    }
    std::printf("ok %ld\n", cases);
    return 0;
}
