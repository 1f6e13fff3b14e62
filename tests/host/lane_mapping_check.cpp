// CPU check of the lane mapping over sizes, strides and addresses: vectors for aligned rows only where every row of B and C is aligned
// and n is a multiple of the vector, column tiles that cover the n columns, and, in the plan-free call, the scouts' variant for 64-column
// slices only where there are such slices.  Prints "ok <cases>" or the first failure.
#include <cstdio>
#include <initializer_list>

#include "lane_mapping.h"

using namespace scorch;

#define EXPECT(cond)                                                                                                        \
    do {                                                                                                                    \
        if (!(cond)) {                                                                                                      \
            std::printf("line %d: %s (m=%d k=%d n=%d +%d +%d B%+d C%+d)\n", __LINE__, #cond, m, k, n, pb, pc, ob, oc);      \
            return 1;                                                                                                       \
        }                                                                                                                   \
    } while (0)

int main() {
    long cases = 0, slices = 0;
    const char *base = reinterpret_cast<const char *>(1 << 20);
    for (int m : {1, 64, 200, 683, 1000, 1023, 1024, 1500, 2047, 2048, 5000, 100000, 199999, 200000, 400000, 2000000})
        for (int k : {10, 11000, 17000, 200000})
            for (int n : {1, 2, 3, 4, 5, 8, 20, 32, 33, 64, 100, 127, 128, 130, 192, 256, 320, 448, 512, 576, 1000, 1024})
                for (int pb : {0, 1, 2, 4})
                    for (int pc : {0, 3, 4})
                        for (int ob : {0, 4, 8, 16})
                            for (int oc : {0, 12}) {
                                const float *B = reinterpret_cast<const float *>(base + ob);
                                const float *C = reinterpret_cast<const float *>(base + oc);
                                const int64_t ldb = n + pb, ldc = n + pc;
                                const NaturalMapping nm = natural_mapping(m, k, n, B, ldb, C, ldc);
                                const Mapping plain = pick_mapping(n, B, ldb, C, ldc, 0);
                                for (const Mapping &mp : {nm.mp, plain}) {
                                    const int bytes = 4 * mp.V;
                                    const bool aligned = (ldb * 4) % bytes == 0 && (ldc * 4) % bytes == 0 && ob % bytes == 0 && oc % bytes == 0 && n % mp.V == 0;
                                    EXPECT(mp.UA ? mp.V == 4 && n >= 4 : aligned);
                                    EXPECT(mp.V <= n && mp.G >= 1 && mp.G <= kLanes && (mp.G & (mp.G - 1)) == 0);
                                    EXPECT(mp.T == 1 || (mp.T == 2 && mp.G == kLanes && mp.V == 4));
                                    EXPECT((int64_t)mp.G * mp.V * mp.T * mp.ncoltiles >= n);
                                }
                                const bool sliced_variant = nm.scout_gathers == 8 && nm.mp.G != 8;
                                EXPECT(nm.scout_gathers == 8 || nm.scout_gathers == 16);
                                if (sliced_variant) EXPECT(nm.mp.V == 4 && !nm.mp.UA && nm.mp.G == 16 && nm.mp.T == 1 && nm.mp.xcd_slices == 1 && n % 64 == 0);
                                slices += sliced_variant;
                                ++cases;
                            }
    if (slices == 0) {
        std::printf("no case with slices\n");
        return 1;
    }
    std::printf("ok %ld\n", cases);
    return 0;
}
