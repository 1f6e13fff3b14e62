// CPU check of how long rows are cut by columns: buckets of row lengths, and the layout of the pieces, which has to fit its
// capacity, give every piece of every row a place of its own, and take all rows of a length or none.  Prints "ok" or the first failure.
#include <cstdio>
#include <random>
#include <vector>

#include "cut_classes.h"

using namespace scorch;

#define EXPECT(cond)                                             \
    do {                                                         \
        if (!(cond)) {                                           \
            std::printf("line %d: %s\n", __LINE__, #cond);       \
            return 1;                                            \
        }                                                        \
    } while (0)

int main() {
    for (int b = 0; b < kCutBuckets; ++b) {
        EXPECT(cut_bucket(cut_bucket_len(b)) == b);
        if (b > 0) EXPECT(cut_bucket(cut_bucket_len(b) - 1) == b - 1);
    }
    EXPECT(cut_bucket_len(0) == kCutMinLen && cut_bucket(INT32_MAX) == kCutBuckets - 1);
    std::mt19937 rng(1);
    for (int i = 0; i < 100000; ++i) {
        const int32_t m = 1 + (int32_t)(rng() >> (1 + rng() % 30)), k = 1 + (int32_t)(rng() >> (1 + rng() % 30));
        const int64_t nnz = rng() >> (1 + rng() % 30);
        const int finest = (int)(rng() % kCutClasses);
        const int64_t cap = cut_capacity(m, k, nnz, finest);
        EXPECT(cap >= 0 && cap <= nnz / (finest > 0 ? 40 : 16) && cap / kXcds <= INT32_MAX);
        EXPECT(nnz >= kCutAllLong * (int64_t)m ? cap <= (int64_t)m * (kXcds << finest) + nnz / 128 : cap <= ((int64_t)m + k) / 2);
        // rows that are all long and alike are cut whenever the finest division leaves it at 8 pieces for each
        if (nnz >= kCutAllLong * (int64_t)m && finest == 0) {
            int32_t rows[kCutBuckets] = {};
            rows[cut_bucket((int32_t)(nnz / m))] = m;
            CutInfo c{};
            cut_layout(rows, finest, cap, c);
            EXPECT(c.n_rows == m);
        }
    }
    for (int round = 0; round < 3000; ++round) {
        int32_t rows[kCutBuckets];
        for (int b = 0; b < kCutBuckets; ++b) rows[b] = rng() % 3 ? (int32_t)(rng() % 40) : 0;
        const int finest = (int)(rng() % kCutClasses);
        const int64_t cap = rng() % 30000;
        CutInfo c{};
        cut_layout(rows, finest, cap, c);
        EXPECT((int64_t)c.pieces * kXcds <= cap);
        int taken = 0;
        int64_t next = 0;  // pieces of the longest bucket that was left out
        for (int b = 0; b < kCutBuckets; ++b) {
            EXPECT(b == 0 || cut_class(b, finest) >= cut_class(b - 1, finest));
            if (cut_bucket_len(b) >= c.len) taken += rows[b];
            else next = (int64_t)rows[b] << cut_class(b, finest);
        }
        EXPECT(taken == c.n_rows);
        if (c.len > kCutMinLen) EXPECT(((int64_t)c.pieces + next) * kXcds > cap);
        std::vector<char> seen(c.pieces, 0);
        int row = 0;
        for (int j = kCutClasses - 1; j >= 0; --j) {
            EXPECT(c.row_off[j] == row);
            row += c.rows[j];
            for (int s = 0; s < 1 << j; ++s)
                for (int i = 0; i < c.rows[j]; ++i) {
                    const int q = c.piece_off[j] + s * c.rows[j] + i;
                    EXPECT(q >= 0 && q < c.pieces && !seen[q]);
                    seen[q] = 1;
                }
        }
        EXPECT(row == c.n_rows);
        for (char x : seen) EXPECT(x);
    }
    std::printf("ok\n");
    return 0;
}
