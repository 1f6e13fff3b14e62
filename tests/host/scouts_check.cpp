// CPU check of how the plan-free kernel deals its long rows to workgroups (scouts).  For row counts, run lengths and numbers
// of column tiles over the whole range it verifies that
//   * the scouts together look at every row exactly once, and at none past the end,
//   * a scout that takes runs of rows as well is one of the workgroups that take them.
// Then, for matrices with long rows at a regular distance, in a cluster, longest first and in random order, it adds up the entries of
// the long rows on every scout: the busiest may hold no more than its longest row and a few times its even share.
// Prints "ok <cases>" or the first failure.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <vector>

#include "scouts.h"

using namespace scorch;

static int cover(int32_t m, int32_t run_blocks, int32_t tiles) {
    const Scouts s = scouts_for(m, run_blocks, tiles);
    if (s.count < 1 || (!s.beside && s.count > run_blocks)) { std::printf("m=%d: %d scouts of %d workgroups\n", m, s.count, run_blocks); return 0; }
    std::vector<unsigned char> seen(m, 0);
    for (int32_t b = 0; b < s.count; ++b)
        for (int64_t first = scout_first(b, s.count, s.shift); first < m; first += 256 * (int64_t)s.count)
            for (int i = 0; i < 256; ++i) {
                const int64_t row = first + scout_place(i, s.count, s.shift);
                if (row < 0) { std::printf("m=%d row %lld\n", m, (long long)row); return 0; }
                if (row < m && seen[row]++) { std::printf("m=%d count=%d: row %lld twice\n", m, s.count, (long long)row); return 0; }
            }
    for (int32_t r = 0; r < m; ++r)
        if (!seen[r]) { std::printf("m=%d count=%d: row %d never\n", m, s.count, r); return 0; }
    return 1;
}

// Entries of long rows on the busiest scout against the longest row and the even share.
static int balance(const char *what, const std::vector<int> &lens, int32_t run_blocks, int32_t tiles) {
    const int32_t m = (int32_t)lens.size();
    long long nnz = 0, longs = 0;
    for (int x : lens) nnz += x;
    const int32_t limit = long_row_limit((uint32_t)nnz, (uint32_t)m);
    const Scouts s = scouts_for(m, run_blocks, tiles);
    long long busiest = 0, longest = 0;
    for (int32_t b = 0; b < s.count; ++b) {
        long long sum = 0;
        for (int64_t first = scout_first(b, s.count, s.shift); first < m; first += 256 * (int64_t)s.count)
            for (int i = 0; i < 256; ++i) {
                const int64_t row = first + scout_place(i, s.count, s.shift);
                if (row < m && lens[row] > limit) {
                    sum += lens[row];
                    longest = std::max<long long>(longest, lens[row]);
                }
            }
        busiest = std::max(busiest, sum);
        longs += sum;
    }
    // groups of 2^shift neighbours go to one scout, and a matrix of m rows with one long row in `count` is uneven by one row
    if (busiest > (longest << s.shift) + 3 * (longs / s.count)) {
        std::printf("%s, %d rows: %lld entries on one of %d scouts, longest row %lld, even share %lld\n", what, m, busiest, s.count, longest, longs / s.count);
        return 0;
    }
    return 1;
}

int main() {
    long cases = 0;
    for (int32_t blocks = 1; blocks <= 2100; ++blocks)  // every number of scouts
        for (int32_t m : {1, blocks * 4 - 3, blocks * 4, blocks * 64}) {
            if (!cover(m, blocks, 1)) return 1;
            ++cases;
        }
    for (int32_t m : {524287, 524288, 524289, 3000001})
        for (int32_t tiles : {1, 2, 16}) {
            if (!cover(m, m / 16, tiles)) return 1;
            ++cases;
        }
    for (int32_t m : {300, 1000, 2500, 4096, 16384, 40000, 169343, 600000})
        for (int32_t run : {4, 8, 16, 64})  // rows of a workgroup: 4, and up to 64 with 8192 rows for each four
            for (int32_t tiles : {1, 2, 4}) {
                if (run > 4 && m < 1024 * run) continue;
                const int32_t blocks = (m + run - 1) / run;
                for (int every : {5, 8, 10, 16, 31, 32, 64, 100, 128, 250}) {
                    std::vector<int> lens(m, 3);
                    for (int32_t r = 0; r < m; r += every) lens[r] = 2000;
                    if (!balance("regular", lens, blocks, tiles)) return 1;
                    ++cases;
                }
                std::vector<int> cluster(m, 3), hubs(m), mixed(m);
                for (int32_t r = m / 2; r < m / 2 + m / 16; ++r) cluster[r] = 1000;
                for (int32_t r = 0; r < m; ++r) hubs[r] = (int)std::min(m / 16.0, m / 16.0 * std::pow(r + 1.0, -0.9) + 3);
                for (int32_t r = 0; r < m; ++r) mixed[(int64_t)r * 7919 % m] = hubs[r];
                if (!balance("cluster", cluster, blocks, tiles) || !balance("longest first", hubs, blocks, tiles) ||
                    (m % 7919 != 0 && !balance("random order", mixed, blocks, tiles)))
                    return 1;
                cases += 3;
            }
    std::printf("ok %ld\n", cases);
    return 0;
}
