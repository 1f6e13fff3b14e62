// CPU check of how the plan-free kernel deals its long rows to workgroups (scouts).  For row counts over the whole range it
// verifies that the scouts together look at every row exactly once, and at none before the first.  Then, for matrices with long rows at
// a regular distance, in a cluster, longest first and in random order, it adds up the entries of the long rows on every
// scout: the busiest may hold no more than its longest row and a few times its even share.
// Prints "ok <cases>" or the first failure.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <vector>

#include "scouts.h"

using namespace scorch;

static int cover(int32_t m) {
    const Scouts s = scouts_for(m);
    if (s.count < 1) { std::printf("m=%d: %d scouts\n", m, s.count); return 0; }
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
static int balance(const char *what, const std::vector<int> &lens) {
    const int32_t m = (int32_t)lens.size();
    long long nnz = 0, longs = 0;
    for (int x : lens) nnz += x;
    const int32_t limit = long_row_limit((uint32_t)nnz, 1.f / (float)m);
    const Scouts s = scouts_for(m);
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
    for (int32_t m = 1; m < 8192; ++m) {
        if (!cover(m)) return 1;
        ++cases;
    }
    for (int32_t m : {8192, 8193, 9999, 16384, 32767, 32768, 32769, 65000, 169343, 524287, 524288, 524289, 3000001}) {
        if (!cover(m)) return 1;
        ++cases;
    }
    for (int32_t m : {2500, 4096, 8192, 16384, 40000, 169343, 600000}) {
        for (int every : {5, 8, 10, 16, 31, 32, 64, 100, 128, 250}) {
            std::vector<int> lens(m, 3);
            for (int32_t r = 0; r < m; r += every) lens[r] = 2000;
            if (!balance("regular", lens)) return 1;
            ++cases;
        }
        std::vector<int> cluster(m, 3), hubs(m), mixed(m);
        for (int32_t r = m / 2; r < m / 2 + m / 16; ++r) cluster[r] = 1000;
        for (int32_t r = 0; r < m; ++r) hubs[r] = (int)std::min(m / 16.0, m / 16.0 * std::pow(r + 1.0, -0.9) + 3);
        for (int32_t r = 0; r < m; ++r) mixed[(int64_t)r * 7919 % m] = hubs[r];
        if (!balance("cluster", cluster) || !balance("longest first", hubs) || !balance("random order", mixed)) return 1;
        cases += 3;
    }
    // the limits: 256, four times the mean; no overflow
    if (long_row_limit(1000, 1e-3f) != 256 || long_row_limit(1000000, 1e-3f) < 3999 || long_row_limit(1000000, 1e-3f) > 4001 ||
        long_row_limit(0x7fffffffu, 1.f) != 1000000000) {
        std::printf("limits\n");
        return 1;
    }
    std::printf("ok %ld\n", cases);
    return 0;
}
