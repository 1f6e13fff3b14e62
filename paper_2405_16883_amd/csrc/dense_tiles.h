// How many 16-row tiles a wavefront of the dense layer (dense_tall.hip) takes.  Plain integer arithmetic with no HIP dependency, so that
// the host tests can compile and check it on the CPU.
#pragma once

#include <algorithm>
#include <stdint.h>

namespace scorch {

constexpr int64_t kDenseCacheFloats = 64ll << 20;  // memory-side cache

// m x k times k x n in `parts` parts of n, `resident` wavefronts of each at a time.
// Two tiles (each fragment of W out of LDS feeds both) unless one gives fewer rounds of the resident wavefronts, with 4 % for the second
// reading of W.  us with two from 1024 units of two on / now: 169 343 rows (1.3 rounds of two or 2.6 of one) 128 -> 128 62.7 / 56.5, 64 -> 128
// 39.8 / 33.9, 40 -> 100 32.1 / 26.4; 60 000 rows 64 -> 128 18.9 / 16.6; 1 M rows 128 -> 128 318 / 306 (and 337 / 342 with two / one).
// Where X and Y do not fit the memory-side cache and the product of a row is short against its stores (up to three steps of 16 columns, the
// last not full, and 100 columns of Y; or 16 -> 49 and more), the stores decide, and a wavefront with two tiles writes twice as much side by side.  us
// with two / one, although one has fewer rounds: 16 -> 53 1 368 044 rows 129 / 146, 16 -> 128 573 630 98 / 116, 20 -> 128 97 / 117, 25 -> 208 330 557 94 / 107,
// 25 -> 400 200 002 97 / 122, 32 -> 240 743 413 236 / 295, 33 -> 100 565 655 96 / 107, 40 -> 128 447 690 88 / 101, 44 -> 128 445 694 93 / 104 (over 33 such widths
// and 150 row counts 0.80 to 1.04).  By the rounds: less than the cache holds (25 -> 208, 282 622 rows, 251 MB 59 / 55), narrower Y (20 -> 64, 1 236 259 130 / 114;
// 32 -> 64, 957 334 112 / 100), longer products (48 -> 144, 541 527 155 / 146; 64 -> 192, 670 984 213 / 206; 48 -> 200, 614 308 214 / 235 is the exception), and
// fewer than 16 columns of X, which are even.  Behind by the rounds: 16 -> 64 at 200 to 250 MB (693 444 rows 36.5 / 37.9).
inline int dense_row_tiles(int64_t m, int32_t k, int32_t n, int64_t resident) {
    if (m * ((int64_t)k + n) > kDenseCacheFloats && ((k >= 16 && k < 48 && n >= 100) || (k == 16 && n > 48))) return 2;
    const int64_t waves = std::max<int64_t>(1, resident);
    auto rounds = [&](int t) { return ((m + 16 * t - 1) / (16 * t) + waves - 1) / waves * t; };
    return 100 * rounds(2) <= 104 * rounds(1) ? 2 : 1;
}

}  // namespace scorch
