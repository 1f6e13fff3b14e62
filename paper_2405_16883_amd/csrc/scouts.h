// Plan-free SpMM: which rows are long, and which workgroup looks for them (a scout; see spmm_natural_kernel).
// Plain integer arithmetic with no HIP dependency, so that the host tests can compile and check it on the CPU.
#pragma once

#include <stdint.h>

#if defined(__HIPCC__)
#define SCORCH_SCOUTS_HOST_DEVICE __host__ __device__
#else
#define SCORCH_SCOUTS_HOST_DEVICE
#endif

namespace scorch {

constexpr int32_t kNaturalMid = 256;

// Row length beyond which a row is left to a scout: four times the mean, so that such rows are the outliers of a matrix of
// whatever density, and no row that a wavefront walks in four steps.  Every workgroup has the mean from rowptr[m].  Measured
// with the limit at 2 / 4 times the mean, n = 64, every fourth row of 1000 entries, the others nearly empty: 16 384 rows
// 53.1 / 45.6 us; random graphs the same.
SCORCH_SCOUTS_HOST_DEVICE inline int32_t long_row_limit(uint32_t nnz, float one_over_m) {
    const float limit = 4.f * (float)nnz * one_over_m;  // the same on every workgroup
    return limit > 1e9f ? 1000000000 : limit > (float)kNaturalMid ? (int32_t)limit : kNaturalMid;
}
struct Scouts {
    int32_t count;  // workgroups per column tile, at the front of the grid
    int32_t shift;  // they are dealt groups of 2^shift rows
};

// One for 32 rows of a small matrix, and on a large one few enough that they leave room for the others to start beside them:
// with 1021 and more the others wait until the scouts have seen their row pointers (169 343 rows, two column tiles, 2039 / 1021 / 509
// per tile: 142.5 / 140.9 / 137.4 us).  From 524 288 rows on they look at groups of four rows, which share a cache line
// (2 M rows, single rows 728 us, groups 693).  The number is a prime, so that neither rows that are long at a regular
// distance nor neighbouring ones meet on a scout.
inline Scouts scouts_for(int32_t m) {
    Scouts s{1, m < 524288 ? 0 : 2};
    for (const int32_t prime : {3, 7, 13, 31, 61, 127})
        if (m >= 32 * prime) s.count = prime;
    if (m >= 8192) s.count = m < 32768 ? 251 : m < 524288 ? 509 : 1021;
    return s;
}

constexpr uint32_t kScoutStep = 97;  // a prime that is no count: neighbouring rows, and those 64 apart, go to different compute units

// First row of scout b, and the distance from there to the i-th row it looks at (0 <= i < 256); then it goes on 256 * count
// rows further.
SCORCH_SCOUTS_HOST_DEVICE inline int64_t scout_first(uint32_t b, int32_t count, int32_t shift) {
    return (int64_t)((b * kScoutStep) % (uint32_t)count) << shift;
}
SCORCH_SCOUTS_HOST_DEVICE inline int32_t scout_place(int32_t i, int32_t count, int32_t shift) {
    return (i >> shift) * (count << shift) + (i & ((1 << shift) - 1));
}

}  // namespace scorch
