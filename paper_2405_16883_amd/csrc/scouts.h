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
// 53.1 / 45.6 us, 4096 rows 20.6 / 19.8; random graphs the same.
SCORCH_SCOUTS_HOST_DEVICE inline int32_t long_row_limit(uint32_t nnz, uint32_t m) {
    const uint32_t mean = nnz / m;
    const int32_t limit = 4 * (int32_t)(mean < (1u << 28) ? mean : 1u << 28);
    return limit > kNaturalMid ? limit : kNaturalMid;
}

constexpr uint32_t kScoutStep = 97;  // a prime that is no count: neighbouring rows, and those 64 apart, go to different compute units

struct Scouts {
    int32_t count;
    int32_t shift;  // they are dealt groups of 2^shift rows
    bool beside;    // they are workgroups of their own, at the front of the grid; otherwise the first ones of the others
};

// run_blocks: workgroups that take the rows in runs, per column tile.
//
// Where all workgroups are resident at once it does not matter who starts first, and those that are there look as well.
// Otherwise the scouts come first, about as many as the chip holds at once (four per compute unit), over the column tiles:
// every one has to be started, 2 ns each (169 343 rows, two column tiles, 2039 / 1021 / 509 per tile: 142.5 / 140.9 / 137.4 us).
// From 524 288 rows on they look at groups of four rows, which share a cache line (2 M rows, single rows 728 us, groups 693).
// The number is a prime, so that neither rows that are long at a regular distance nor neighbouring ones meet on a scout.
inline Scouts scouts_for(int32_t m, int32_t run_blocks, int32_t coltiles) {
    if ((int64_t)run_blocks * coltiles > 2048) return Scouts{coltiles == 1 ? 1021 : 509, m < 524288 ? 0 : 2, true};
    int32_t count = run_blocks < 2039 ? run_blocks : 2039;
    for (int32_t d = 2; d * d <= count;) {
        if (count % d == 0 || count == (int32_t)kScoutStep) {
            --count;
            d = 2;
        } else {
            ++d;
        }
    }
    return Scouts{count, 0, false};
}

// First row of scout b, and the distance from there to the i-th row it looks at (0 <= i < 256); then it goes on 256 * count
// rows further.
SCORCH_SCOUTS_HOST_DEVICE inline int64_t scout_first(uint32_t b, int32_t count, int32_t shift) {
    return (int64_t)((b * kScoutStep) % (uint32_t)count) << shift;
}
SCORCH_SCOUTS_HOST_DEVICE inline int32_t scout_place(int32_t i, int32_t count, int32_t shift) {
    return (i >> shift) * (count << shift) + (i & ((1 << shift) - 1));
}

}  // namespace scorch
