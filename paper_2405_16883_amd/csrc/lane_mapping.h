// How the columns of C are laid over the lanes of a wavefront: floats per load, lanes per group, column tiles.  A function of the
// sizes, strides and addresses alone, with no HIP dependency, so that the host tests can compile and check it on the CPU.
#pragma once

#include <stdint.h>

#include "xcd_map.h"

namespace scorch {

constexpr int kLanes = 64;

struct Mapping {
    int V, G, T, ncoltiles;
    bool UA;  // four floats per lane at float alignment, last vector of a row moved back to end at column n
    int xcd_slices;  // 0: tile-major grid; 1: column slices dealt over the XCDs (see tile_of_workgroup)
};

inline Mapping pick_mapping(int32_t n, const float *B, int64_t ldb, const float *C, int64_t ldc, int slice_cols) {
    Mapping mp{};
    const uintptr_t pb = reinterpret_cast<uintptr_t>(B), pc = reinterpret_cast<uintptr_t>(C);
    if (n % 4 == 0 && ldb % 4 == 0 && ldc % 4 == 0 && pb % 16 == 0 && pc % 16 == 0) mp.V = 4;
    else if (n >= 4) {
        // rows that are not 16-byte aligned, or n not a multiple of 4: still four floats per lane
        mp.V = 4;
        mp.UA = true;
    } else if (n % 2 == 0 && ldb % 2 == 0 && ldc % 2 == 0 && pb % 8 == 0 && pc % 8 == 0) mp.V = 2;
    else mp.V = 1;
    mp.xcd_slices = 0;
    if (slice_cols > 0 && mp.V == 4 && !mp.UA) {
        // column slices of B (32 columns = one 128-byte line of a row, or 64 or 128), one slice per XCD at a time
        mp.G = slice_cols / 4;
        mp.T = 1;
        mp.ncoltiles = (n + slice_cols - 1) / slice_cols;
        mp.xcd_slices = 1;
        return mp;
    }
    const int lanes = (n + mp.V - 1) / mp.V;
    if (lanes <= kLanes) {
        // n <= 4 (SpMV and its neighbours): one lane per group, the 64 lanes of a wavefront take 64 entries
        // of a row (or 64 short rows of a window) per step and are combined by the xor butterfly
        int g = 1;
        while (g < lanes) g <<= 1;
        mp.G = g;
        mp.T = 1;
        mp.ncoltiles = 1;
    } else {
        mp.G = kLanes;
        mp.T = 2;
        const int tw = mp.G * mp.V * mp.T;
        mp.ncoltiles = (n + tw - 1) / tw;
    }
    return mp;
}

// The plan-free call's mapping, and which kernel it takes.
struct NaturalMapping {
    Mapping mp;
    bool row_kernel;     // a workgroup per row and 32-column tile
    int64_t row_units;   // so many pairs of these
    int scout_gathers;   // gathers in flight per group of a scout
};

inline NaturalMapping natural_mapping(int32_t m, int32_t k, int32_t n, const float *B, int64_t ldb, const float *C, int64_t ldc) {
    // Column slices dealt over the XCDs (tile_of_workgroup) need no plan, only the shape: with B of 8 MB or more every
    // XCD walks all rows for one slice of columns at a time, so that the part of B it gathers from is 1/s of B.  Measured
    // on the plan-free call: uniform 1 % pattern, n = 128: 90 -> 69 us with 64-column slices; pruned 4096 x 16384 weight,
    // n = 2048: 5.03 -> 2.26 ms with 128-column slices (64 columns: 3.0 ms, 32: 4.3 ms, 256: 4.2 ms); mid-size graph,
    // n = 128: 168 -> 166 us.  A ragged last slice costs more than it gains, hence the multiples.
    int slice_cols = 0;
    if ((int64_t)k * n * 4 >= (8ll << 20)) {
        if (n >= 256 && n % 128 == 0) slice_cols = 128;
        else if (n >= 128 && n % 64 == 0) slice_cols = 64;
    }
    NaturalMapping nm{};
    Mapping &mp = nm.mp;
    mp = pick_mapping(n, B, ldb, C, ldc, slice_cols);
    // Few rows, up to 2048 pairs of a row and a 32-column tile: a workgroup for each pair (spmm_row_kernel).  Measured with
    // n = 256: 64 rows of 2458 entries 62.0 -> 11.7 us, 16 rows of 6000 66 -> 8.8, 256 rows (2048 pairs) of 5000 71 -> 58,
    // of 1000 even; with twice the pairs the run kernel is ahead for long rows (256 rows of 5000, n = 512: 98 against 114).
    const int row_tile = 8 * mp.V;
    nm.row_units = (int64_t)m * ((n + row_tile - 1) / row_tile);
    nm.row_kernel = nm.row_units <= 2048;
    // More rows than that, but fewer than two wavefronts per SIMD at one row each: narrower column tiles, at least 8
    // lanes wide (1024 rows, n = 128, mean 1024 / 256 entries: one tile 32.4 / 16.6 us, two 21.0 / 10.7, four 26.1 / 10.6).
    while (!nm.row_kernel && mp.G * mp.T > 8 && (int64_t)m * mp.ncoltiles < 2048) {
        if (mp.T == 2) mp.T = 1;
        else mp.G /= 2;
        mp.ncoltiles = (n + mp.G * mp.V - 1) / (mp.G * mp.V);
        mp.xcd_slices = 1;
    }
    // Gathers in flight per group of a scout: 16, which takes 84 to 124 VGPRs, or 8, which leaves room for one or two more wavefronts
    // per SIMD (2.7 -> 3.3 on the mid-size graph, n = 128).  More wavefronts hide more latency, and share the L2s with more rows of B: which
    // counts for more was measured, us with 16 / 8.  Groups of 8 lanes, 169 343 rows, n = 32 49.6 / 41.4.  64-column slices, rows of 15: 30 000
    // rows, n = 128 29.1 / 28.6, 100 000 76.5 / 70.4, 195 000 149 / 140, 250 000 200 / 199, 400 000 320 / 328; n = 192 130 000 rows 145 / 137, 169 343
    // 191 / 192, 250 000 311 / 321; n = 320 79 000 rows 136 / 128, 250 000 506 / 500; n = 448 56 000 rows 136 / 121; rows of 6 5 to 16 % less, of 40 0 to 3 %.
    // The line lies between the last gains and the first losses of n = 128 and 192; wider B still gains beyond it.  Whole rows, 30 000
    // rows, n = 64 23.2 / 25.9.
    // Slices were asked for by the shape alone: rows that are not aligned have none, and keep the loads for any alignment.
    const bool slices_of_64 = slice_cols == 64 && mp.V == 4 && !mp.UA && mp.G == 16 && mp.T == 1;
    nm.scout_gathers = mp.G == 8 || (slices_of_64 && (int64_t)m * mp.ncoltiles < 400000) ? 8 : 16;
    return nm;
}

}  // namespace scorch
