// How long rows are cut by columns (spmm_cut.hip): which rows, into how many pieces, and where a piece's partial row
// stands.  Plain integer arithmetic with no HIP dependency, so that the host tests can compile and check it on the CPU.
#pragma once

#include <stdint.h>

#include "xcd_map.h"

namespace scorch {

constexpr int kCutMinLen = 128;  // shorter rows are never cut: a piece per XCD of less than 16 entries costs more than it gives
constexpr int kCutBuckets = 15;  // row lengths from kCutMinLen on, two buckets per power of two; the last holds 16 384 and more
constexpr int kCutClasses = 5;   // class j: 2^j pieces per XCD
constexpr int kCutBounds = kXcds << (kCutClasses - 1);  // finest division of the columns
constexpr int kCutAllLong = 320; // mean row from which all rows are taken to be long: 40 entries for each of 8 pieces
constexpr int kCutBins = 2048;   // column histogram that the division is read off

// Bucket of a row of `len` >= kCutMinLen entries, and the shortest row of a bucket.
SCORCH_HOST_DEVICE inline int cut_bucket(int32_t len) {
    const int e = 31 - __builtin_clz((unsigned)len);
    const int b = 2 * (e - 7) + ((len >> (e - 1)) & 1);
    return b < kCutBuckets ? b : kCutBuckets - 1;
}
SCORCH_HOST_DEVICE inline int32_t cut_bucket_len(int b) { return (2 + (b & 1)) << (6 + b / 2); }

// A row is cut into 2^class pieces per XCD: as many as leave 16 entries per piece in the mean, 2^finest at most, but enough
// for pieces of 256 entries in the mean (a piece is one wavefront's chain).
SCORCH_HOST_DEVICE inline int cut_class(int b, int finest) {
    const int by_reuse = b / 2 < finest ? b / 2 : finest;
    const int by_chain = b / 2 - 3;
    const int j = by_reuse > by_chain ? by_reuse : by_chain;
    return j < 0 ? 0 : (j < kCutClasses ? j : kCutClasses - 1);
}

// What the planner found, in the workspace and in the plan.  Piece (x, s, i) of class j -- XCD x, s-th part of its columns, i-th row of the
// class -- has the index x * pieces + piece_off[j] + s * rows[j] + i, in the order in which the XCDs take them: longest rows first,
// one part of the columns after the other.
struct CutInfo {
    int32_t len;      // rows of at least this many entries are cut (INT32_MAX: none)
    int32_t pieces;   // per XCD
    int32_t n_rows;
    int32_t longest;  // longest piece; beyond `limit` the pieces are not used
    int32_t limit;
    int32_t rows[kCutClasses], row_off[kCutClasses], piece_off[kCutClasses];
    int32_t bound[kCutBounds];  // first column of every part of the finest division
};

// Pieces that there is room for, over all XCDs: as many as cut_class gives at most, but one for 40 stored entries where B is so large that
// an XCD's range of columns is divided (2.4 M nodes, 122 M entries, n = 100: one for 20 / 40 / 64 6659 / 6625 / 6681 us), else one for 16.  A
// piece leaves a row of n floats.  Where not all rows are long there are no more of them than half the rows of B and C together, so that a
// plan takes no more than half of what those take, whatever the lengths turn out to be.
SCORCH_HOST_DEVICE inline int64_t cut_capacity(int32_t m, int32_t k, int64_t nnz, int finest) {
    const int64_t rows = nnz / kCutMinLen < m ? nnz / kCutMinLen : m;
    int64_t cap = rows * (kXcds << finest) + nnz / 128;
    if (cap > nnz / (finest > 0 ? 40 : 16)) cap = nnz / (finest > 0 ? 40 : 16);
    if (nnz < kCutAllLong * (int64_t)m && cap > ((int64_t)m + k) / 2) cap = ((int64_t)m + k) / 2;
    return cap;
}

// Chooses the shortest rows to cut so that their pieces fit `cap_pieces` (over all XCDs), and lays the classes out.
SCORCH_HOST_DEVICE inline void cut_layout(const int32_t (&rows_in)[kCutBuckets], int finest, int64_t cap_pieces, CutInfo &c) {
    int64_t pieces = 0;
    int first = kCutBuckets;
    for (int b = kCutBuckets - 1; b >= 0; --b) {
        pieces += (int64_t)rows_in[b] << cut_class(b, finest);
        if (pieces * kXcds > cap_pieces) break;
        first = b;
    }
    for (int j = 0; j < kCutClasses; ++j) c.rows[j] = 0;
    for (int b = first; b < kCutBuckets; ++b) c.rows[cut_class(b, finest)] += rows_in[b];
    c.len = first < kCutBuckets ? cut_bucket_len(first) : INT32_MAX;
    c.n_rows = c.pieces = 0;
    for (int j = kCutClasses - 1; j >= 0; --j) {
        c.row_off[j] = c.n_rows;
        c.piece_off[j] = c.pieces;
        c.n_rows += c.rows[j];
        c.pieces += c.rows[j] << j;
    }
}

}  // namespace scorch
