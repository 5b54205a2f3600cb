// Which rows a workgroup of the sparse product takes.  No HIP here, so that the
// schedule can be checked on the host.
#pragma once
#include <algorithm>
#include <cstdint>

namespace gplhr {

struct SpmmShape {
    int lpr;        // lanes per row
    int inv;        // ceil(65536 / lpr): lane / lpr as a multiplication
    int rpw;        // rows per wavefront
    int rpb;        // rows per workgroup
    int sp;         // >0: plane-slab row schedule with planes of sp rows; 0: natural order
    int ss;         // slab: sp / 8 rows of each plane
    int nbs;        // workgroups per slab of a plane; natural order: per eighth
    int order;      // natural order: SPMM_EIGHTHS, SPMM_TURN or SPMM_CHECK
};
// The eighths of the rows, one to an XCD; the rows in turn; or whichever the row
// pointers ask for.
enum : int { SPMM_EIGHTHS, SPMM_TURN, SPMM_CHECK };
struct SpmmRows {
    int64_t row0;
    int nr;         // <= 0: none
};

// The rows of workgroup blk: XCD x is workgroups x, x + 8, ...
constexpr SpmmRows spmm_plane_rows(const SpmmShape &s, uint32_t blk) {
    // XCD x takes slab x of every plane, planes in order
    const uint32_t x = blk & 7, k = blk >> 3, z = k / (uint32_t)s.nbs;
    const int i = (int)(k - z * s.nbs) * s.rpb;
    return {(int64_t)z * s.sp + (int64_t)x * s.ss + i, s.rpb < s.ss - i ? s.rpb : s.ss - i};
}
// eighths: XCD x takes the x-th eighth of the rows, else the rows go in turn
constexpr SpmmRows spmm_natural_rows(const SpmmShape &s, int64_t n, uint32_t blk, bool eighths) {
    const int64_t k = eighths ? (int64_t)(blk & 7) * s.nbs + (blk >> 3) : (int64_t)blk;
    const int64_t row0 = k * s.rpb, left = n - row0;
    return {row0, left < s.rpb ? (int)left : s.rpb};
}

// Natural order: may XCD x take the x-th eighth (nbs workgroups)?  The products end
// when the XCD with the most entries does, so only where no eighth has more than a
// sixteenth above the mean.  Dealt in turn, the rows load the XCDs evenly whatever
// their order, but each XCD fetches nearly every block row of a banded pattern.
// Before the rule, always by eighths (us, eighths / in turn): 262144 rows, the first
// eighth of 65 entries, the others of 5, 16 complex64 columns 225 / 68; rows sorted by
// length, 1 to 40 entries, 10 complex128 columns 286 / 196; 10 to 14 entries in a
// band, rising (an eighth with 15 % above the mean): 29 / 41 and with 64 complex128
// columns 304 / 288; even bands of 7 entries 18 / 30.
constexpr bool spmm_even(int32_t most, int32_t total) {   // entries of the fullest eighth, of all
    return most <= total / 8 + total / 128;
}

// The shape for b columns, cols of them per lane.  row_len: typical entries of a row;
// stage: entries a wavefront can stage; cut: fewer rows to a wavefront may bring them
// there.  grid: workgroups.
inline SpmmShape spmm_shape(int64_t n, int b, int cols, int plane, int64_t row_len, int stage, bool cut,
                            int64_t &grid) {
    SpmmShape s{};
    s.lpr = (b + cols - 1) / cols;
    s.inv = (65536 + s.lpr - 1) / s.lpr;
    s.rpw = 64 / s.lpr;
    // fewer rows per wavefront where that brings its entries (and a quarter more, as
    // rows differ) into the stage and keeps half of the lanes; not with few, wide rows
    const int64_t fit = (int64_t)stage * 4 / (5 * std::max<int64_t>(row_len, 1));
    if (cut && s.rpw > 4 && s.rpw > fit && 2 * fit >= s.rpw) s.rpw = (int)fit;
    s.rpb = 4 * s.rpw;
    // a plane whose slabs are less than four workgroups' rows would leave lanes idle at
    // their ends; three of it fit an L2 whole, so that the natural order serves it as
    // well (us, slabs / natural order: planes of 512 rows of 5 entries, complex64, 1
    // column 12.6 / 8.7, 5 columns 21.3 / 16.3; of 4096 rows of 7 entries, 2 columns
    // 8.1 / 7.2; at four workgroups' rows, planes of 512, 16 complex128 78.5 / 86.3)
    s.sp = plane / 8 < 4 * s.rpb ? 0 : plane;
    if (s.sp > 0) {
        // workgroups stay within a slab and share its rows evenly
        s.ss = plane / 8;
        s.nbs = (s.ss + s.rpb - 1) / s.rpb;
        s.rpb = (s.ss + s.nbs - 1) / s.nbs;
        s.rpw = (s.rpb + 3) / 4;
        grid = (int64_t)8 * s.nbs * (n / plane);
    } else {
        s.nbs = (int)((n + 8 * (int64_t)s.rpb - 1) / (8 * (int64_t)s.rpb));
        grid = 8 * (int64_t)s.nbs;
        // Up to one workgroup per CU all run at once, however the rows differ.  With
        // one row to a wavefront the check costs more than the eighths bring (262144
        // rows of 7 entries in a band, 33 complex64 columns: in turn 96 us, by eighths
        // 89, checked 103).  (The check counts rows in 32 bits.)
        s.order = grid <= 256 ? SPMM_EIGHTHS : s.rpw < 2 || n >= (int64_t)1 << 31 ? SPMM_TURN : SPMM_CHECK;
    }
    return s;
}

// The shape of one launch, which has less than 2^32 threads: where planes and lanes
// would ask for more workgroups (tiny planes, wide blocks of 10^8 rows), as few as the
// rows allow, `most` columns to a lane (cols is what it then runs with) and, for the
// last few, not by eighths.  grid = 0: more rows than one launch takes.
inline SpmmShape spmm_launch_shape(int64_t n, int b, int &cols, int most, int plane, int64_t row_len, int stage,
                                   bool cut, int64_t &grid) {
    constexpr int64_t limit = (int64_t)1 << 24;
    SpmmShape s = spmm_shape(n, b, cols, plane, row_len, stage, cut, grid);
    if (grid < limit) return s;
    cols = most;
    s = spmm_shape(n, b, cols, 0, row_len, stage, false, grid);
    if (grid < limit) return s;
    s.order = SPMM_TURN;
    grid = (n + s.rpb - 1) / s.rpb;
    if (grid >= limit) grid = 0;
    return s;
}

}  // namespace gplhr
