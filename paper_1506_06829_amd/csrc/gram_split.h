// Row blocks of a Gram and the scratch their partials take.  No HIP here, so that
// the rules can be checked on the host.
#pragma once
#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace gplhr {

constexpr int gram_units(int w) { return (w + 7) / 8; }

// Up to 1024 rows, and up to 2048 where there are more than 16 tiles, one workgroup
// per tile takes all rows (gram_tile_kernel) and there are no partials.
inline bool gram_few_rows(int64_t n, int tiles) { return n <= 1024 || (n <= 2048 && tiles > 16); }

// Row blocks of the kernels with partials: one per 32 rows while that leaves half of the
// CUs idle (us at 16 / 32 / 64 / 128 rows: 3000 rows, complex128, 10 x 10 7.5 / 7.1 / 7.2 /
// 7.4, 64 x 64 18.1 / 15.6 / 17.9 / 24.2; 8192 rows 11.2 / 8.2 / 7.4 / 7.8 and 28 / 22 /
// 20 / 26, with 128 blocks of 64), up to one per CU at 128 rows (20000 rows, 10 x 10
// 14.4 / 14.4 / 10.5 / 8.3), and from some row count on two per CU.  Nothing in between:
// with 273 blocks (140000 rows) 17 CUs had two, for longer than all with two take (us,
// 256 / 273 / 512 blocks: complex128, 64 x 64 116 / 149 / 100, 56 x 48 63 / 102 / 73,
// 24 x 24 25 / 31 / 28).  The partials cost 2 KiB per tile and block, written and read.
//   One per CU reads best where the operands are the bound and a block has enough of
// them in flight: complex128 up to 8 tiles (1200000 rows, 256 / 512 / 1024: 16 x 16
// 108 / 111 / 120, 48 x 8 185 / 186 / 198; 3000000 rows, 32 x 16 384 / 391 / 399).
// complex64 has half the bytes in flight: 3000000 rows, 16 x 16 147 / 142 / 150,
// 32 x 16 272 / 241 / 236, but 800000 rows 38 / 40 / 46 and 79 / 73 / 76.  So has
// complex128 with a second Y (and scale) to 16 columns (4000000 rows, [16 16] scaled
// 569 / 519 / 531, [10 10] 393 / 362 / 370, not scaled 496 / 506 / 520).
//   Two per CU (two waves per SIMD) where the matrix unit is: from 262144 rows
// (complex128, 40 x 24 55 / 51, 64 x 64 198 / 165), with more than 21 tiles of
// complex128 from half of that (180000 rows, 40 x 40 53 / 49, 64 x 64 143 / 119;
// complex64 64 x 64 102 / 107).
inline int64_t gram_row_blocks(int64_t n, int tiles, bool c64, bool pair = false) {
    const int64_t two = tiles > 8                     ? (tiles > 21 && !c64 ? 1 << 17 : 1 << 18)
                        : c64 || (pair && tiles == 8) ? 1 << 20
                                                      : INT64_MAX;
    return n >= two ? 512 : std::max({std::min<int64_t>(128, n / 32), std::min<int64_t>(256, n / 128), (int64_t)1});
}

// Scratch (complex128 entries) at which no n-row Gram of these widths runs with
// fewer row blocks than it wants, whatever its type and tile list (X and Y apart, or Y
// among X's columns, whose two ranges may take one unit more): more tiles want no
// fewer blocks.
inline size_t gram_part_entries(int64_t n, int bx, int by) {
    if (n <= 1024) return 0;
    const int tiles = (gram_units(bx) + 1) * gram_units(by);
    return (size_t)128 * tiles * std::max(gram_row_blocks(n, tiles, false), gram_row_blocks(n, tiles, true));
}

// Scratch of gplhr_gram_noalloc, kept on each GPU (64 MiB): X and Y apart always run
// with the row blocks they want, as in gplhr_gram.  With 16 MiB, 63 x 61 complex128
// had 128 blocks of 512 (1200000 rows: 1661 us, 686 with them all).
constexpr size_t GRAM_NOALLOC_ENTRIES = (size_t)4 << 20;

}  // namespace gplhr
