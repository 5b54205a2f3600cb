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

// Row blocks of the kernels with partials: one per 32 rows while that leaves CUs idle
// (a wave then has two K steps, both in flight at once), up to one per CU at 128
// rows, then two per CU (more than 8 tiles: two waves per SIMD) or four.  The
// partials cost 2 KiB per tile and block, written and read: 262144 rows, complex128,
// 14 x 14 20.1 us with 1024 blocks and 15.1 with 256, 40 x 40 91 us with 256 and 75
// with 512; 4096000 rows, complex64, 16 x 16 118 us with 1024 blocks and 141 with
// 256; 20000 rows, 10 x 10 9.9 us with 256 blocks, 7.5 with 156.
inline int64_t gram_row_blocks(int64_t n, bool wide) {
    return std::max({std::min<int64_t>(128, n / 32), std::min<int64_t>(256, n / 128),
                     std::min<int64_t>(wide ? 512 : 1024, n / (wide ? 512 : 1024)), (int64_t)1});
}

// Scratch (complex128 entries) at which no n-row Gram of these widths runs with
// fewer row blocks than it wants, whatever its tile list (X and Y apart, or Y
// among X's columns, whose two ranges may take one unit more).
inline size_t gram_part_entries(int64_t n, int bx, int by) {
    if (n <= 1024) return 0;
    const size_t tiles = (size_t)(gram_units(bx) + 1) * gram_units(by);
    return 128 * std::max(tiles * gram_row_blocks(n, true), std::min<size_t>(tiles, 8) * gram_row_blocks(n, false));
}

}  // namespace gplhr
