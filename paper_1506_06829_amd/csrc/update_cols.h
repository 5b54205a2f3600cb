// Which column of a slab a lane of update_stream_kernel reads.  No HIP here, so
// that the rule can be checked on the host.
#pragma once

namespace gplhr {

// A slab holds `lim` (1..8) columns of a term; lane group lk (0..3) owns entries
// 2 lk and 2 lk + 1 (h = 0, 1).  Entries past the slab read a column inside it
// and enter the product as zeros: a term may end its rows, and its last row the
// allocation.  pairs: both entries come from one 16-byte load at h = 0's column
// (lim is even then).
constexpr int upd_slab_column(int lim, int lk, int h, bool pairs) {
    return 2 * lk + h < lim ? 2 * lk + h : pairs ? h : 0;
}

}  // namespace gplhr
