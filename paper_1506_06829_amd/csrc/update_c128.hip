// Block-update kernels of complex128 blocks.
#include "update.h"

namespace gplhr {
template <> UpdFn<double2> update_pick<double2>(int nt, int sl, UpdKind k) {
    return update_pick_impl<double2>(nt, sl, k);
}
}  // namespace gplhr
