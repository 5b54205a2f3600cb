// Block-update kernels of complex64 blocks.
#include "update.h"

namespace gplhr {
template <> UpdFn<float2> update_pick<float2>(int nt, int sl, UpdKind k) {
    return update_pick_impl<float2>(nt, sl, k);
}
}  // namespace gplhr
