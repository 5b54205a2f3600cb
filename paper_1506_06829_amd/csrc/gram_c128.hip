// Gram kernels of complex128 blocks.
#include "gram.h"

namespace gplhr {
template <> GramFn<double2> gram_pick<double2>(int kind, int ma, int mb, int a1) {
    return gram_pick_impl<double2>(kind, ma, mb, a1);
}
}  // namespace gplhr
