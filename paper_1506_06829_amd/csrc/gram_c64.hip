// Gram kernels of complex64 blocks.
#include "gram.h"

namespace gplhr {
template <> GramFn<float2> gram_pick<float2>(int kind, int ma, int mb, int a1) {
    return gram_pick_impl<float2>(kind, ma, mb, a1);
}
}  // namespace gplhr
