// Sparse products of complex64 blocks.
#include "spmm.h"

namespace gplhr {
template void launch_spmm<float2>(hipStream_t, int64_t, const int32_t *, const int32_t *, const float2 *,
                               const float2 *, int, float2 *, int, int, int, const float2 *, int, const float2 *,
                               int, int64_t, const unsigned long long *);
template void launch_jacobi2<float2>(hipStream_t, int64_t, const int32_t *, const int32_t *, const double2 *,
                                  const double2 *, const float2 *, const float2 *, int, float2 *, int, int, int,
                                  int64_t, const unsigned long long *);
}  // namespace gplhr
