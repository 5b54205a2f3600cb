// Sparse products of complex128 blocks.
#include "spmm.h"

namespace gplhr {
template void launch_spmm<double2>(hipStream_t, int64_t, const int32_t *, const int32_t *, const double2 *,
                               const double2 *, int, double2 *, int, int, int, const double2 *, int, const double2 *,
                               int, int64_t, const unsigned long long *);
template void launch_jacobi2<double2>(hipStream_t, int64_t, const int32_t *, const int32_t *, const double2 *,
                                  const double2 *, const double2 *, const double2 *, int, double2 *, int, int, int,
                                  int64_t, const unsigned long long *);
}  // namespace gplhr
