// Launch of the Gram kernels (gram.h): shape, row split and reduction.
#include "gram.h"

#include <algorithm>

namespace gplhr {

// Entry by entry, for leading dimensions whose four rows of a K step span more
// than 32-bit byte offsets (blocks of at most a few hundred rows).
template <typename T>
__global__ __launch_bounds__(256) void gram_strided_kernel(GramArgs<T> a) {
    __shared__ double2 sh[256];
    const int p = blockIdx.x % a.bx, q = blockIdx.x / a.bx;
    double2 acc = make_double2(0.0, 0.0);
    for (int64_t i = threadIdx.x; i < a.n; i += 256) {
        double2 y = to_d(a.Y2 && q >= a.by1 ? a.Y2[i * a.ldy2 + q - a.by1] : a.Y[i * a.ldy + q]);
        if (a.yscale && (!a.Y2 || q >= a.by1)) y = cmul(to_d(a.yscale[i]), y);
        cfma_cj(acc, to_d(a.X[i * a.ldx + p]), y);
    }
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) sh[threadIdx.x] = cadd(sh[threadIdx.x], sh[threadIdx.x + s]);
        __syncthreads();
    }
    if (threadIdx.x == 0) a.out[p + (int64_t)q * a.ldo] = sh[0];
}

size_t gram_part_entries(int bx, int by) {
    const size_t tiles = (size_t)((bx + 7) / 8 + 1) * ((by + 7) / 8);
    return std::min<size_t>(1024 * tiles, 32768) * 128;
}

template <typename T>
static void launch_gram_impl(hipStream_t st, int64_t n, const T *X, int ldx, int bx, const T *Y, int ldy, int by,
                             const T *yscale, double2 *part, size_t part_cap, double2 *out, int ldo,
                             const T *Y2 = nullptr, int ldy2 = 0, int by1 = 0) {
    if (bx < 1 || by < 1 || bx > 64 || by > 64) throw Error(-1, "gram: width out of range");
    if (n <= 0) throw Error(-1, "gram: empty block");
    GramArgs<T> a{};
    a.n = n; a.X = X; a.Y = Y; a.Y2 = Y2; a.ldx = ldx; a.ldy = ldy; a.ldy2 = ldy2; a.bx = bx; a.by = by;
    a.by1 = by1; a.yscale = yscale; a.part = reinterpret_cast<double *>(part); a.out = out; a.ldo = ldo;
    if ((int64_t)std::max({ldx, ldy, ldy2}) * 3 * (int64_t)sizeof(T) + 4096 > (int64_t)UINT32_MAX) {
        hipLaunchKernelGGL(gram_strided_kernel<T>, dim3(bx * by), dim3(256), 0, st, a);
        GPLHR_HIP_CHECK(hipGetLastError());
        return;
    }
    auto units = [](int w) { return (w + 7) / 8; };
    GramFn<T> fn = nullptr;
    if (Y2) {
        a.ma = units(bx); a.mb1 = units(by1); a.mb = a.mb1 + units(by - by1);
        if (a.mb1 == a.ma && a.mb == 2 * a.ma) fn = gram_pick<T>(yscale ? 3 : 4, a.ma, a.mb, 0);
        a.ma1 = a.ma;
    } else if (yscale) {
        a.ma = a.ma1 = units(bx); a.mb = a.mb1 = units(by);
        if (a.ma == a.mb) fn = gram_pick<T>(2, a.ma, a.mb, 0);
    } else {
        const int wy = bx - by;
        if (ldx == ldy && wy >= 0 && Y == X + wy) {
            a.tri = 1;
            a.ma1 = units(wy); a.mb = a.mb1 = units(by); a.ma = a.ma1 + a.mb;
            fn = gram_pick<T>(1, a.ma, a.mb, a.ma1);
        }
        if (!fn) {
            a.tri = 0;
            if (units(bx) < units(by)) {   // the wider block's units are A's
                a.swap = 1;
                std::swap(a.X, a.Y); std::swap(a.ldx, a.ldy); std::swap(a.bx, a.by);
            }
            a.ma = a.ma1 = units(a.bx); a.mb = a.mb1 = units(a.by);
            fn = gram_pick<T>(0, a.ma, a.mb, 0);
        }
    }
    if (!fn) throw Error(-1, "gram: no tile layout for this shape");
    a.ntile = gram_tiles(a.ma, a.mb, a.ma1, a.tri);
    const int ks = 4 / gram_groups(a.ma, a.mb, a.ma1, a.tri);
    // Row blocks: one per 32 rows while that leaves CUs idle (a wave then has
    // two K steps, both in flight at once; 1024 rows, complex128, 32 x 32: 8.7 us
    // against 9.4 at 64 rows and 11.2 at 96), up to one per CU at 128 rows, then
    // two per CU (more than 8 tiles: two waves per SIMD) or four.  The partials
    // cost 2 KiB per tile and block, written and read: 262144 rows, complex128,
    // 14 x 14 20.1 us with 1024 blocks and 15.1 with 256, 40 x 40 91 us with 256
    // and 75 with 512; 4096000 rows, complex64, 16 x 16 118 us with 1024 blocks
    // and 141 with 256; 20000 rows, 10 x 10 9.9 us with 256 blocks, 7.5 with 156.
    // (X^H X as X^H Y of its width, see gram_groups.)
    const bool wide = (a.tri && a.ma1 == 0 ? a.ma * a.mb : a.ntile) > 8;
    int64_t nblk = std::max({std::min<int64_t>(128, n / 32), std::min<int64_t>(256, n / 128),
                             std::min<int64_t>(wide ? 512 : 1024, n / (wide ? 512 : 1024)), (int64_t)1});
    nblk = std::min<int64_t>(nblk, (int64_t)(part_cap / (128 * (size_t)a.ntile)));
    if (nblk < 1) throw Error(-1, "gram: partial buffer too small");
    a.rows_per_blk = ((n + nblk - 1) / nblk + 4 * ks - 1) / (4 * ks) * (4 * ks);
    a.nblk = (int)((n + a.rows_per_blk - 1) / a.rows_per_blk);
    hipLaunchKernelGGL(fn, dim3(a.nblk), dim3(GRAM_THREADS), 0, st, a);
    GPLHR_HIP_CHECK(hipGetLastError());
    hipLaunchKernelGGL(gram_reduce_kernel<T>, dim3(a.ntile * 4), dim3(1024), 0, st, a);
    GPLHR_HIP_CHECK(hipGetLastError());
}

template <typename T>
void launch_gram(hipStream_t st, int64_t n, const T *X, int ldx, int bx, const T *Y, int ldy, int by,
                 const T *yscale, double2 *part, size_t part_cap, double2 *out, int ldo) {
    launch_gram_impl<T>(st, n, X, ldx, bx, Y, ldy, by, yscale, part, part_cap, out, ldo);
}
template <typename T>
void launch_gram2(hipStream_t st, int64_t n, const T *X, int ldx, int bx, const T *Y1, int ldy1, int by1,
                  const T *Y2, int ldy2, int by2, const T *yscale2, double2 *part, size_t part_cap,
                  double2 *out, int ldo) {
    if (!Y1 || !Y2 || by1 < 1 || by2 < 1) throw Error(-1, "gram: two-part Y needs both parts");
    if (bx == by1 && bx == by2 && bx <= 16) {
        launch_gram_impl<T>(st, n, X, ldx, bx, Y1, ldy1, by1 + by2, yscale2, part, part_cap, out, ldo, Y2, ldy2, by1);
        return;
    }
    launch_gram_impl<T>(st, n, X, ldx, bx, Y1, ldy1, by1, nullptr, part, part_cap, out, ldo);
    launch_gram_impl<T>(st, n, X, ldx, bx, Y2, ldy2, by2, yscale2, part, part_cap, out + (size_t)by1 * ldo, ldo);
}
#define GPLHR_INST(T)                                                                                       \
    template void launch_gram<T>(hipStream_t, int64_t, const T *, int, int, const T *, int, int, const T *, \
                                 double2 *, size_t, double2 *, int);                                        \
    template void launch_gram2<T>(hipStream_t, int64_t, const T *, int, int, const T *, int, int,           \
                                  const T *, int, int, const T *, double2 *, size_t, double2 *, int);
GPLHR_INST(double2)
GPLHR_INST(float2)
#undef GPLHR_INST

}  // namespace gplhr
