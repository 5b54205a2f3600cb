// Launch of the Gram kernels (gram.h): shape, row split and reduction.
#include "gram.h"
#include "gram_split.h"

#include <algorithm>
#include <type_traits>

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

// One workgroup per tile over all rows, for blocks of few rows: no partials and
// no second kernel.  Wavefront w takes the K steps (4 rows) w, w + 16, ..., up to
// PF of them in flight, and the wavefronts' tiles are summed in that order; a
// tile's sum does not depend on the other columns.
//
// What bounds it: the launch, two dependent latencies (operands, LDS) and one
// CU's matrix rate per tile (4 cycles a row).  Against the kernels with partials
// (us, parts / tile): 64 rows 5.9 / 3.5, 64 x 64 10.0 / 3.8; 1024 rows, complex128
// 16 x 16 6.3 / 6.0, 64 x 64 11.8 / 6.2, complex64 16 x 16 6.3 / 5.2; 2048 rows,
// complex128 16 x 16 6.8 / 9.4, 64 x 64 14.1 / 9.8.  Hence: up to 1024 rows, and up
// to 2048 where there are more than 16 tiles.
template <typename T>
__global__ __launch_bounds__(1024) void gram_tile_kernel(GramArgs<T> a) {
    using R = typename RealOf<T>::R;
    constexpr int PF = 8;
    __shared__ double red[16][256];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int li = lane & 15, lk = lane >> 4;
    int i = blockIdx.x, j = 0;
    if (a.tri) {
        while (i >= a.ma1 + j + 1) { i -= a.ma1 + j + 1; ++j; }
    } else {
        j = i / a.ma;
        i -= j * a.ma;
    }
    // A's and B's unit: first column and columns left from there on (TRI: X holds
    // wy columns, then w; B's units are those of w)
    const int wy = a.bx - a.by;
    const bool two = a.Y2 && j >= a.mb1;
    const int xc = a.tri ? (i < a.ma1 ? i * 8 : wy + (i - a.ma1) * 8) : i * 8;
    const int xw = (a.tri && i < a.ma1 ? wy : a.bx) - xc;
    const int yc = a.tri ? wy + j * 8 : (two ? j - a.mb1 : j) * 8;
    const int yw = (a.tri ? a.bx : a.Y2 ? (two ? a.by - a.by1 : a.by1) : a.by) - yc;
    const T *Y = a.tri ? a.X : two ? a.Y2 : a.Y;
    const int ldy = a.tri ? a.ldx : two ? a.ldy2 : a.ldy;
    const T *sc = a.yscale && (!a.Y2 || two) ? a.yscale : nullptr;
    auto offs = [&](int ld, int w, int k) {   // bytes; columns past the block repeat its last one
        return (uint32_t)((k * (int64_t)ld) * sizeof(T) + min(li, 2 * w - 2 + (li & 1)) * sizeof(R));
    };
    const uint32_t oa = offs(a.ldx, xw, lk), ob = offs(ldy, yw, lk), os = lk * (uint32_t)sizeof(T);
    d4v acc = d4v{0.0, 0.0, 0.0, 0.0};
    // PF K steps from row r0 on; rows past the end (not `full`) read the last row
    // and enter as zeros
    auto steps = [&](int r0, auto full, auto scaled) {
        constexpr bool FULL = decltype(full)::value, SC = decltype(scaled)::value;
        R va[PF], vb[PF];
        T vs[PF];
#pragma unroll
        for (int p = 0; p < PF; ++p) {
            const int r = FULL ? r0 + 64 * p : min(r0 + 64 * p, (int)a.n - 1);
            const int back = FULL ? 0 : max(r + lk - ((int)a.n - 1), 0);   // rows past the end, this lane
            const char *px = reinterpret_cast<const char *>(a.X + xc + (int64_t)r * a.ldx);
            const char *py = reinterpret_cast<const char *>(Y + yc + (int64_t)r * ldy);
            va[p] = *reinterpret_cast<const R *>(px + (FULL ? oa : offs(a.ldx, xw, lk - back)));
            vb[p] = *reinterpret_cast<const R *>(py + (FULL ? ob : offs(ldy, yw, lk - back)));
            if constexpr (SC) vs[p] = *reinterpret_cast<const T *>(reinterpret_cast<const char *>(sc + r) + os -
                                                                   back * sizeof(T));
        }
#pragma unroll
        for (int p = 0; p < PF; ++p) {
            if (!FULL && r0 + 64 * p >= a.n) break;
            const bool ok = FULL || r0 + 64 * p + lk < a.n;
            double y = (double)vb[p];
            if constexpr (SC) {
                const double2 f = to_d(vs[p]);
                y = f.x * y + ((li & 1) ? f.y : -f.y) * (double)other_part(vb[p]);
            }
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(ok ? (double)va[p] : 0.0, ok ? y : 0.0, acc, 0, 0, 0);
        }
    };
    auto rows = [&](auto scaled) {
        int r0 = 4 * wave;
        for (; r0 + 64 * (PF - 1) + 4 <= a.n; r0 += 64 * PF) steps(r0, std::true_type{}, scaled);
        if (r0 < a.n) steps(r0, std::false_type{}, scaled);
    };
    if (sc) rows(std::true_type{});
    else rows(std::false_type{});
#pragma unroll
    for (int v = 0; v < 4; ++v) red[wave][v * 64 + lane] = acc[v];
    __syncthreads();
    if (wave < 4) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < 16; ++w) s += red[w][threadIdx.x];
        gram_put_rows(a, blockIdx.x, wave, s);
    }
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
    const auto units = gram_units;
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
    // X^H X takes the path of X^H Y of its width, so that the same block passed as
    // a copy gives the same bits
    const int tiles = a.tri && a.ma1 == 0 ? a.ma * a.mb : a.ntile;
    if (gram_few_rows(n, tiles)) {
        hipLaunchKernelGGL(gram_tile_kernel<T>, dim3(a.ntile), dim3(1024), 0, st, a);
        GPLHR_HIP_CHECK(hipGetLastError());
        return;
    }
    const int ks = 4 / gram_groups(a.ma, a.mb, a.ma1, a.tri);
    int64_t nblk = gram_row_blocks(n, tiles, sizeof(T) == 8, Y2 != nullptr);
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
