// CSR sparse matrix times row-major block: the kernel and its launch.
// Instantiated by spmm_c128.hip and spmm_c64.hip (one file per block type, so
// that they compile side by side).
//
// A group of `lpr` consecutive lanes owns one matrix row; lane l of the group
// owns CPL consecutive columns of the block (CPL = 2 for complex64 so every
// lane moves 16 bytes).  The gathered block rows are contiguous segments, and no
// cross-lane reduction is needed.
#pragma once
#include <algorithm>
#include <type_traits>

#include "device_math.h"
#include "spmm_shape.h"

namespace gplhr {

// CPL consecutive complex values per lane, moved as 16-byte vectors.
template <typename T, int CPL>
__device__ __forceinline__ void load_vec(const T *p, T (&x)[CPL]) {
    if constexpr (sizeof(T) == 16 || CPL == 1) {
#pragma unroll
        for (int c = 0; c < CPL; ++c) x[c] = p[c];
    } else {
#pragma unroll
        for (int c = 0; c < CPL; c += 2) {
            const float4 v = *reinterpret_cast<const float4 *>(p + c);
            x[c] = make_float2(v.x, v.y);
            x[c + 1] = make_float2(v.z, v.w);
        }
    }
}
template <typename T, int CPL>
__device__ __forceinline__ void store_vec(T *p, const T (&x)[CPL]) {
    if constexpr (sizeof(T) == 16 || CPL == 1) {
#pragma unroll
        for (int c = 0; c < CPL; ++c) p[c] = x[c];
    } else {
#pragma unroll
        for (int c = 0; c < CPL; c += 2)
            *reinterpret_cast<float4 *>(p + c) = make_float4(x[c].x, x[c].y, x[c + 1].x, x[c + 1].y);
    }
}
// The same with non-temporal stores (streamed past the caches): for outputs
// too large to stay in the Infinity Cache until they are read again.
template <typename T, int CPL>
__device__ __forceinline__ void store_vec_nt(T *p, const T (&x)[CPL]) {
    typedef float f2n __attribute__((ext_vector_type(2)));
    typedef float f4n __attribute__((ext_vector_type(4)));
    typedef double d2n __attribute__((ext_vector_type(2)));
    if constexpr (sizeof(T) == 16) {
#pragma unroll
        for (int c = 0; c < CPL; ++c)
            __builtin_nontemporal_store(d2n{x[c].x, x[c].y}, reinterpret_cast<d2n *>(p + c));
    } else if constexpr (CPL == 1) {
        __builtin_nontemporal_store(f2n{x[0].x, x[0].y}, reinterpret_cast<f2n *>(p));
    } else {
#pragma unroll
        for (int c = 0; c < CPL; c += 2)
            __builtin_nontemporal_store(f4n{x[c].x, x[c].y, x[c + 1].x, x[c + 1].y},
                                        reinterpret_cast<f4n *>(p + c));
    }
}

template <typename T>
struct SpmmArgs {
    int64_t n;
    const int32_t *rp;
    const int32_t *ci;
    const T *val;
    const T *X;
    int ldx;
    T *Y;
    int ldy;
    int b;
    const T *Rhs;
    int ldr;
    const T *dw;
    const double2 *dval, *dcs;        // MODE 3: C's values and dw
    const unsigned long long *stop;   // not null and not zero: leave Y alone
    SpmmShape s;
    int nt;         // 1: non-temporal stores of Y
};

// MODE 0: Y = C X; MODE 1: the damped Jacobi sweep Y = X + dw .* (Rhs - C X);
// MODE 2: the first two sweeps from w_0 = 0 in one pass, Y = w + dw .* (Rhs -
// C w) with w = dw .* Rhs: X is Rhs and val holds the values of C diag(dw)
// (launch_scale_cols), so C w is gathered from Rhs directly; MODE 3: the same
// with the values formed while they are staged (rounded as launch_scale_cols and
// a conversion to complex64 do).  Compile-time, so the plain product carries no
// epilogue registers.  BATCH entries of a row
// have their block-row gathers in flight together.
//
// Index/value stream through LDS: where the entries of a wavefront's rows (always
// consecutive) fit in SPMM_STAGE entries, it first copies its row
// pointers and its whole segment of column indices and values into LDS with
// coalesced loads, all in flight together; each lane group then reads its row's
// entries from LDS.  Otherwise every lane group reads its row's entries from
// global memory.  Both paths take a row's entries in the same order, so the
// results are the same bit for bit.
//
// What bounds it: on operators whose neighbours stay in the L2, memory (X, Y and
// the matrix once each); on random patterns, the fabric behind the L2 (262144
// rows of 17 entries, 10 complex128 columns: 152 us whatever the kernel's shape,
// 713 MB of block rows at 4.7 TB/s).  Close behind the first came the instructions
// around the 4 CPL FMAs per entry and the serial loads before the gather.  Hence:
// indices staged as byte offsets of their block rows (S32: X spans less than
// 4 GiB), one multiplication per entry, not one per lane and entry; no masks in a
// batch that all rows of the wavefront fill; no vector divisions; and stages of one
// wavefront, without workgroup barriers or a wait for the row pointers.  Before ->
// now: 160^3 operator, 16 complex64 columns 340 -> 316 us (4.4 TB/s); 16 and 10
// complex128 676 -> 633 and 493 -> 425; 64^3, 10 complex128 26.1 -> 21.0.  (Resident
// workgroups that load the next rows' entries during the gather: 381 us, as they
// drift apart and lose the L2's neighbours.)
// entries per wavefront
template <typename T> constexpr int SPMM_STAGE = sizeof(T) == 16 ? 256 : 320;

// The batch of unstaged rows, whose values take registers before the block rows do:
// shorter where the whole one costs a wave per SIMD (30000 rows of 30, 16 complex64
// columns 14.7 us with 17 in 136 VGPRs, 12.4 with 15 in 120; 262144 rows of 10 to
// 14 in a band, 64 complex128 columns 325 with 12 in 170, 297 with 10 in 164; mode 3
// with 17 complex128 entries took 312 registers).
template <typename T, int CPL, int MODE, int BATCH>
constexpr int spmm_unstaged() {
    if (CPL == 1) return BATCH;
    if (sizeof(T) == 8) return BATCH == 17 ? 15 : BATCH;
    return BATCH == 12 ? 10 : BATCH == 17 && MODE == 3 ? 12 : BATCH;
}

// CHECK: the kernel asks the row pointers for the order of the rows; a kernel of its
// own, as a plane schedule lost 5 % to these lines without taking them (160^3 operator,
// 16 complex128 columns 636 us, 666 with them).
template <typename T, int CPL, int MODE, int BATCH, bool S32, bool CHECK>
__global__ __launch_bounds__(256) void spmm_kernel(SpmmArgs<T> a) {
    constexpr int WS = SPMM_STAGE<T>;
    __shared__ uint32_t s_ci[4 * WS];   // S32: byte offset of the block row
    __shared__ T s_val[4 * WS];
    __shared__ int32_t s_rp[260];
    const int tid = threadIdx.x, lane = tid & 63;
    if constexpr (MODE == 1 || MODE == 3)   // (the modes that are launched with one)
        if (a.stop && *a.stop) return;
    auto value_of = [&](int e, int32_t j) {
        if constexpr (MODE == 3) return from_d<T>(cmul(a.dval[e], a.dcs[j]));
        else return a.val[e];
    };
    // this wavefront's rows, row0 .. row0 + nr - 1, and entries, ne from e0 on
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const auto mine = [&](SpmmRows r) {
        return SpmmRows{r.row0 + wv * a.s.rpw, min(a.s.rpw, r.nr - wv * a.s.rpw)};
    };
    int ends = 0;   // lanes 0 .. 8: the row pointers at the eighths' ends
    if constexpr (CHECK) ends = a.rp[min(min(lane, 8) * ((uint32_t)a.s.nbs * (uint32_t)a.s.rpb), (uint32_t)a.n)];
    SpmmRows rows = mine(a.s.sp > 0 ? spmm_plane_rows(a.s, blockIdx.x)
                                    : spmm_natural_rows(a.s, a.n, blockIdx.x, a.s.order != SPMM_TURN));
    const auto entries = [&](const SpmmRows &r, int &first, int &count) {
        const int64_t r0 = CHECK ? min(r.row0, a.n) : r.row0;   // (CHECK: also waves without rows)
        first = __builtin_amdgcn_readfirstlane(a.rp[r0]);
        count = __builtin_amdgcn_readfirstlane(a.rp[r0 + (CHECK ? max(r.nr, 0) : r.nr)]) - first;
    };
    if (!CHECK && rows.nr <= 0) return;
    int e0, ne;
    entries(rows, e0, ne);
    if constexpr (CHECK) {
        const int more = __builtin_amdgcn_update_dpp(0, ends, 0x101, 0xf, 0xf, false) - ends;   // entries of eighth `lane`
        const int total = __builtin_amdgcn_readlane(ends, 8) - __builtin_amdgcn_readfirstlane(ends);
        if (__ballot(lane < 8 && !spmm_even(more, total))) {
            rows = mine(spmm_natural_rows(a.s, a.n, blockIdx.x, false));
            entries(rows, e0, ne);
        }
    }
    if (CHECK && rows.nr <= 0) return;
    const int64_t row0 = rows.row0;
    const int nr = rows.nr;
    uint32_t *w_ci = s_ci + wv * WS;
    T *w_val = s_val + wv * WS;
    int32_t *w_rp = s_rp + wv * 65;
    const bool staged = ne <= WS;
    const std::conditional_t<S32, uint32_t, uint64_t> rowb = (uint64_t)a.ldx * sizeof(T);
    if (staged) {
        int32_t rp = 0, ci[WS / 64];
        typedef decltype(T::x) vec __attribute__((ext_vector_type(2)));
        vec val[WS / 64];
        if (lane < nr) rp = a.rp[row0 + lane];
#pragma unroll
        for (int q = 0; q < WS / 64; ++q)
            if (64 * q < ne) {   // entries past the last repeat it
                const int e = e0 + min(64 * q + lane, ne - 1);
                ci[q] = a.ci[e];
                if constexpr (MODE != 3) val[q] = reinterpret_cast<const vec *>(a.val)[e];
            }
        if constexpr (MODE == 3)
#pragma unroll
            for (int q = 0; q < WS / 64; ++q)
                if (64 * q < ne) {
                    const T f = value_of(e0 + min(64 * q + lane, ne - 1), ci[q]);
                    val[q] = vec{f.x, f.y};
                }
        if (lane < nr) w_rp[lane] = rp - e0;
        if (lane == 0) w_rp[nr] = ne;
#pragma unroll
        for (int q = 0; q < WS / 64; ++q)
            if (64 * q < ne) {
                w_ci[64 * q + lane] = S32 ? (uint32_t)(ci[q] * rowb) : (uint32_t)ci[q];
                reinterpret_cast<vec *>(w_val)[64 * q + lane] = val[q];
            }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    const int r = (lane * a.s.inv) >> 16, c0 = (lane - r * a.s.lpr) * CPL;
    if (r >= nr || c0 >= a.b) return;
    const int64_t row = row0 + r;

    // epilogue operands first, so their latency overlaps the gather
    T xo[CPL], rh[CPL], w = czero<T>();
    if constexpr (MODE == 1) {
        load_vec<T, CPL>(a.X + row * a.ldx + c0, xo);
        load_vec<T, CPL>(a.Rhs + row * a.ldr + c0, rh);
        w = a.dw[row];
    } else if constexpr (MODE >= 2) {
        load_vec<T, CPL>(a.Rhs + row * a.ldr + c0, rh);
        w = a.dw[row];
#pragma unroll
        for (int c = 0; c < CPL; ++c) xo[c] = cmul(w, rh[c]);
    }
    T acc[CPL];
#pragma unroll
    for (int u = 0; u < CPL; ++u) acc[u] = czero<T>();
    const char *__restrict__ X = reinterpret_cast<const char *>(a.X);
    const uint32_t cb = (uint32_t)c0 * (uint32_t)sizeof(T);
    constexpr int UNSTAGED = spmm_unstaged<T, CPL, MODE, BATCH>();
    // entries p .. p + NB - 1 of the row; those past its end leave the sums
    // alone, wherever their loads point (NaN there must not reach them)
    auto batch = [&](int p, int p1, auto index, auto value, auto full, auto lds) {
        constexpr bool FULL = decltype(full)::value, LDS = decltype(lds)::value;
        constexpr int NB = LDS ? BATCH : UNSTAGED;
        T x[NB][CPL], v[NB];
        uint32_t j[NB];
        auto block_row = [&](int u) {
            if constexpr (S32) load_vec<T, CPL>(reinterpret_cast<const T *>(X + (j[u] + cb)), x[u]);
            else load_vec<T, CPL>(reinterpret_cast<const T *>(X + j[u] * rowb + cb), x[u]);
        };
        // entries past the row's end (p1) repeat its last one; its block row is
        // loaded again where that is cheaper than masked loads (short rows: 160^3
        // operator, 10 complex128 columns 425 us against 444; 131072 rows of 1 to 35
        // entries, 10 columns: 76 against 73.5)
        auto at = [&](int u) { return FULL ? p + u : min(p + u, p1 - 1); };
#pragma unroll
        for (int u = 0; u < NB; ++u) j[u] = index(at(u));
        if constexpr (!LDS)
#pragma unroll
            for (int u = 0; u < NB; ++u) v[u] = value(at(u));
#pragma unroll
        for (int u = 0; u < NB; ++u)
            if (FULL || NB <= 7 || p + u < p1) block_row(u);
        if constexpr (LDS)
#pragma unroll
            for (int u = 0; u < NB; ++u) v[u] = value(at(u));
#pragma unroll
        for (int u = 0; u < NB; ++u)
#pragma unroll
            for (int c = 0; c < CPL; ++c) {
                T s = acc[c];
                cfma(s, v[u], x[u][c]);
                if (FULL || p + u < p1) acc[c] = s;
            }
    };
    auto walk = [&](int p, int p1, auto index, auto value, auto lds) {
        constexpr int NB = decltype(lds)::value ? BATCH : UNSTAGED;
        for (; p < p1; p += NB) {
            if (__all(p + NB <= p1)) batch(p, p1, index, value, std::true_type{}, lds);
            else batch(p, p1, index, value, std::false_type{}, lds);
        }
    };
    if (staged)
        walk(w_rp[r], w_rp[r + 1], [&](int e) { return w_ci[e]; }, [&](int e) { return w_val[e]; },
             std::true_type{});
    else
        walk(a.rp[row], a.rp[row + 1],
             [&](int e) { return S32 ? (uint32_t)(a.ci[e] * rowb) : (uint32_t)a.ci[e]; },
             [&](int e) { return value_of(e, MODE == 3 ? a.ci[e] : 0); }, std::false_type{});
    T out[CPL];
    if constexpr (MODE == 0) {
#pragma unroll
        for (int c = 0; c < CPL; ++c) out[c] = acc[c];
    } else {
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            out[c] = xo[c];
            cfma(out[c], w, csub(rh[c], acc[c]));
        }
    }
    if (a.nt) store_vec_nt<T, CPL>(a.Y + row * a.ldy + c0, out);
    else store_vec<T, CPL>(a.Y + row * a.ldy + c0, out);
}

// Row schedule.  Without a plane, XCD x runs the x-th eighth of the rows where the
// eighths have about the same number of entries, so that rows gathered by
// neighbouring blocks are fetched into one L2 (in turn, each XCD fetches nearly
// every block row: 45^3 operator, 16 complex64 columns 11.4 us, by eighths 7.3 to
// 8.1; 10 complex128 16.4 and 9.6; random patterns the same), else they run in turn
// (spmm_even).  With a
// plane of P rows (all couplings within +-P rows, n a multiple of P, P a multiple
// of 8), XCD x runs slab x (rows x P/8 ... (x+1) P/8 - 1) of every plane, plane
// after plane: the three planes of one slab that a block touches fit in that XCD's
// L2, and every block row is fetched about once (160^3 operator, 16 complex64
// columns: 1.96 -> 0.93 GB read per product).
//
// Batch length.  A row's entries are taken BATCH at a time: their indices first,
// then all their block-row gathers, so a row of at most BATCH entries costs one
// round of dependent latencies.  BATCH follows the typical row length (nnz / n):
// 5 or 7 slots (stencils of 5 and 7 points, without idle slots), 12 or 17.  17 is the
// most the complex128 kernel with two columns per lane keeps within 256 VGPRs.
// Measured at n = 262144, 17 random entries per row, 10 complex128 columns: 176 us
// with 8 slots, 166 us with 12, 153 us with 17.  Shorter than that
// - for rows of 8, whose 12 slots idle (60000 rows, 16 complex128 columns: 20.3 us
//   with 12, 19.1 with 7; with few columns, where the entries' latency counts, 12: 4
//   columns 6.7 and 7.3);
// - for longer rows of blocks that stay in the L2, where the last batch's idle slots
//   cost more than latencies (30000 rows of 1 to 60, 8 complex128 columns 20.1 with 17,
//   17.4 with 7; not with few columns: 300000 rows of 30, one column 115 and 162), and
//   for wide complex64 blocks of long rows (20000 rows of 100, 64 columns 80 with 17,
//   69 with 5; beyond about 16 MB 100000 rows of 300, 24 columns 612 and 765).
template <typename T, int MODE, int BATCH>
static void spmm_go(hipStream_t st, const SpmmArgs<T> &a, int cpl, int grid) {
    // block rows and columns within 32-bit byte offsets
    const bool s32 = (double)a.n * a.ldx * sizeof(T) + (double)a.b * sizeof(T) < 4294967296.0;
    const auto pick = [&](auto check) {
        constexpr bool C = decltype(check)::value;
        return cpl == 2 ? (s32 ? spmm_kernel<T, 2, MODE, BATCH, true, C> : spmm_kernel<T, 2, MODE, BATCH, false, C>)
                        : (s32 ? spmm_kernel<T, 1, MODE, BATCH, true, C> : spmm_kernel<T, 1, MODE, BATCH, false, C>);
    };
    const auto fn = a.s.order == SPMM_CHECK ? pick(std::true_type{}) : pick(std::false_type{});
    hipLaunchKernelGGL(fn, dim3(grid), dim3(256), 0, st, a);
}

template <typename T, int MODE>
static void spmm_batch(hipStream_t st, const SpmmArgs<T> &a, int cpl, int grid, int row_len) {
    const double x = (double)a.n * a.b * sizeof(T);   // bytes the gathers spread over
    if (row_len <= 5) spmm_go<T, MODE, 5>(st, a, cpl, grid);
    else if (row_len <= 7 || (row_len == 8 && sizeof(T) == 16 && a.b >= 8)) spmm_go<T, MODE, 7>(st, a, cpl, grid);
    else if (row_len > 17 && row_len <= 40 && a.b >= 8 && x <= 8e6) spmm_go<T, MODE, 7>(st, a, cpl, grid);
    else if (row_len > 40 && sizeof(T) == 8 && a.b >= 24 && x <= 16e6) spmm_go<T, MODE, 5>(st, a, cpl, grid);
    else if (row_len <= 12) spmm_go<T, MODE, 12>(st, a, cpl, grid);
    else spmm_go<T, MODE, 17>(st, a, cpl, grid);
}

template <typename T>
static void spmm_launch(hipStream_t st, SpmmArgs<T> a, int mode, int plane, int64_t nnz) {
    const int64_t n = a.n;
    const int b = a.b;
    if (n <= 0) return;
    if (plane < 0 || (plane > 0 && (n % plane != 0 || plane % 8 != 0)))
        throw Error(-1, "spmm: the plane must divide n and be a multiple of 8");
    // an output block larger than the 256 MB Infinity Cache cannot stay there
    // until it is read again: stream it past the caches
    a.nt = ((double)n * b * sizeof(T) > 256.0 * 1024 * 1024) ? 1 : 0;
    // typical entries per row, rounded up
    const int64_t row_len = nnz > 0 ? (nnz + n - 1) / n : 0;
    // Columns per lane: 16 bytes, two complex64 or one complex128 (the 160^3
    // operator, 16 complex64 columns: two beat one and four; 10 complex128 columns:
    // 425 us with one, 464 with two, as registers halve).  Two complex128 columns
    // - where a row would leave lanes of its wavefront idle (22 to 24 columns, over 32:
    //   us with one / two columns, 64^3 operator, 24 columns 53.9 / 47.4, 40 154 / 121);
    // - with wide blocks of rows of more than 7 entries (24 columns, 262144 rows of 12 in
    //   a band 99 / 76; 32 columns, 60000 rows of 40 156 / 150; 20000 rows of 25, 20
    //   columns 16.7 / 19.0, 24 19.6 / 19.2), and from 16 columns on with rows that no
    //   stage holds (16 columns, 30000 rows of 130 78.6 / 67.6; 50000 of 50 69.4 / 75.3);
    // - where a row is one batch of 13 to 17 entries and the blocks fill the chip
    //   (262144 rows of 17 random entries, 10 columns 154 / 151; longer rows want the
    //   wavefronts in flight, 60000 rows of 40, 16 columns 71.7 / 73.8).
    const uintptr_t align = reinterpret_cast<uintptr_t>(a.X) | reinterpret_cast<uintptr_t>(a.Y) |
                            (mode != 0 ? reinterpret_cast<uintptr_t>(a.Rhs) : 0);
    int cpl = 1;
    if constexpr (sizeof(T) == 8) {
        const bool ok2 = (b % 2 == 0) && (a.ldx % 2 == 0) && (a.ldy % 2 == 0) &&
                         (mode == 0 || a.ldr % 2 == 0) && align % 16 == 0;
        cpl = ok2 ? 2 : 1;
    } else if (b > 32 || (64 / b) * b < 50 || (row_len > 7 && b > 20) || (row_len > 50 && b >= 16) ||
               (row_len > 12 && (row_len <= 17 || b > 16) && n * b >= (1 << 20))) {
        cpl = b % 2 == 0 ? 2 : 1;
    }
    if ((b + cpl - 1) / cpl > 64) throw Error(-1, "spmm: block too wide");
    int64_t grid = 0;
    a.s = spmm_launch_shape(n, b, cpl, sizeof(T) == 16 && b % 2 == 0 ? 2 : cpl, plane, row_len, SPMM_STAGE<T>,
                            sizeof(T) == 8 || cpl == 1 || row_len <= 17, grid);
    if (grid == 0) throw Error(-3, "spmm: more rows of this width than one launch takes");
    const int rl = (int)std::min<int64_t>(row_len, 1 << 20);
    if (mode == 0) spmm_batch<T, 0>(st, a, cpl, (int)grid, rl);
    else if (mode == 1) spmm_batch<T, 1>(st, a, cpl, (int)grid, rl);
    else if (mode == 2) spmm_batch<T, 2>(st, a, cpl, (int)grid, rl);
    else spmm_batch<T, 3>(st, a, cpl, (int)grid, rl);
    GPLHR_HIP_CHECK(hipGetLastError());
}

template <typename T>
void launch_spmm(hipStream_t st, int64_t n, const int32_t *rp, const int32_t *ci, const T *val,
                 const T *X, int ldx, T *Y, int ldy, int b, int mode, const T *Rhs, int ldr,
                 const T *dw, int plane, int64_t nnz, const unsigned long long *stop) {
    SpmmArgs<T> a{};
    a.n = n; a.rp = rp; a.ci = ci; a.val = val; a.X = X; a.ldx = ldx; a.Y = Y; a.ldy = ldy; a.b = b;
    a.Rhs = Rhs; a.ldr = ldr; a.dw = dw; a.stop = stop;
    spmm_launch<T>(st, a, mode, plane, nnz);
}

template <typename T>
void launch_jacobi2(hipStream_t st, int64_t n, const int32_t *rp, const int32_t *ci, const double2 *val,
                    const double2 *dw, const T *dwT, const T *R, int ldr, T *Y, int ldy, int b, int plane,
                    int64_t nnz, const unsigned long long *stop) {
    SpmmArgs<T> a{};
    a.n = n; a.rp = rp; a.ci = ci; a.X = R; a.ldx = ldr; a.Y = Y; a.ldy = ldy; a.b = b;
    a.Rhs = R; a.ldr = ldr; a.dw = dwT; a.dval = val; a.dcs = dw; a.stop = stop;
    spmm_launch<T>(st, a, 3, plane, nnz);
}

}  // namespace gplhr
