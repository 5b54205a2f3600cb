// Gram matrices G = X^H diag(yscale) Y in FP64, deterministic: the kernel.
// Instantiated by gram_c128.hip and gram_c64.hip (one file per block type, so
// that they compile side by side).
//
// The complex product is the real GEMM [Re X, Im X]^T [Re Y, Im Y] over the
// interleaved real views (n x 2bx and n x 2by) on the FP64 matrix instruction
// (16x16x4, FP64 accumulation; complex64 inputs are widened, so every product
// is exact).  A unit is 8 complex columns (16 reals, one tile edge); the
// output is a list of 16x16 tiles, known at compile time from the unit counts.
//
// What bounds it: on gfx950 the FP64 matrix instruction holds the vector ALU
// for its whole 64 cycles (a loop with one v_mov per 4 cycles of matrix work
// ran at half rate, also with other waves to fill in), so every vector
// instruction of the loop adds to the matrix time.  The loop therefore has
// none but the widening of complex64 operands and the row scale: operands come
// from global memory straight into the operand layout (lane 16 k + i reads real
// column i of row k), at a scalar base that the scalar unit advances, with no
// masks (columns past the block repeat a valid one and their products are not
// stored; rows past the end are a masked step of their own after the loop).
//
// The four waves of a workgroup form G tile groups times KS = 4 / G row
// splits.  G = 1 up to 21 tiles (TRI: 17), 2 up to 34, else 4 (at most 168 accumulator
// registers, two waves per SIMD); each group is a range of the tile list with
// a body of its own, so that the groups differ by one tile at most.  The waves of one row
// split read the same rows at about the same time, from L1.  A range of a few whole
// columns of the list reads all of A again, so one group is the better while its
// accumulators fit (1200000 rows, us, two groups / one): complex128 47 x 21 326 / 229,
// 40 x 32 308 / 247, 56 x 24 401 / 269; complex64 48 x 24 197 / 186, 40 x 32 210 / 200.
// 24 tiles in one group spill (complex64 48 x 32 250 / 264).
//
// TRI: Y is X's last `w` columns (X^H X of a Cholesky-QR step, [Y X]^H X of a
// projection): operands are loaded once, and of the Hermitian part only the
// tiles on and above the diagonal are formed; their mirror images are written
// conjugated (the same products in the same order).
//
// Measured against an LDS-staged kernel with per-tile masks that this one
// replaced (4096000 rows unless said, us before -> now): 64 x 64 complex64
// 2318 -> 1985 (67.6 of the 77 TFLOP/s that a register-only loop reaches),
// complex128 2450 -> 2290; X^H X of 48 columns 1366 -> 655 / 1350 -> 876;
// [Y X]^H X of 16 + 48 columns 1810 -> 1035 / 1816 -> 1215, of 48 + 16 complex128
// 590 -> 531 (5.9 TB/s); 262144 rows, complex128, 40 x 40 95 -> 75, 56 x 56
// 219 -> 150.
#pragma once
#include "device_math.h"

namespace gplhr {

template <typename T> struct RealOf;
template <> struct RealOf<double2> { using R = double; };
template <> struct RealOf<float2> { using R = float; };

constexpr int GRAM_THREADS = 256;

template <typename T>
struct GramArgs {
    int64_t n;
    const T *X;        // rows of A's units: bx columns (TRI: wy columns, then w)
    const T *Y;        // rect: Y's first part
    const T *Y2;       // rect: Y's columns from by1 on, or null
    int ldx, ldy, ldy2;
    int bx, by, by1;   // TRI: bx = wy + w, by = w
    const T *yscale;   // row scale of Y (of Y2's part where there is one)
    double *part;      // [block][tile][256]
    int64_t rows_per_blk;
    int nblk, ntile;
    int ma, mb, ma1, mb1;   // units of A and B; TRI: of wy; Y2: of by1 (else mb)
    int tri, swap;     // swap: G is written conjugate-transposed
    double2 *out;
    int ldo;
};

// Tiles in column order: unit pair (i, j), i fastest; TRI (a1 units before the
// Hermitian part) leaves out i - a1 > j.
constexpr int gram_tiles(int ma, int mb, int a1, bool tri) {
    int t = 0;
    for (int j = 0; j < mb; ++j)
        for (int i = 0; i < ma; ++i)
            if (!tri || i - a1 <= j) ++t;
    return t;
}
// Most tiles of a wave (of a kernel with one tile group; two have 17, four 16).
constexpr int GRAM_MAX_TILES = 21;
constexpr int gram_groups(int tiles, bool tri) { return tiles <= (tri ? 17 : GRAM_MAX_TILES) ? 1 : tiles <= 34 ? 2 : 4; }
// Tile groups of a kernel.  X^H X of up to 5 units splits its rows as X^H Y of
// those widths does, so that the same block passed as a copy gives the same bits.
constexpr int gram_groups(int ma, int mb, int a1, bool tri) {
    return tri && a1 == 0 && ma <= 5 ? gram_groups(ma * mb, false) : gram_groups(gram_tiles(ma, mb, a1, tri), tri);
}
// Four groups of a rectangular product: quadrants (of an odd unit count, halves
// that share the middle unit), which read fewer units than ranges of the list
// and share one body, so that the registers of several bodies don't add up.
// Ranges stay where they are the faster ones, as their groups share less work
// (2000000 rows, us as ranges / as quadrants): complex128, 56 x 56 1043 / 1086;
// complex64, 56 x 40 706 / 806, scaled 56 x 56 1007 / 1090; 262144 rows, 56 x 48
// 106 / 112 (1200000 471 / 481, 4000000 1699 / 1688).  These spill a little at the
// limit of 256 registers (28 to 52 bytes a lane; 56 x 40 does not), as does X^H X of
// 48 with 24 more columns (complex128, 16 bytes).  Elsewhere quadrants: complex128,
// 56 x 40 1322 / 835, 64 x 40 1050 / 845, 64 x 56 2565 / 1145, scaled 56 x 56
// 2313 / 1170; complex64, 64 x 56 2069 / 985, 56 x 56 1166 / 982.
template <typename T>
constexpr bool gram_quads(int ma, int mb, bool tri, bool scaled) {
    if (tri || gram_groups(ma * mb, false) != 4) return false;
    if (ma % 2 == 0 && mb % 2 == 0) return true;
    return sizeof(T) == 16 ? ma != mb || scaled : mb == 7 && !scaled;
}

struct GramPlan {
    int n;             // tiles of the group
    int ti[GRAM_MAX_TILES], tj[GRAM_MAX_TILES];
    bool ua[9], ub[9]; // units read
};
template <int MA, int MB, int A1, bool TRI>
constexpr GramPlan gram_plan(int g) {
    constexpr int NT = gram_tiles(MA, MB, A1, TRI), G = gram_groups(MA, MB, A1, TRI);
    GramPlan p{};
    const int lo = NT * g / G, hi = NT * (g + 1) / G;
    int t = 0;
    for (int j = 0; j < MB; ++j)
        for (int i = 0; i < MA; ++i) {
            if (TRI && i - A1 > j) continue;
            if (t >= lo && t < hi) {
                p.ti[p.n] = i;
                p.tj[p.n] = j;
                ++p.n;
                p.ua[i] = true;
                if (TRI) p.ua[A1 + j] = true;
                else p.ub[j] = true;
            }
            ++t;
        }
    return p;
}

// K steps in flight per wave: about 48 registers of operands, fewer beside
// many accumulators.  complex64 with 13 or 14 tiles would spill with four (us, four /
// three: 1200000 rows, 56 x 16 155 / 145, 56 x 32 289 / 267, scaled 40 x 40 277 / 269;
// 262144 rows 44.2 / 42.8, 70.2 / 67.8, 66.7 / 66.5).
template <typename T, int MA, int MB, int A1, bool TRI, int SC0>
constexpr int gram_pf() {
    constexpr int NT = gram_tiles(MA, MB, A1, TRI), G = gram_groups(MA, MB, A1, TRI);
    int most = 0, tiles = 0;
    for (int g = 0; g < G; ++g) {
        const GramPlan p = gram_plan<MA, MB, A1, TRI>(g);
        int c = 0;
        for (int i = 0; i < 9; ++i) c += p.ua[i] + p.ub[i];
        if (c > most) most = c;
        if (p.n > tiles) tiles = p.n;
    }
    const int regs = most * (int)sizeof(T) / 8 + (SC0 < MB ? (int)sizeof(T) / 4 : 0);
    const int pf = (tiles > 12 ? G == 4 && !gram_quads<T>(MA, MB, TRI, SC0 < MB) ? 30 : 40 : 56) / regs;
    if (sizeof(T) == 8 && (tiles == 13 || tiles == 14) && pf == 4) return 3;
    return pf < 2 ? 2 : pf > 8 ? 8 : pf;
}

// One complex entry from the four reals of its 2x2 block: entry (u, v) of tile
// (i, j), and its mirror image where the tile lies above the diagonal.
template <typename T>
__device__ __forceinline__ void gram_put(const GramArgs<T> &a, int i, int j, int u, int v, double rr, double ri,
                                         double ir, double ii) {
    const double2 g = make_double2(rr + ii, ri - ir);
    int p, q;
    bool okp, okq;
    if (i < a.ma1) {
        p = i * 8 + u;
        okp = p < (a.tri ? a.bx - a.by : a.bx);
    } else {
        p = a.bx - a.by + (i - a.ma1) * 8 + u;   // TRI only
        okp = p < a.bx;
    }
    if (j < a.mb1) {
        q = j * 8 + v;
        okq = q < (a.Y2 ? a.by1 : a.by);
    } else {
        q = a.by1 + (j - a.mb1) * 8 + v;
        okq = q < a.by;
    }
    if (!okp || !okq) return;
    if (a.swap) {
        a.out[q + (int64_t)p * a.ldo] = make_double2(g.x, -g.y);
        return;
    }
    a.out[p + (int64_t)q * a.ldo] = g;
    if (a.tri && i >= a.ma1 && i - a.ma1 != j)
        a.out[(a.bx - a.by + q) + (int64_t)(p - (a.bx - a.by)) * a.ldo] = make_double2(g.x, -g.y);
}

// The complex entries of one accumulator register's 64 reals (rows 4 v ..
// 4 v + 3 of tile t): lane 16 k + c holds entry (4 v + k, c).
template <typename T>
__device__ __forceinline__ void gram_put_rows(const GramArgs<T> &a, int t, int v, double s) {
    const int lane = threadIdx.x & 63;
    const double right = __shfl_down(s, 1), down = __shfl_down(s, 16), diag = __shfl_down(s, 17);
    if (!((lane >> 4) & 1) && !(lane & 1)) {
        int i = t, j = 0;
        if (a.tri) {
            while (i >= a.ma1 + j + 1) { i -= a.ma1 + j + 1; ++j; }
        } else {
            j = t / a.ma;
            i = t - j * a.ma;
        }
        gram_put(a, i, j, (4 * v + (lane >> 4)) >> 1, (lane & 15) >> 1, s, right, down, diag);
    }
}

// Sum of the blocks' partials: workgroup (t, v) takes 64 reals; group g of its
// 16 x 64 threads sums the blocks g, g + 16, ... in that order and the groups
// are added in order, so the result is reproducible bit for bit.
template <typename T>
__global__ __launch_bounds__(1024) void gram_reduce_kernel(GramArgs<T> a) {
    __shared__ double sh[16][64];
    const int t = blockIdx.x >> 2, v = blockIdx.x & 3;
    const int lane = threadIdx.x & 63, g = threadIdx.x >> 6;
    double acc = 0.0;
    const double *src = a.part + (int64_t)t * 256 + v * 64 + lane;
    const int64_t step = (int64_t)a.ntile * 256;
#pragma unroll 8
    for (int b = g; b < a.nblk; b += 16) acc += src[b * step];
    sh[g][lane] = acc;
    __syncthreads();
    if (threadIdx.x < 64) {
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < 16; ++i) s += sh[i][lane];
        gram_put_rows(a, t, v, s);
    }
}

// The value of lane l ^ 1: the other part of the complex entry whose real (even
// lane) or imaginary part this lane holds.
__device__ __forceinline__ float other_part(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xb1, 0xf, 0xf, false));
}
__device__ __forceinline__ double other_part(double v) {
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(v), 0xb1, 0xf, 0xf, false),
                            __builtin_amdgcn_update_dpp(0, __double2loint(v), 0xb1, 0xf, 0xf, false));
}

// The rows of one wave: tile group GI, every KS-th K step.  M1: B units of the
// first part (MB: Y alone); SC0: the first B unit that takes the row scale (MB:
// none); u0, v0: the first unit of A and of B (quadrants).
template <typename T, int MA, int MB, int A1, bool TRI, int M1, int SC0, int GI, int KS>
__device__ __forceinline__ void gram_rows(const GramArgs<T> &a, int kh, int u0, int v0, d4v (&acc)[GRAM_MAX_TILES]) {
    using R = typename RealOf<T>::R;
    constexpr GramPlan P = gram_plan<MA, MB, A1, TRI>(GI);
    constexpr int PF = gram_pf<T, MA, MB, A1, TRI, SC0>();
    constexpr bool SC = SC0 < MB, TWO = !TRI && M1 < MB;
    constexpr int XA1 = TRI ? A1 : MA;   // A units of the first column range
    constexpr int US = 16 * sizeof(R);   // bytes of a unit
    const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
    const int64_t rb = (int64_t)blockIdx.x * a.rows_per_blk + 4 * kh;
    const int64_t re = min(a.n, (int64_t)(blockIdx.x + 1) * a.rows_per_blk);
    // byte offsets of the lane's element within a K step: the last unit of a
    // column range may be ragged, its columns past the end repeat the last one
    auto offs = [&](int ld, int c0, int w, int u, int first = 0) {
        return (uint32_t)((lk * (int64_t)ld + c0) * sizeof(T) +
                          min(u * 16 + li, 2 * w - 2 + (li & 1) - first * 16) * sizeof(R));
    };
    const int wy = TRI ? a.bx - a.by : a.bx, w1 = TWO ? a.by1 : a.by;
    const uint32_t oa = offs(a.ldx, 0, 64, 0), oal = XA1 ? offs(a.ldx, 0, wy, XA1 - 1, u0) : 0;
    const uint32_t ox = TRI ? offs(a.ldx, wy, 64, 0) : 0, oxl = TRI ? offs(a.ldx, wy, a.by, MB - 1) : 0;
    const uint32_t oy = TRI ? 0 : offs(a.ldy, 0, 64, 0), oyl = TRI ? 0 : offs(a.ldy, 0, w1, M1 - 1, v0);
    const uint32_t oz = TWO ? offs(a.ldy2, 0, 64, 0) : 0, ozl = TWO ? offs(a.ldy2, 0, a.by - a.by1, MB - M1 - 1) : 0;
    const char *px = reinterpret_cast<const char *>(a.X + rb * a.ldx) + u0 * US;
    const char *py = TRI ? nullptr : reinterpret_cast<const char *>(a.Y + rb * a.ldy) + v0 * US;
    const char *pz = TWO ? reinterpret_cast<const char *>(a.Y2 + rb * a.ldy2) : nullptr;
    const char *ps = SC ? reinterpret_cast<const char *>(a.yscale + rb) : nullptr;
    R va[PF][9], vb[PF][9];
    T vs[PF];
    // the operands of the K step at the running pointers, which then move on
    // by `rows`; back: rows to step back (the masked tail)
    auto load = [&](int p, int64_t rows, int64_t back) {
        auto get = [&](const char *base, uint32_t o, int imm, int ld) {
            return *reinterpret_cast<const R *>(base - back * ld * (int64_t)sizeof(T) + o + imm);
        };
#pragma unroll
        for (int u = 0; u < MA; ++u)
            if (P.ua[u])
                va[p][u] = u < XA1 ? (u == XA1 - 1 ? get(px, oal, 0, a.ldx) : get(px, oa, u * US, a.ldx))
                                   : (u == MA - 1 ? get(px, oxl, 0, a.ldx) : get(px, ox, (u - XA1) * US, a.ldx));
        if constexpr (!TRI) {
#pragma unroll
            for (int u = 0; u < MB; ++u)
                if (P.ub[u]) {
                    const bool z = TWO && u >= M1, l = z ? u == MB - 1 : u == M1 - 1;
                    const uint32_t o = z ? (l ? ozl : oz) : (l ? oyl : oy);
                    const int imm = l ? 0 : (z ? u - M1 : u) * US;
                    vb[p][u] = get(z ? pz : py, o, imm, z ? a.ldy2 : a.ldy);
                }
        }
        if constexpr (SC) vs[p] = *reinterpret_cast<const T *>(ps - back * (int64_t)sizeof(T) + (uint32_t)(lk * sizeof(T)));
        px += rows * a.ldx * (int64_t)sizeof(T);
        if constexpr (!TRI) py += rows * a.ldy * (int64_t)sizeof(T);
        if constexpr (TWO) pz += rows * a.ldy2 * (int64_t)sizeof(T);
        if constexpr (SC) ps += rows * (int64_t)sizeof(T);
    };
    auto step = [&](int p, bool ok) {
        double xa[9], xb[9];
        double sr = 0.0, si = 0.0;
        if constexpr (SC) {
            const double2 s = to_d(vs[p]);
            sr = s.x;
            si = (li & 1) ? s.y : -s.y;   // s y: even reals sr yr - si yi, odd ones sr yi + si yr
        }
#pragma unroll
        for (int u = 0; u < MA; ++u)
            if (P.ua[u]) xa[u] = ok ? (double)va[p][u] : 0.0;
        if constexpr (!TRI) {
#pragma unroll
            for (int u = 0; u < MB; ++u)
                if (P.ub[u]) {
                    double v = (double)vb[p][u];
                    if (u >= SC0) v = sr * v + si * (double)other_part(vb[p][u]);
                    xb[u] = ok ? v : 0.0;
                }
        }
#pragma unroll
        for (int t = 0; t < P.n; ++t)
            acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(xa[P.ti[t]], TRI ? xa[A1 + P.tj[t]] : xb[P.tj[t]], acc[t], 0, 0, 0);
    };
    constexpr int64_t SR = 4 * KS;   // rows between the wave's K steps
    const int64_t span = re - rb;
    const int nfull = span >= 4 ? (int)((span - 4) / SR + 1) : 0;   // whole K steps
    const int nmain = nfull / PF * PF;
    if (nmain > 0) {
#pragma unroll
        for (int p = 0; p < PF; ++p) load(p, p < PF - 1 || nmain > PF ? SR : 0, 0);
        // the pointers stop at the last step of the loop (read again, unused)
        for (int j = PF; j < nmain; j += PF) {
#pragma unroll
            for (int p = 0; p < PF; ++p) {
                step(p, true);
                load(p, p < PF - 1 || j + PF < nmain ? SR : 0, 0);
            }
        }
#pragma unroll
        for (int p = 0; p < PF; ++p) step(p, true);
        px += SR * a.ldx * (int64_t)sizeof(T);
        if constexpr (!TRI) py += SR * a.ldy * (int64_t)sizeof(T);
        if constexpr (TWO) pz += SR * a.ldy2 * (int64_t)sizeof(T);
        if constexpr (SC) ps += SR * (int64_t)sizeof(T);
    }
    // the last few K steps, masked: rows past the end read the block's last
    // row and enter as zeros
    const int64_t r0 = rb + nmain * SR;
    if (r0 < re) {
#pragma unroll
        for (int p = 0; p < PF; ++p) load(p, SR, max(r0 + p * SR + lk - (re - 1), (int64_t)0));
#pragma unroll
        for (int p = 0; p < PF; ++p)
            if (r0 + p * SR < re) step(p, r0 + p * SR + lk < re);
    }
}

template <typename T, int MA, int MB, int A1, bool TRI, int M1, int SC0>
__global__ __launch_bounds__(GRAM_THREADS) __attribute__((amdgpu_waves_per_eu(2, 8)))
void gram_kernel(GramArgs<T> a) {
    constexpr int NT = gram_tiles(MA, MB, A1, TRI), G = gram_groups(MA, MB, A1, TRI), KS = 4 / G;
    constexpr bool QUADS = gram_quads<T>(MA, MB, TRI, SC0 < MB);
    constexpr int TMAX = QUADS ? ((MA + 1) / 2) * ((MB + 1) / 2) : (NT + G - 1) / G;
    __shared__ double red[G == 4 ? 256 : G * 8 * 256];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int kh = wave / G, g = wave - kh * G;
    d4v acc[GRAM_MAX_TILES];
#pragma unroll
    for (int t = 0; t < TMAX; ++t) acc[t] = d4v{0.0, 0.0, 0.0, 0.0};
    double *part = a.part + (int64_t)blockIdx.x * NT * 256;
    // the block's partial: register v of lane 16 k + c holds entry (4 v + k, c)
    if constexpr (QUADS) {
        constexpr int HA = (MA + 1) / 2, HB = (MB + 1) / 2;
        const int u0 = (g & 1) * (MA - HA), v0 = (g >> 1) * (MB - HB);
        gram_rows<T, HA, HB, HA, false, HB, SC0 ? HB : 0, 0, 1>(a, kh, u0, v0, acc);
#pragma unroll
        for (int t = 0; t < HA * HB; ++t) {
            // a shared middle unit is the first halves'
            if ((MA % 2 && (g & 1) && t % HA == 0) || (MB % 2 && (g >> 1) && t < HA)) continue;
#pragma unroll
            for (int v = 0; v < 4; ++v)
                part[(u0 + t % HA + (v0 + t / HA) * MA) * 256 + v * 64 + lane] = acc[t][v];
        }
    } else if constexpr (G == 4) {
        if (g == 0) gram_rows<T, MA, MB, A1, TRI, M1, SC0, 0, 1>(a, kh, 0, 0, acc);
        if (g == 1) gram_rows<T, MA, MB, A1, TRI, M1, SC0, 1, 1>(a, kh, 0, 0, acc);
        if (g == 2) gram_rows<T, MA, MB, A1, TRI, M1, SC0, 2, 1>(a, kh, 0, 0, acc);
        if (g == 3) gram_rows<T, MA, MB, A1, TRI, M1, SC0, 3, 1>(a, kh, 0, 0, acc);
        const int id0 = NT * g / G, cnt = NT * (g + 1) / G - id0;
#pragma unroll
        for (int t = 0; t < TMAX; ++t)
            if (t < cnt)
#pragma unroll
                for (int v = 0; v < 4; ++v) part[(id0 + t) * 256 + v * 64 + lane] = acc[t][v];
    } else {
        if (g == 0) gram_rows<T, MA, MB, A1, TRI, M1, SC0, 0, KS>(a, kh, 0, 0, acc);
        if constexpr (G == 2)
            if (g == 1) gram_rows<T, MA, MB, A1, TRI, M1, SC0, 1, KS>(a, kh, 0, 0, acc);
        // row splits summed in LDS in the order kh, eight tiles at a time; the
        // group's tiles are NT g / G, ... of the list
        const int id0 = NT * g / G, cnt = NT * (g + 1) / G - id0;
        double *r = red + g * 8 * 256;
#pragma unroll
        for (int t0 = 0; t0 < TMAX; t0 += 8) {
#pragma unroll
            for (int h = 0; h < KS; ++h) {
                if (kh == h) {
#pragma unroll
                    for (int t = t0; t < t0 + 8 && t < TMAX; ++t)
                        if (t < cnt)
#pragma unroll
                            for (int v = 0; v < 4; ++v) {
                                double &d = r[(t - t0) * 256 + v * 64 + lane];
                                const double s = h == 0 ? acc[t][v] : d + acc[t][v];
                                if (h < KS - 1) d = s;
                                else part[(id0 + t) * 256 + v * 64 + lane] = s;
                            }
                }
                __syncthreads();
            }
        }
    }
}

template <typename T> using GramFn = void (*)(GramArgs<T>);

// The kernel of a shape, or null: kind 0 rect (ma >= mb), 1 TRI (a1 units,
// then mb), 2 rect with every B unit row-scaled (ma = mb), 3 and 4 rect
// ma x 2 ma for [X^H Y, X^H diag(s) Y2] with and without the scale (ma <= 2).
template <typename T> GramFn<T> gram_pick(int kind, int ma, int mb, int a1);

template <typename T, int KIND, int I>
constexpr GramFn<T> gram_fn() {
    constexpr int p = I / 9, q = I % 9;
    if constexpr (KIND == 0 && p <= 8 && q >= 1 && q <= p) return gram_kernel<T, p, q, p, false, q, q>;
    else if constexpr (KIND == 1 && q >= 1 && (p == 0 ? q <= 8 : p <= 6 && q <= 6 && p + q <= 9))
        return gram_kernel<T, p + q, q, p, true, q, q>;
    else if constexpr (KIND == 2 && p == q && p >= 1 && p <= 8) return gram_kernel<T, p, p, p, false, p, 0>;
    else if constexpr (KIND == 3 && p >= 1 && p <= 2 && q == 2 * p) return gram_kernel<T, p, q, p, false, p, p>;
    else if constexpr (KIND == 4 && p >= 1 && p <= 2 && q == 2 * p) return gram_kernel<T, p, q, p, false, p, q>;
    else return nullptr;
}
template <typename T, int KIND, int... I>
GramFn<T> gram_table(int i, std::integer_sequence<int, I...>) {
    static constexpr GramFn<T> t[] = {gram_fn<T, KIND, I>()...};
    return t[i];
}
template <typename T>
GramFn<T> gram_pick_impl(int kind, int ma, int mb, int a1) {
    const int p = kind == 1 ? a1 : ma;
    if (p < 0 || p > 8 || mb < 0 || mb > 8) return nullptr;
    const int i = p * 9 + mb;
    using Seq = std::make_integer_sequence<int, 81>;
    switch (kind) {
        case 0: return gram_table<T, 0>(i, Seq{});
        case 1: return gram_table<T, 1>(i, Seq{});
        case 2: return gram_table<T, 2>(i, Seq{});
        case 3: return gram_table<T, 3>(i, Seq{});
        default: return gram_table<T, 4>(i, Seq{});
    }
}

}  // namespace gplhr
