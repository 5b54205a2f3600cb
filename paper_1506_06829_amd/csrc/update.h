// Row-local block update Out = beta Out + Add + sum_t alpha_t diag(rs_t) In_t M_t
// for up to 64 input columns: the kernel.  Instantiated by update_c128.hip and
// update_c64.hip (one file per block type, so that they compile side by side).
//
// The complex product is one real GEMM
//   [Re o_c, Im o_c] = sum_j [Re x_j, Im x_j] [[Re m, Im m], [-Im m, Re m]]_jc
// on the FP64 (complex128) or FP32 (complex64) 16x16x4 matrix instruction, with
// the coefficients as its left and the block's rows as its right operand: lane
// 16 k + i holds real K index k of row i, so that a row's entries go from memory
// straight into operand registers, and the product's registers of a lane are
// consecutive output entries of one row, stored as 16-byte pieces.
//
// What bounds it: HBM, except complex128 shapes with many products per byte,
// where the FP64 matrix instruction is; that instruction holds the vector ALU
// (see gram.h), so the loop has no vector instruction besides it.  The
// coefficients stand in LDS in operand order (lane-linear reads at immediate
// offsets) in their real form, formed once per workgroup.  A wave owns groups
// of 16 rows; as soon as a slab of 8 input columns has been multiplied its
// registers take the same slab of the wave's next row group, so all of the
// next group's reads are in flight behind the products of this one at one
// register buffer, and two to four waves fit a SIMD.
//
// Measured against a kernel with two register buffers, LDS-transposed outputs
// and coefficient selects in the loop, one wave per SIMD, that this one replaced
// (4096000 rows, us before -> now, complex64 / complex128): 64 -> 32 1030 -> 670 /
// 1935 -> 1285 (4.9 TB/s), 64 -> 48 1250 -> 925 / 2600 -> 1772, 64 -> 16 580 -> 493 /
// 1072 -> 1000, 16 -> 16 192 -> 181 / 380 -> 375; 262144 rows, 56 -> 28 76 -> 43 /
// 177 -> 84; 1000003 rows, 20 -> 5 complex64 accumulated 56 -> 38.5.
//
// A wave reads every input of its rows before it writes them (the slabs of a
// later group are other rows), so Out may alias any input.
#pragma once
#include "device_math.h"
#include "update_cols.h"

namespace gplhr {

template <typename T>
struct UpdArgs {
    int64_t n;
    T *out;
    int ldo, wout, ocol, split, ocol2;
    double2 beta;
    int nterms;
    UpdTerm<T> t[3];
    int wtot;
    const T *add;    // added block (column c at add[c]) or null
    int ldadd;
};

// With what update_stream_kernel takes besides: a struct of its own, as a launch's
// argument bytes cost time (these 224 took 0.25 us of update_mfma_kernel's 5 on small
// blocks).
template <typename T>
struct UpdStreamArgs : UpdArgs<T> {
    // the slabs of 8 input columns of all terms in order
    struct Slab {
        const void *p;   // row 0, the slab's first column
        int64_t ldb;     // bytes of a row
        int lim;         // columns the slab holds (1..8)
    } slab[8];
    unsigned scaled;     // bit i: slab i takes the row scale rs
    unsigned waves, nw;  // waves of a workgroup, of the launch
    const T *rs;
};

template <typename T> struct UpdMma;
template <> struct UpdMma<double2> {
    using R = double;
    using V = d4v;
    static __device__ __forceinline__ V mma(R a, R b, V c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    // accumulator register v of lane (i, k) holds output row 4v + k
    static __device__ __forceinline__ int row(int v, int k) { return 4 * v + k; }
    // matrix row of part p of entry c of a tile: a lane's registers are entry k
    // (0, 1) and entry 4 + k (2, 3)
    static __device__ __forceinline__ int place(int c, int p) { return 8 * (c >> 2) + 4 * p + (c & 3); }
    static __device__ __forceinline__ int entry(int h, int k) { return 4 * h + k; }
};
template <> struct UpdMma<float2> {
    using R = float;
    using V = f4v;
    static __device__ __forceinline__ V mma(R a, R b, V c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    // accumulator register v of lane (i, k) holds output row 4k + v
    static __device__ __forceinline__ int row(int v, int k) { return 4 * k + v; }
    // a lane's registers are entries 2k and 2k + 1
    static __device__ __forceinline__ int place(int c, int p) { return 2 * c + p; }
    static __device__ __forceinline__ int entry(int h, int k) { return 2 * k + h; }
};

__host__ __device__ __forceinline__ int pad8(int w) { return (w + 7) & ~7; }

// NT: output tiles of 8 columns; SL: slabs (the last one may be absent).
// BETA: Out is read.  TRI: the first term's coefficients are upper triangular
// and fill NT slabs, so slab i meets only the tiles nt >= i.  RAG: a term's last
// slab may hold fewer than 8 columns.  SCL: slabs of a.scaled take the row
// scale.  VEC: complex64 entries are moved in pairs of 16 bytes (even widths,
// offsets and leading dimensions).  A row group is 16 MT rows: MT = 2 for
// complex64 of up to two slabs, whose 2 KiB per 16 rows leave too little in
// flight (16 -> 16 columns, 4096000 rows: 232 us with one).
// RUN: the outputs pass through a tile of LDS and leave row after row, past the caches if
// nts (pieces never do: update_stream).
template <typename T, int NT, int SL, bool BETA, bool TRI, bool RAG, bool SCL, bool VEC, bool RUN = false>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 8)))
void update_stream_kernel(UpdStreamArgs<T> a, int nslab, int nts) {
    using M = UpdMma<T>;
    using R = typename M::R;
    using V = typename M::V;
    constexpr int MT = sizeof(T) == 8 && SL == 2 ? 2 : 1, ROWS = 16 * MT;
    static_assert(!RUN || (VEC && !BETA && !SCL), "runs of 16-byte pieces, overwriting");
    extern __shared__ double2 sh_upd_stream[];
    R *sM = reinterpret_cast<R *>(sh_upd_stream);   // [slab][step][tile][lane]
    {
        const int p0 = pad8(a.t[0].w), p1 = a.nterms > 1 ? pad8(a.t[1].w) : 0;
        for (int e = threadIdx.x; e < nslab * 8 * 8 * NT; e += a.waves * 64) {
            const int j = e / (8 * NT), c = e - j * (8 * NT);
            int t = 0, jj = j;
            if (jj >= p0) {
                jj -= p0;
                t = 1;
                if (jj >= p1) { jj -= p1; t = 2; }
            }
            T v = czero<T>();
            if (t < a.nterms && c < a.wout && jj < a.t[t].w)
                v = from_d<T>(cmul(a.t[t].alpha, a.t[t].M[jj + (int64_t)c * a.t[t].ldm]));
            // input entry j: lane group (j % 8) / 2, steps 2 (j % 2) (its real
            // part) and 2 (j % 2) + 1 (its imaginary part)
            R *d = sM + (((j >> 3) * 4 + 2 * (j & 1)) * NT + (c >> 3)) * 64 + ((j & 7) >> 1) * 16;
            const int re = M::place(c & 7, 0), im = M::place(c & 7, 1);
            d[re] = v.x;
            d[im] = v.y;
            d[NT * 64 + re] = -v.y;
            d[NT * 64 + im] = v.x;
        }
        __syncthreads();
    }
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int li = lane & 15, lk = lane >> 4;
    const bool last = nslab == SL;
    // whole row groups, this wave's first one and the distance of its groups
    // (32-bit and uniform by readfirstlane: comparisons of 64 bits are vector
    // instructions, and what depends on them would be too)
    const uint32_t ngrp = (uint32_t)(a.n / ROWS);
    const uint32_t nw = __builtin_amdgcn_readfirstlane(a.nw);
    const uint32_t w0 = __builtin_amdgcn_readfirstlane(blockIdx.x * a.waves + wave);
    // per slab: the next group's first row (advanced by the scalar unit) and
    // the byte offsets of the lane's two entries in a group; entries past the
    // term's width read its slab's first one (complex64 in pairs: first pair)
    // and enter as zeros
    const char *next[SL];
    uint32_t off[SL][2];
#pragma unroll
    for (int i = 0; i < SL; ++i) {
        const auto &sb = a.slab[i];
        next[i] = static_cast<const char *>(sb.p) + (int64_t)min(w0, ngrp) * ROWS * sb.ldb;
#pragma unroll
        for (int h = 0; h < 2; ++h)
            off[i][h] = (uint32_t)(li * sb.ldb) +
                        (uint32_t)(upd_slab_column(RAG ? sb.lim : 8, lk, h, VEC && sizeof(T) == 8) * sizeof(T));
    }
    // Output pieces.  A lane's registers hold pieces of row li that are 64 bytes
    // of a tile apart (complex128: entries lk and 4 + lk) or in two neighbouring
    // tiles (complex64 pairs).  Lanes li and li ^ 8 exchange one of each two, so
    // that every store instruction writes 128 consecutive bytes of 8 rows: then
    // lane li holds piece li / 8 of rows li % 8 and 8 + li % 8.  (Complex64 entries
    // moved one by one, and a last odd tile, are stored from where they are.)
    constexpr bool SWAP = VEC && !RUN, PAIR = SWAP && sizeof(T) == 8;
    constexpr int NP = PAIR ? NT / 2 : NT;   // exchanged pairs
    const int64_t ldob = (int64_t)a.ldo * sizeof(T);
    const int lp = li >> 3;
    auto col_off = [&](int c) { return (uint32_t)((c < a.split ? a.ocol + c : a.ocol2 + c - a.split) * sizeof(T)); };
    int pc[NP > 0 ? NP : 1];                 // output column of the lane's piece
    uint32_t pof[NP > 0 ? NP : 1], oof[NT][2];
#pragma unroll
    for (int q = 0; q < NP; ++q) {
        pc[q] = PAIR ? (2 * q + lp) * 8 + M::entry(0, lk) : q * 8 + M::entry(lp, lk);
        pof[q] = (uint32_t)((li & 7) * ldob) + col_off(pc[q]);
    }
#pragma unroll
    for (int nt = SWAP ? (PAIR ? 2 * NP : NT) : 0; nt < NT; ++nt)
#pragma unroll
        for (int h = 0; h < 2; ++h) oof[nt][h] = (uint32_t)(li * ldob) + col_off(nt * 8 + M::entry(h, lk));
    // RUN: a wave's tile of ROWS rows of 16-byte pieces, and the places of the lane's
    // piece of its it-th store in the tile and in Out
    constexpr int PE = 16 / (int)sizeof(T), NIT = RUN ? ROWS * NT * 8 / PE / 64 : 1;
    constexpr int LDT = NT * 8 / PE + 1;     // pieces of a tile row (odd: rows spread over the banks)
    f4v *tile = nullptr;
    uint32_t tof[NIT], gof[NIT], grow[NIT];
    if constexpr (RUN) {
        tile = reinterpret_cast<f4v *>(sM + nslab * 4 * NT * 64) + wave * (ROWS * LDT);
        const int wp = a.wout / PE;
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            const int e = it * 64 + lane, row = e / wp, c = e - row * wp;
            tof[it] = row < ROWS ? row * LDT + c : 0;
            grow[it] = row;
            gof[it] = (uint32_t)(min(row, ROWS - 1) * ldob) + col_off(c * PE);
        }
    }
    const T beta = from_d<T>(a.beta);
    T x[SL][MT][2];
    auto load = [&](int i, int rows) {   // rows past the `rows` of the last, partial group repeat its last one
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const char *p = next[i] + (16 * mt - (rows < ROWS ? max(16 * mt + li - (rows - 1), 0) : 0)) * a.slab[i].ldb;
            if constexpr (VEC && sizeof(T) == 8) {
                const float4 v = *reinterpret_cast<const float4 *>(p + off[i][0]);
                x[i][mt][0] = make_float2(v.x, v.y);
                x[i][mt][1] = make_float2(v.z, v.w);
            } else {
                x[i][mt][0] = *reinterpret_cast<const T *>(p + off[i][0]);
                x[i][mt][1] = *reinterpret_cast<const T *>(p + (RAG ? off[i][1] : off[i][0] + (uint32_t)sizeof(T)));
            }
        }
    };
    const R *m = sM + lane;
    // one group: rows of it that exist, rows to its next group (prefetched)
    auto group = [&](int64_t g, int rows, bool more, int step) {
        // the coefficients stay in LDS: read once before the loop they would
        // take (and spill) hundreds of registers
        asm volatile("" ::: "memory");
        V acc[MT][NT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = V{0, 0, 0, 0};
        char *po = reinterpret_cast<char *>(a.out) + g * ldob;
        // the exchanged piece q of half-group hf (8 rows each), and entry (nt, h)
        auto at = [&](int hf, int q) { return reinterpret_cast<f4v *>(po + 8 * hf * ldob + pof[q]); };
        auto mine = [&](int hf, int q) { return pc[q] < a.wout && 8 * hf + (li & 7) < rows; };
        auto at1 = [&](int mt, int nt, int h) { return po + 16 * mt * ldob + oof[nt][h]; };
        auto mine1 = [&](int mt, int nt, int h) { return nt * 8 + M::entry(h, lk) < a.wout && 16 * mt + li < rows; };
        f4v bp[2 * MT][BETA && NP > 0 ? NP : 1];
        T bd[MT][BETA ? NT : 1][2], rs[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            if constexpr (BETA) {
#pragma unroll
                for (int hf = 2 * mt; hf < 2 * mt + 2; ++hf)
#pragma unroll
                    for (int q = 0; q < NP; ++q)
                        if (SWAP) {
                            bp[hf][q] = f4v{0, 0, 0, 0};
                            if (mine(hf, q)) bp[hf][q] = *at(hf, q);
                        }
#pragma unroll
                for (int nt = SWAP ? (PAIR ? 2 * NP : NT) : 0; nt < NT; ++nt)
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        bd[mt][nt][h] = czero<T>();
                        if (mine1(mt, nt, h)) bd[mt][nt][h] = *reinterpret_cast<const T *>(at1(mt, nt, h));
                    }
            }
            if constexpr (SCL) rs[mt] = a.rs[g + min(16 * mt + li, rows - 1)];
        }
        auto slab = [&](int i) {
            T xi[MT][2];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    xi[mt][h] = x[i][mt][h];
                    if constexpr (SCL)
                        if (a.scaled >> i & 1) xi[mt][h] = cmul(rs[mt], xi[mt][h]);
                    if constexpr (RAG)
                        if (2 * lk + h >= a.slab[i].lim) xi[mt][h] = czero<T>();
                }
#pragma unroll
            for (int s = 0; s < 4; ++s) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    if (!(TRI && i < NT && nt < i)) {
                        const R cv = m[((i * 4 + s) * NT + nt) * 64];
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt)
                            acc[mt][nt] = M::mma(cv, (s & 1) ? xi[mt][s >> 1].y : xi[mt][s >> 1].x, acc[mt][nt]);
                    }
            }
            if (more) {
                next[i] += (int64_t)step * a.slab[i].ldb;
                load(i, ROWS);
            }
        };
#pragma unroll
        for (int i = 0; i < SL - 1; ++i) slab(i);
        if (last) slab(SL - 1);
        auto add_beta = [&](T &o, const T &d) {
            o.x += beta.x * d.x - beta.y * d.y;
            o.y += beta.x * d.y + beta.y * d.x;
        };
        if constexpr (RUN) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    const V d = acc[mt][nt];
                    f4v *row = tile + (16 * mt + li) * LDT + nt * 8 / PE;
                    if constexpr (sizeof(T) == 8) row[lk] = f4v{d[0], d[1], d[2], d[3]};
                    else {
                        row[lk] = __builtin_bit_cast(f4v, make_double2(d[0], d[1]));
                        row[4 + lk] = __builtin_bit_cast(f4v, make_double2(d[2], d[3]));
                    }
                }
            // LDS operations of a wave complete in order
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int it = 0; it < NIT; ++it)
                if ((int)grow[it] < rows) {
                    const f4v o = tile[tof[it]];
                    f4v *dst = reinterpret_cast<f4v *>(po + gof[it]);
                    // (empty asm: two plain branches would be merged into one store
                    // without the hint)
                    if (nts) {
                        asm volatile("");
                        __builtin_nontemporal_store(o, dst);
                        asm volatile("");
                    } else {
                        *dst = o;
                    }
                }
            // the next group's tile may not overtake these reads
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            return;
        }
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
            for (int q = 0; q < NP; ++q) {
                if constexpr (SWAP) {
                    // pieces c[0], c[1] of row li as 32-bit words
                    int c[2][4];
                    const V d0 = PAIR ? acc[mt][2 * q] : acc[mt][q], d1 = PAIR ? acc[mt][2 * q + 1] : acc[mt][q];
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        if constexpr (PAIR) {
                            c[0][v] = __float_as_int(d0[v]);
                            c[1][v] = __float_as_int(d1[v]);
                        } else {
                            c[0][v] = (v & 1) ? __double2hiint(d0[v >> 1]) : __double2loint(d0[v >> 1]);
                            c[1][v] = (v & 1) ? __double2hiint(d0[2 + (v >> 1)]) : __double2loint(d0[2 + (v >> 1)]);
                        }
                        // from lane li ^ 8 (16 lanes rotated by 8)
                        const int got = __builtin_amdgcn_update_dpp(0, lp ? c[0][v] : c[1][v], 0x128, 0xf, 0xf, false);
                        c[0][v] = lp ? got : c[0][v];
                        c[1][v] = lp ? c[1][v] : got;
                    }
#pragma unroll
                    for (int hf = 0; hf < 2; ++hf) {
                        f4v o{__int_as_float(c[hf][0]), __int_as_float(c[hf][1]), __int_as_float(c[hf][2]),
                              __int_as_float(c[hf][3])};
                        if constexpr (BETA) {
                            const f4v d = bp[2 * mt + hf][q];
                            if constexpr (PAIR) {
                                T e0 = make_float2(o.x, o.y), e1 = make_float2(o.z, o.w);
                                add_beta(e0, make_float2(d.x, d.y));
                                add_beta(e1, make_float2(d.z, d.w));
                                o = f4v{e0.x, e0.y, e1.x, e1.y};
                            } else {
                                double2 e = __builtin_bit_cast(double2, o);
                                add_beta(e, __builtin_bit_cast(double2, d));
                                o = __builtin_bit_cast(f4v, e);
                            }
                        }
                        if (mine(2 * mt + hf, q)) *at(2 * mt + hf, q) = o;
                    }
                }
            }
#pragma unroll
            for (int nt = SWAP ? (PAIR ? 2 * NP : NT) : 0; nt < NT; ++nt)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    T o;
                    o.x = acc[mt][nt][2 * h];
                    o.y = acc[mt][nt][2 * h + 1];
                    if constexpr (BETA) add_beta(o, bd[mt][nt][h]);
                    if (mine1(mt, nt, h)) {
                        typedef R r2n __attribute__((ext_vector_type(2)));
                        *reinterpret_cast<r2n *>(at1(mt, nt, h)) = r2n{o.x, o.y};
                    }
                }
        }
    };
    if (w0 < ngrp) {
#pragma unroll
        for (int i = 0; i < SL - 1; ++i) load(i, ROWS);
        if (last) load(SL - 1, ROWS);
        // after its last group a wave reads that group again (unused)
        for (uint32_t w = w0; w < ngrp; w += nw)
            group((int64_t)w * ROWS, ROWS, true, w + nw < ngrp ? (int)nw * ROWS : 0);
    }
    const int rest = (int)(a.n % ROWS);
    if (rest && w0 == ngrp % nw) {
#pragma unroll
        for (int i = 0; i < SL; ++i)
            if (i < SL - 1 || last) {
                next[i] = static_cast<const char *>(a.slab[i].p) + (int64_t)ngrp * ROWS * a.slab[i].ldb;
                load(i, rest);
            }
        group((int64_t)ngrp * ROWS, rest, false, 0);
    }
}

template <typename T> using UpdFn = void (*)(UpdStreamArgs<T>, int, int);
struct UpdKind {
    bool beta, tri, rag, scl, vec, run;
};
// Most coefficient tiles (slabs by output tiles) of a run kernel.
constexpr int UPD_RUN_TILES = 40;
// The kernel for nt output tiles and sl slabs, or null.  At the limit of 256 registers
// three complex128 ones spill 12 to 36 bytes a lane: 8 slabs by 5 and by 6 tiles
// accumulated into Out, 8 by 6 row-scaled.
template <typename T> UpdFn<T> update_pick(int nt, int sl, UpdKind k);

template <typename T, int NT, int SL>
UpdFn<T> update_pick_shape(UpdKind k) {
    // kernel<T, NT, SL, BETA, TRI, RAG, SCL, VEC>
    if constexpr (sizeof(T) == 8) {
        if (!k.vec) {
            if (k.scl) return k.beta ? nullptr : update_stream_kernel<T, NT, SL, false, false, true, true, false>;
            return k.beta ? update_stream_kernel<T, NT, SL, true, false, true, false, false>
                          : update_stream_kernel<T, NT, SL, false, false, true, false, false>;
        }
    }
    if (k.scl) return k.beta ? nullptr : update_stream_kernel<T, NT, SL, false, false, true, true, true>;
    if (k.beta) return update_stream_kernel<T, NT, SL, true, false, true, false, true>;
    if (k.run) {
        if constexpr (NT * (SL - 1) > UPD_RUN_TILES) return nullptr;   // SL - 1 slabs or SL
        else {
            if constexpr (NT >= 2 && NT <= SL)
                if (k.tri) return update_stream_kernel<T, NT, SL, false, true, true, false, true, true>;
            return update_stream_kernel<T, NT, SL, false, false, true, false, true, true>;
        }
    }
    if constexpr (NT >= 2 && NT <= SL)
        if (k.tri)
            return k.rag ? update_stream_kernel<T, NT, SL, false, true, true, false, true>
                         : update_stream_kernel<T, NT, SL, false, true, false, false, true>;
    return k.rag ? update_stream_kernel<T, NT, SL, false, false, true, false, true>
                 : update_stream_kernel<T, NT, SL, false, false, false, false, true>;
}
template <typename T, int NT>
UpdFn<T> update_pick_slabs(int sl, UpdKind k) {
    if (sl <= 2) return update_pick_shape<T, NT, 2>(k);
    if (sl <= 4) return update_pick_shape<T, NT, 4>(k);
    if (sl <= 6) return update_pick_shape<T, NT, 6>(k);
    return update_pick_shape<T, NT, 8>(k);
}
template <typename T>
UpdFn<T> update_pick_impl(int nt, int sl, UpdKind k) {
    if (sl < 1 || sl > 8) return nullptr;
    switch (nt) {
        case 1: return update_pick_slabs<T, 1>(sl, k);
        case 2: return update_pick_slabs<T, 2>(sl, k);
        case 3: return update_pick_slabs<T, 3>(sl, k);
        case 4: return update_pick_slabs<T, 4>(sl, k);
        case 5: return update_pick_slabs<T, 5>(sl, k);
        case 6: return update_pick_slabs<T, 6>(sl, k);
    }
    return nullptr;
}

}  // namespace gplhr
