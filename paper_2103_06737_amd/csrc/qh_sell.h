// Sparse products y_i = sum_j a_ij x_j for the solvers (FP64 or FP32 values and vectors, FP64
// products and sums) and the learned factor (BF16 entries); shared by qh_solver.hip and
// qh_learned.hip.
//
// Layout: rows in slices of 64, one row per lane of a wave; entry k of a slice's 64 rows is stored
// side by side (shorter rows padded with zero values on columns of their own), so a wave reads a
// slice's values and columns coalesced, sums each row in its lane's registers and needs neither LDS
// nor a block barrier. The edge unknowns are numbered on the device so that the 64 rows of a slice
// are edges of one kind at consecutive nodes, or neighbours in space on meshes whose nodes are not numbered
// line by line (HostMesh::order): the k-th entries of a slice then
// gather from a few runs of neighbouring vector entries. What bounds the products is the gathers'
// misses in the first-level cache; the entries of a tile of rows in storage order (products in LDS,
// then one thread per row) touched about 25 cache lines per 64 gathers, these slices about 4 on
// the box meshes (8.5 with the rows in edge-number order). Columns are 16 bits from a scalar base per slice entry, and a
// round of loads has exactly as many entries as it needs: with four column windows per slice to select
// from and a test per entry, the products at 64^3 (FP32, learned; us) took 54.4 for A, 28.9 for the
// update with G, 23.0 for G^T, now 50.6, 24.9, 19.9; at 48^3 19.4, 12.9, 10.3, now 16.3, 10.9, 8.3.
// At 64^3 the three read and write about 406 MB with their vectors, more than the last-level cache holds, at
// 4.3 TB/s (counted in HBM: 222 + 123 + 82 MB).
#pragma once

#include <type_traits>

#include "qh_internal.h"

constexpr int kSlice = 64;                     // rows per slice: one per lane
constexpr int kSellThreads = 512;
constexpr int kSellWaves = kSellThreads / 64;  // slices a block works on side by side
// Entries of the learned factor in flight per lane: a whole row (at most 16 on the box meshes) of a
// small matrix, fewer for larger ones (more waves). 5 / 8 / 12 / 16 for the update with G: 26.8 / 24.9 /
// 28.0 / 28.0 us at 64^3, 11.7 / 10.9 / 10.4 / 14.1 at 48^3.
constexpr int kUPrec = 8, kUPrecAll = 16;
constexpr int kSellOneWidth = 2048;            // matrices of at most this many slices get one width for all
constexpr int kSellMaxBlocks = 1024;           // 8192 waves: what the 256 CUs hold at eight waves per SIMD

// Slices of a CSR matrix. rows: matrix row of each position (null: the same), cpos: gather index
// of each column (null: the same), wide: 32-bit columns throughout, packed: short rows from the first slot
// on instead of beside the longest row's entries (where the rows of a slice have nothing to do with each other,
// that takes time and gains none: 100,000 Delaunay points 3.34 -> 2.97 s for the assembly, the same products).
// Row entries keep their order.
void qh_build_sell(int32_t n, const int32_t *ptr, const int32_t *col, const int32_t *rows, const int32_t *cpos,
                   SellHost &out, bool wide = false, bool packed = false);

// Sum over the wave's 64 lanes, the same in every lane: shifts within rows of 16, then across rows, as
// data-parallel moves (a shuffle through LDS costs several times a move's latency, six in a chain:
// about 0.2 us of a solver kernel's 3 to 7 us).
template <int CTRL, int ROWS>
__device__ __forceinline__ double wave_move(double v) {
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, ROWS, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROWS, 0xf, true);
    return __builtin_bit_cast(double, (long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}
__device__ __forceinline__ double wave_sum(double v) {
    v += wave_move<0x111, 0xf>(v);  // row_shr:1, 2, 4, 8: lane 15 of each row has the row's sum
    v += wave_move<0x112, 0xf>(v);
    v += wave_move<0x114, 0xf>(v);
    v += wave_move<0x118, 0xf>(v);
    v += wave_move<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
    v += wave_move<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3: lane 63 has the total
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_readlane((int)b, 63), hi = __builtin_amdgcn_readlane((int)(b >> 32), 63);
    return __builtin_bit_cast(double, (long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}

// Entry values: FP64, FP32, or BF16 (the high half of a packed word), all widened to FP64.
__device__ __forceinline__ double sell_val(double v) { return v; }
__device__ __forceinline__ double sell_val(float v) { return (double)v; }

// Slices of this wave: begin, begin + step, ... below end. The block index is remapped so that each
// of the 8 XCDs (which receive blocks round-robin) covers one contiguous span of slices, and an
// XCD's waves take consecutive slices at a time: they sweep the span together, so that the vector
// entries that neighbouring slices share stay in the XCD's L2 although the matrix streams through
// it. Grids (sell_grid) are multiples of 8.
struct SellRange {
    int32_t begin, end, step;
};
__device__ __forceinline__ SellRange sell_range(int32_t ns) {
    const int32_t per_x = (int32_t)gridDim.x / 8, xcd = (int32_t)blockIdx.x & 7;
    const int32_t span = (ns + 7) / 8;
    const int32_t w = ((int32_t)blockIdx.x >> 3) * kSellWaves + (int32_t)(threadIdx.x >> 6);
    SellRange r;
    r.begin = __builtin_amdgcn_readfirstlane(xcd * span + w);
    r.end = (xcd + 1) * span < ns ? (xcd + 1) * span : ns;
    r.step = per_x * kSellWaves;
    return r;
}

// Every wave gets the same number of slices, as few waves as that needs: at 64^3 (28,099 slices)
// 880 blocks of eight waves with four slices each.
inline unsigned sell_grid(int32_t ns) {
    const int64_t most = (int64_t)kSellMaxBlocks * kSellWaves;
    const int64_t per = ns > most ? (ns + most - 1) / most : 1;
    const int64_t waves = (ns + per - 1) / per;
    const int64_t b = (waves + kSellWaves - 1) / kSellWaves;
    return (unsigned)(b < 8 ? 8 : (b + 7) / 8 * 8);
}

// Where slice s's entries start (units of 64) and how many each row has. Small matrices have one
// width for all slices, so that the address of the first entries needs no load.
__device__ __forceinline__ void sell_extent(const SellCols &S, int32_t s, int32_t &o0, int32_t &w) {
    if (S.width > 0) {
        o0 = s * S.width;
        w = S.width;
    } else {
        o0 = __builtin_amdgcn_readfirstlane(S.off[s]);
        w = __builtin_amdgcn_readfirstlane(S.off[s + 1]) - o0;
    }
}

// What the 16-bit columns of the slice entries from o0 on count from, -1: they are 32-bit. Read-only
// and the same for the whole wave: scalar loads and registers.
typedef const __attribute__((address_space(4))) int32_t *SellScalars;
__device__ __forceinline__ SellScalars sell_bases(const SellCols &S, int32_t o0) {
    return (SellScalars)(uintptr_t)(S.base + o0);
}

// A round of H entries per lane: their loads, then H gathers, are in flight together. With 16-bit
// columns a gather's address is a scalar one (x + base) and a 32-bit offset.
template <int H, typename VT, typename XT, typename Op>
__device__ __forceinline__ void sell_round(const SellCols &S, const VT *__restrict__ val, const XT *__restrict__ x,
                                           int32_t o0, bool wide, Op &op) {
    const uint32_t lane = threadIdx.x & 63;
    const int64_t e0 = (int64_t)o0 * kSlice;
    const VT *vp = val + e0;
    VT v[H];
    XT xv[H];
#pragma unroll
    for (int u = 0; u < H; ++u) v[u] = vp[u * kSlice + lane];
    if (!wide) {
        const uint16_t *cp = S.c16 + e0;
        const SellScalars base = sell_bases(S, o0);
        uint32_t c[H];
#pragma unroll
        for (int u = 0; u < H; ++u) c[u] = cp[u * kSlice + lane];
#pragma unroll
        for (int u = 0; u < H; ++u) xv[u] = (x + base[u])[c[u]];
    } else {
        const int32_t *cp = S.c32 + e0;
        int32_t c[H];
#pragma unroll
        for (int u = 0; u < H; ++u) c[u] = cp[u * kSlice + lane];
#pragma unroll
        for (int u = 0; u < H; ++u) xv[u] = x[c[u]];
    }
#pragma unroll
    for (int u = 0; u < H; ++u) op(sell_val(v[u]), (double)xv[u]);
}

// The same with BF16 entries packed with their 16-bit columns (value bits << 16 | column), one load
// per entry; in a slice without 16-bit columns the low half is unused.
template <int H, typename XT, typename Op>
__device__ __forceinline__ void sell_round(const SellCols &S, const uint32_t *__restrict__ pk,
                                           const XT *__restrict__ x, int32_t o0, bool wide, Op &op) {
    const uint32_t lane = threadIdx.x & 63;
    const int64_t e0 = (int64_t)o0 * kSlice;
    const uint32_t *ep = pk + e0;
    uint32_t e[H];
    XT xv[H];
#pragma unroll
    for (int u = 0; u < H; ++u) e[u] = ep[u * kSlice + lane];
    if (!wide) {
        const SellScalars base = sell_bases(S, o0);
#pragma unroll
        for (int u = 0; u < H; ++u) xv[u] = (x + base[u])[e[u] & 0xffffu];
    } else {
        const int32_t *cp = S.c32 + e0;
        int32_t c[H];
#pragma unroll
        for (int u = 0; u < H; ++u) c[u] = cp[u * kSlice + lane];
#pragma unroll
        for (int u = 0; u < H; ++u) xv[u] = x[c[u]];
    }
#pragma unroll
    for (int u = 0; u < H; ++u) op((double)__uint_as_float(e[u] & 0xffff0000u), (double)xv[u]);
}

// The round of h entries, 1 <= LO <= h <= HI: each length has its own straight code, found in
// log2(HI) scalar branches. (One code for all lengths, with a test per entry, became branches with
// waits for all loads between them.)
template <int LO, int HI, typename VT, typename XT, typename Op>
__device__ __forceinline__ void sell_pick(int32_t h, const SellCols &S, const VT *__restrict__ val,
                                          const XT *__restrict__ x, int32_t o0, bool wide, Op &op) {
    if constexpr (LO == HI) {
        sell_round<LO>(S, val, x, o0, wide, op);
    } else {
        constexpr int MID = (LO + HI) / 2;
        if (h <= MID) sell_pick<LO, MID>(h, S, val, x, o0, wide, op);
        else sell_pick<MID + 1, HI>(h, S, val, x, o0, wide, op);
    }
}

// op(value, x) for every entry of this lane's row of slice s, in the row's order (padding: zero
// values), in rounds of at most U entries, as equal as they can be. part of parts: the entries k of
// [w part / parts, w (part + 1) / parts) only.
template <int U, typename VT, typename XT, typename Op>
__device__ __forceinline__ void sell_each(const SellCols &S, const VT *__restrict__ val, const XT *__restrict__ x,
                                          int32_t s, Op &&op, int32_t part = 0, int32_t parts = 1) {
    int32_t o0, w;
    sell_extent(S, s, o0, w);
    if (parts > 1) {
        const int32_t lo = w * part / parts, hi = w * (part + 1) / parts;
        o0 += lo;
        w = hi - lo;
    }
    if (w <= 0) return;
    const bool wide = *sell_bases(S, o0) < 0;
    for (int32_t rounds = (w + U - 1) / U; rounds > 0; --rounds) {
        const int32_t h = (w + rounds - 1) / rounds;
        sell_pick<1, U>(h, S, val, x, o0, wide, op);
        o0 += h;
        w -= h;
    }
}

// This lane's row of slice s times x.
template <int U, typename VT, typename XT>
__device__ __forceinline__ double sell_dot(const SellCols &S, const VT *__restrict__ val, const XT *__restrict__ x,
                                           int32_t s) {
    double acc = 0.0;
    sell_each<U>(S, val, x, s, [&](double v, double xv) { acc = fma(v, xv, acc); });
    return acc;
}
