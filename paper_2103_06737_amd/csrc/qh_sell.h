// Sparse products y_i = sum_j a_ij x_j for the solvers (FP64 or FP32 values and vectors, FP64
// products and sums) and the learned factor (BF16 entries); shared by qh_solver.hip and
// qh_learned.hip.
//
// Layout: rows in slices of 64, one row per lane of a wave; entry k of a slice's 64 rows is stored
// side by side (shorter rows padded with zero values on their own first column), so a wave reads a
// slice's values and columns coalesced, sums each row in its lane's registers and needs neither LDS
// nor a block barrier. The edge unknowns are numbered on the device so that the 64 rows of a slice
// are edges of one kind at consecutive nodes (HostMesh::order): the k-th entries of a slice then
// gather from a few runs of neighbouring vector entries. What bounds the products is the gathers'
// misses in the first-level cache; the entries of a tile of rows in storage order (products in LDS,
// then one thread per row) touched about 25 cache lines per 64 gathers, these slices about 4 on
// the box meshes (8.5 with the rows in edge-number order; 1024-node groups instead of 256: 3.8, but
// the columns of a slice then no longer fit four windows at 96^3).
#pragma once

#include <type_traits>

#include "qh_internal.h"

constexpr int kSlice = 64;                     // rows per slice: one per lane
constexpr int kSellThreads = 512;
constexpr int kSellWaves = kSellThreads / 64;  // slices a block works on side by side
// Entries of the learned factor in flight per lane: a whole row (at most 16 on the box meshes) of a
// small matrix, fewer for larger ones (more waves).
constexpr int kUPrec = 8, kUPrecAll = 16;
constexpr int kSellPad = 20 * kSlice;          // entries past the last that rounds of loads may touch
constexpr int kSellOneWidth = 2048;            // matrices of at most this many slices get one width for all
constexpr int kSellMaxBlocks = 1024;           // 8192 waves: what the 256 CUs hold at eight waves per SIMD

// Slices of a CSR matrix. rows: matrix row of each position (null: the same), cpos: gather index
// of each column (null: the same). Row entries keep their order.
void qh_build_sell(int32_t n, const int32_t *ptr, const int32_t *col, const int32_t *rows, const int32_t *cpos,
                   SellHost &out);

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

// Every wave gets the same number of slices, as few waves as that needs: at 64^3 (28,100 slices)
// 879 blocks of eight waves with four slices each.
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

__device__ __forceinline__ int4 sell_base(const SellCols &S, int32_t s) {
    const int4 v = S.base[s];
    return make_int4(__builtin_amdgcn_readfirstlane(v.x), __builtin_amdgcn_readfirstlane(v.y),
                     __builtin_amdgcn_readfirstlane(v.z), __builtin_amdgcn_readfirstlane(v.w));
}

// Gather index of a 16-bit column.
__device__ __forceinline__ int32_t sell_col(uint32_t h, int4 base) {
    const uint32_t q = h >> 14;
    return (q == 0 ? base.x : q == 1 ? base.y : q == 2 ? base.z : base.w) + (int32_t)(h & 0x3fffu);
}

// Rounds of U entries per lane: U entries' loads, then U gathers are in flight together. Loads run
// past a slice's end without a test (the arrays have kSellPad entries to spare), at constant
// distances from one address per array; gathers past it take column `safe`, and their terms are
// left out.
template <int U>
__device__ __forceinline__ void sell_cols(const SellCols &S, int32_t o0, int32_t left, int4 base, int32_t lane,
                                          int32_t safe, int32_t (&c)[U]) {
    static_assert(U * kSlice <= kSellPad, "a round stays inside the padding");
    if (base.x >= 0) {
        const uint16_t *cp = S.c16 + (int64_t)o0 * kSlice + lane;
#pragma unroll
        for (int u = 0; u < U; ++u) c[u] = cp[u * kSlice];
#pragma unroll
        for (int u = 0; u < U; ++u) c[u] = u < left ? sell_col((uint32_t)c[u], base) : safe;
    } else {
        const int32_t *cp = S.c32 + (int64_t)o0 * kSlice + lane;
#pragma unroll
        for (int u = 0; u < U; ++u) c[u] = cp[u * kSlice];
#pragma unroll
        for (int u = 0; u < U; ++u) c[u] = u < left ? c[u] : safe;
    }
}

// op(value, x) for every entry of this lane's row of slice s, in the row's order (padding: zero
// values). part of parts: the entries k of [w part / parts, w (part + 1) / parts) only.
template <int U, typename VT, typename XT, typename Op>
__device__ __forceinline__ void sell_each(const SellCols &S, const VT *__restrict__ val, const XT *__restrict__ x,
                                          int32_t s, Op &&op, int32_t part = 0, int32_t parts = 1) {
    const int32_t lane = (int32_t)(threadIdx.x & 63);
    int32_t o0, w;
    sell_extent(S, s, o0, w);
    if (parts > 1) {
        const int32_t lo = w * part / parts, hi = w * (part + 1) / parts;
        o0 += lo;
        w = hi - lo;
    }
    const int4 base = sell_base(S, s);
    for (; w > 0; w -= U, o0 += U) {
        const VT *vp = val + (int64_t)o0 * kSlice + lane;
        VT v[U];
        int32_t c[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = vp[u * kSlice];
        sell_cols<U>(S, o0, w, base, lane, 0, c);
        XT xv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) xv[u] = x[c[u]];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (u < w) op(sell_val(v[u]), (double)xv[u]);
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

// The same with BF16 entries packed with their 16-bit columns (value bits << 16 | column), one
// load per entry; in a slice without 16-bit columns the low half is unused.
template <int U, typename XT>
__device__ __forceinline__ double sell_dot_pk(const SellCols &S, const uint32_t *__restrict__ pk,
                                              const XT *__restrict__ x, int32_t s) {
    const int32_t lane = (int32_t)(threadIdx.x & 63);
    int32_t o0, w;
    sell_extent(S, s, o0, w);
    const int4 base = sell_base(S, s);
    double acc = 0.0;
    for (; w > 0; w -= U, o0 += U) {
        const uint32_t *ep = pk + (int64_t)o0 * kSlice + lane;
        uint32_t e[U];
        int32_t c[U];
#pragma unroll
        for (int u = 0; u < U; ++u) e[u] = ep[u * kSlice];
        if (base.x >= 0) {
#pragma unroll
            for (int u = 0; u < U; ++u) c[u] = u < w ? sell_col(e[u] & 0xffffu, base) : 0;
        } else {
            sell_cols<U>(S, o0, w, base, lane, 0, c);
        }
        XT xv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) xv[u] = x[c[u]];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (u < w) acc = fma((double)__uint_as_float(e[u] & 0xffff0000u), (double)xv[u], acc);
    }
    return acc;
}
