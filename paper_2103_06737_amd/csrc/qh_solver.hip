// Implicit field update on gfx950 (Sec. IV.B): FP64 products on slices of 64 rows, preconditioned conjugate
// gradients with FP64 dot products reduced in a fixed order (deterministic iteration counts),
// the Gauss-law solve for the non-solenoidal part and the integer Faraday update.
//
// Edge system (trapezoidal rule on eq. maxwell_semi, b^{n+1} eliminated):
//   ([*eps] + tau S) e* = ([*eps] - tau S) e^n + dt C^T [*mu^-1] b^n - u_q g,   tau = dt^2/4
// Gauss law (eq. discreteGauss): G^T [*eps] G delta = rho^{n+1} - G^T [*eps] e*, e = e* + G delta
// Faraday: b^{n+1} = b^n - C round((dt/2)(e^{n+1} + e^n)/u_b)  (D C = 0 keeps D b fixed).
#include <algorithm>
#include <cmath>

#include "qh_internal.h"
#include "qh_sell.h"

namespace {

constexpr int kThreads = kSellThreads;
constexpr int kMaxBlocks = kSellMaxBlocks;  // grids of the reducing kernels (fixed summation order)
static_assert(kMaxBlocks == 2 * kThreads, "a sum of partials takes two per thread");
// Entries in flight per lane. Small matrices (one width for all slices, one slice per wave): a
// launch is one chain of loads, so a row's entries (at most 19 on the box meshes) are issued
// together; larger ones: fewer registers, more waves. FP32 10: 7 / 8 / 12 take 48.4 / 56.3 / 51.1 us at
// 64^3 (10: 50.6) and 16.6 / 16.8 / 16.2 at 48^3 (16.3). FP64 8: 20 entries in the residual and the
// right-hand side at 48^3 take 32.6 and 48.0 us (8: 29.7, 42.4); 5 to 10 are alike.
constexpr int kU64 = 8;   // FP64 products
constexpr int kU32 = 10;  // FP32 products
constexpr int kUAll = 20; // small matrices

// device scalar slots of a CgWork: S_RZ + parity r.z (double-buffered), S_RR r.r, S_THR2 the
// target on r.r, S_BB b.b, S_RES the true-residual sums, S_SCALE the mixed-precision solve's
// residual scale, S_HIST a ring of r.r by iteration
// (the stall rule compares r.r with its value ten iterations before)
enum { S_RZ = 0, S_RZ1, S_RR, S_THR2, S_BB, S_RES = 8, S_SCALE = 10, S_HIST = 16, S_NSCAL = 32 };
constexpr int kHist = 16;
// flags[0] after a solve: why the iteration stopped
enum { CG_RUNNING = 0, CG_CONVERGED = 1, CG_STALLED = 2, CG_NONFINITE = 3 };
// stall rule of the learned solve: r.z <= 0, or ||r|| not 10 % lower than ten iterations before
constexpr int kStallWindow = 10;
constexpr double kStallRatio2 = 0.81;  // (1 - 0.1)^2 on r.r
// FP32 recurrence of the mixed-precision solve: the iterations between two reliable updates end, on the
// device, where r.r has fallen by this much since the last one. Batches are laid out for 1e-8 (1e-4 of
// the residual); far past that the vectors' rounding is what is left of r, and the recurrence no longer
// converges (a constant right-hand side, node system of 33^3 to 1e-12, its last 77 iterations in one
// segment: 20,000 iterations and a Jacobi restart; 141 so, 101 in FP64). Iterations of a point source on
// the node system of 32^3 to 1e-12 (FP64 102) with 1e-10 / 1e-9 / 1e-8: 226 / 163 / 142; with 1e-8 a
// step of the benchmark's kind stops just before its second update and takes a third (48^3, learned: 1961 / 1930
// / 2081 us).
constexpr double kSegment2 = 1e-9;

// Consecutive vector entries per thread in the element-wise kernels: 16 bytes.
template <typename T>
constexpr int kVec = 16 / (int)sizeof(T);
template <typename T>
inline unsigned grid_elems(int64_t n) {
    int64_t b = ((n + kVec<T> - 1) / kVec<T> + kThreads - 1) / kThreads;
    return (unsigned)(b < kMaxBlocks ? (b < 1 ? 1 : b) : kMaxBlocks);
}

// kVec consecutive entries of a vector: one 16-byte access inside the vector, single ones at its
// end.
template <typename T>
using Vec = T __attribute__((ext_vector_type(kVec<T>)));
template <typename T>
__device__ __forceinline__ Vec<T> load_vec(const T *__restrict__ p, int64_t i, int64_t n) {
    if (i + kVec<T> <= n) return *reinterpret_cast<const Vec<T> *>(p + i);
    Vec<T> v = (T)0;
#pragma unroll
    for (int q = 0; q < kVec<T>; ++q)
        if (i + q < n) v[q] = p[i + q];
    return v;
}
template <typename T>
__device__ __forceinline__ void store_vec(T *__restrict__ p, int64_t i, int64_t n, Vec<T> v) {
    if (i + kVec<T> <= n) {
        *reinterpret_cast<Vec<T> *>(p + i) = v;
        return;
    }
#pragma unroll
    for (int q = 0; q < kVec<T>; ++q)
        if (i + q < n) p[i + q] = v[q];
}

// ---------------------------------------------------------------------------------------
// CG kernels. Cross-block sums never use in-kernel synchronisation: a kernel writes one
// partial per block and every block of the NEXT kernel sums all partials itself in the same
// fixed order (a few KB from L2), so the result is identical in every block, deterministic,
// and needs no device-scope fence (which would write back the whole L2 on this part).
// Scalars: scal[S_RZ + parity] holds r.z of the current iterate (double-buffered by the
// iteration parity so no block reads a slot another block of the same kernel writes).

// This thread's share of part[0..m), m <= kMaxBlocks: two loads, issued where a kernel starts, so
// that they are in flight beside its first matrix and vector loads.
__device__ __forceinline__ double load_partials(const double *__restrict__ part, int m) {
    const int t = (int)threadIdx.x;
    const double a = t < m ? part[t] : 0.0;
    const double b = t + kThreads < m ? part[t + kThreads] : 0.0;
    return a + b;
}

// Block-wide sums of NV values per thread in a fixed order, returned to every thread.
template <int NV>
__device__ __forceinline__ void block_sums(double (&v)[NV], double (*sh)[kThreads / 64]) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        v[k] = wave_sum(v[k]);
        if (lane == 0) sh[k][wid] = v[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < kThreads / 64; ++w) t += sh[k][w];
        v[k] = t;
    }
}

// Every block: sum of part[0..m) in a fixed order, returned to all threads.
__device__ __forceinline__ double sum_partials(const double *__restrict__ part, int m, double (*sh)[kThreads / 64]) {
    double v[1] = {load_partials(part, m)};
    __syncthreads();  // a caller's earlier sum has been read
    block_sums<1>(v, sh);
    return v[0];
}

// Block-wide sum of NV values, written as this block's partials part[k * kMaxBlocks + block].
template <int NV>
__device__ __forceinline__ void write_partials(double (&v)[NV], double *__restrict__ part) {
    __shared__ double sh[NV][kThreads / 64];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const double s = wave_sum(v[k]);
        if (lane == 0) sh[k][wid] = s;
    }
    __syncthreads();
    if (threadIdx.x < NV) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < kThreads / 64; ++w) t += sh[threadIdx.x][w];
        part[threadIdx.x * kMaxBlocks + blockIdx.x] = t;
    }
}

// epi(row, product) for every row of this wave's slices.
template <int U, typename VT, typename XT, typename Epi>
__device__ __forceinline__ void sell_rows(int32_t n, int32_t ns, const SellCols &S, const VT *__restrict__ val,
                                          const XT *__restrict__ x, Epi &&epi) {
    const SellRange r = sell_range(ns);
    for (int32_t s = r.begin; s < r.end; s += r.step) {
        const double a = sell_dot<U>(S, val, x, s);
        const int32_t row = s * kSlice + (int32_t)(threadIdx.x & 63);
        if (row < n) epi(row, a);
    }
}

// init: r = b - A x, z = D^-1 r, p_old = 0; partials of r.z, r.r, b.b
template <int U>
__global__ void __launch_bounds__(kThreads) k_cg_init(int32_t n, int32_t ns, const SellCols S,
                                                      const double *__restrict__ val,
                                                      const double *__restrict__ x,
                                                      const double *__restrict__ b,
                                                      const double *__restrict__ dinv,
                                                      double *__restrict__ r, double *__restrict__ z,
                                                      double *__restrict__ p_old, double *__restrict__ part) {
    double acc[3] = {0.0, 0.0, 0.0};
    sell_rows<U>(n, ns, S, val, x, [&](int32_t row, double s) {
        const double bb = b[row];
        const double rr = bb - s;
        const double zz = rr * dinv[row];
        r[row] = rr;
        z[row] = zz;
        p_old[row] = 0.0;
        acc[0] += rr * zz;
        acc[1] += rr * rr;
        acc[2] += bb * bb;
    });
    write_partials<3>(acc, part);
}

// Why an iteration stops, from r.r and r.z of the present iterate (the same sums, so the same
// decision, in every block): non-finite values, convergence, and for the learned
// preconditioner the stall rule (r.z <= 0 means M is not positive definite on r; ||r|| less
// than 10 % lower than ten iterations before). hist: r.r by iteration (ring), or null.
__device__ __forceinline__ int cg_state(double rr, double rz, double thr2, int stall, int32_t k, const double *hist) {
    if (!(rr == rr) || !(rz == rz) || rr > 1.7976931348623157e308) return CG_NONFINITE;
    if (rr <= thr2) return CG_CONVERGED;
    if (stall) {
        if (!(rz > 0.0)) return CG_STALLED;
        if (hist && k >= kStallWindow && rr > kStallRatio2 * hist[(k - kStallWindow) & (kHist - 1)]) return CG_STALLED;
    }
    return CG_RUNNING;
}

// one block: totals of the init partials; threshold; convergence flag. mixed: the FP32 recurrence's
// start, from ||r0||^2 and ||b||^2 in scal[S_RES]: its target on the scaled residual is
// (0.9 tol ||b|| / ||r0||)^2, a little below the FP64 target, which the reliable update then usually
// confirms at once, or the end of the first segment (kSegment2); nothing is iterated if r0 meets the FP64
// target or is not finite.
__global__ void __launch_bounds__(kThreads) k_cg_start(const double *__restrict__ part, int m,
                                                       const double *__restrict__ rz_part, int m_rz, double *scal,
                                                       int32_t *flags, double tol2, const double *abs_thr2, int stall,
                                                       int mixed, HostResults *host) {
    __shared__ double sh[1][kThreads / 64];
    double rz = sum_partials(rz_part, m_rz, sh);
    double rr = sum_partials(part + kMaxBlocks, m, sh);
    double bb = mixed ? 0.0 : sum_partials(part + 2 * kMaxBlocks, m, sh);
    if (threadIdx.x == 0) {
        double thr2, rr0 = rr, target;
        int state;
        if (mixed) {
            rr0 = scal[S_RES];
            bb = scal[S_RES + 1];
            target = tol2 * bb;
            thr2 = fmax(0.81 * target / rr0, kSegment2);
            state = cg_state(rr0, 1.0, target, 0, 0, nullptr);
            if (!state) state = cg_state(rr, rz, thr2, stall, 0, nullptr);
        } else {
            target = thr2 = abs_thr2 ? *abs_thr2 : tol2 * bb;
            state = cg_state(rr, rz, thr2, stall, 0, nullptr);
        }
        scal[S_RZ] = rz;
        scal[S_RR] = rr;
        scal[S_BB] = bb;
        scal[S_THR2] = thr2;
        scal[S_HIST] = rr;
        flags[0] = state;
        flags[1] = 0;
        host->flags[0] = state;
        host->flags[1] = 0;
        host->rr = rr;
        host->thr2 = target;
        host->rr0 = rr0;
        host->bb = bb;
    }
}

// Iteration k (parity par = k & 1). For k > 0 first finish the previous update: r.z and
// r.r from its partials, convergence test, beta. Then, with w = A z (the only gathered
// vector), p = z + beta p and q = A p = w + beta q in place (own rows only), and the
// partials of p.q. Gathering one vector instead of z and p halves the scattered loads.
// VT, XT: the matrix values' and the vectors' types (FP64, or FP32 in the inner iterations of
// the mixed-precision solve; products, sums and dot products are FP64 either way).
// The sums that the previous kernel left, the stop flag and the row's own entries are loaded beside
// the first slice's product, which needs none of them: on small systems a launch is this chain of
// loads and little else.
template <typename VT, typename XT, int U>
__global__ void __launch_bounds__(kThreads) k_cg_spmv(int32_t n, int32_t ns, const SellCols S,
                                                      const VT *__restrict__ val,
                                                      const XT *__restrict__ z,
                                                      XT *__restrict__ p, XT *__restrict__ q,
                                                      const double *__restrict__ rz_part, int m_rz,
                                                      const double *__restrict__ rr_part, int m_rr,
                                                      double *__restrict__ part, double *scal, int32_t *flags,
                                                      int32_t k, int32_t par, int stall) {
    __shared__ double sh[2][kThreads / 64];
    __shared__ int stopped;
    const SellRange r = sell_range(ns);
    const int32_t lane = (int32_t)(threadIdx.x & 63);
    // one thread's reading decides for the block: block 0 may set the flag meanwhile
    if (threadIdx.x == 0) stopped = flags[0];
    double v[2] = {0.0, 0.0};  // r.z, r.r of the present iterate
    if (k > 0) {
        v[0] = load_partials(rz_part, m_rz);
        v[1] = load_partials(rr_part, m_rr);
    }
    const double thr2 = scal[S_THR2], rz_old = scal[S_RZ + (k > 0 ? par : 0)];
    int32_t row = r.begin * kSlice + lane;
    bool have = r.begin < r.end && row < n;
    double zi = 0.0, pi = 0.0, qi = 0.0, s = 0.0;
    if (have) {
        zi = (double)z[row];
        if (k > 0) {
            pi = (double)p[row];
            qi = (double)q[row];
        }
    }
    if (r.begin < r.end) s = sell_dot<U>(S, val, z, r.begin);
    block_sums<2>(v, sh);
    if (stopped) return;
    double beta = 0.0;
    if (k > 0) {
        // the ring slot read (k - 10) differs from the one written (k): no block reads what
        // block 0 writes in this launch
        const int state = cg_state(v[1], v[0], thr2, stall, k, scal + S_HIST);
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            scal[S_RZ + (par ^ 1)] = v[0];
            scal[S_RR] = v[1];
            scal[S_HIST + (k & (kHist - 1))] = v[1];
            flags[1] = k;
            if (state) flags[0] = state;
        }
        if (state) return;  // the same decision in every block (same sums, same order)
        beta = v[0] / rz_old;
    } else if (blockIdx.x == 0 && threadIdx.x == 0) {
        scal[S_RZ + 1] = rz_old;
    }
    double acc[1] = {0.0};
    for (int32_t sl = r.begin; sl < r.end; sl += r.step) {
        if (sl > r.begin) {
            row = sl * kSlice + lane;
            have = row < n;
            if (have) {
                zi = (double)z[row];
                if (k > 0) {
                    pi = (double)p[row];
                    qi = (double)q[row];
                }
            }
            s = sell_dot<U>(S, val, z, sl);
        }
        if (have) {
            const XT pn = (XT)(k > 0 ? zi + beta * pi : zi);
            const XT qn = (XT)(k > 0 ? s + beta * qi : s);
            p[row] = pn;
            q[row] = qn;
            acc[0] += (double)pn * (double)qn;
        }
    }
    write_partials<1>(acc, part);
}

// Jacobi: alpha = r.z / p.q; x += alpha p; r -= alpha q; z = D^-1 r; partials of r.z and r.r of the
// stored values. XT: the vectors' type, as in k_cg_spmv. The first entries are loaded beside the
// sums.
template <typename XT>
__global__ void __launch_bounds__(kThreads) k_cg_update(int32_t n, XT *__restrict__ x,
                                                        XT *__restrict__ r, XT *__restrict__ z,
                                                        const XT *__restrict__ p,
                                                        const XT *__restrict__ q,
                                                        const XT *__restrict__ dinv,
                                                        const double *__restrict__ qpart, double *__restrict__ part,
                                                        int m, const double *scal, const int32_t *flags, int32_t par) {
    __shared__ double sh[1][kThreads / 64];
    __shared__ int stopped;
    if (threadIdx.x == 0) stopped = flags[0];
    double pq[1] = {load_partials(qpart, m)};
    const double rz = scal[S_RZ + (par ^ 1)];
    int64_t i = ((int64_t)blockIdx.x * kThreads + threadIdx.x) * kVec<XT>;
    Vec<XT> xv, rv, pv, qv, dv;
    auto load = [&]() {
        if (i >= n) return;
        xv = load_vec(x, i, n);
        rv = load_vec(r, i, n);
        pv = load_vec(p, i, n);
        qv = load_vec(q, i, n);
        dv = load_vec(dinv, i, n);
    };
    load();
    block_sums<1>(pq, sh);
    if (stopped) return;
    const double alpha = rz / pq[0];
    double acc[2] = {0.0, 0.0};
    while (i < n) {
        Vec<XT> zv;
#pragma unroll
        for (int c = 0; c < kVec<XT>; ++c) {
            xv[c] = (XT)((double)xv[c] + alpha * (double)pv[c]);
            const XT ri = (XT)((double)rv[c] - alpha * (double)qv[c]);
            rv[c] = ri;
            if (i + c >= n) continue;
            const XT zi = (XT)((double)ri * (double)dv[c]);
            zv[c] = zi;
            acc[0] += (double)ri * (double)zi;
            acc[1] += (double)ri * (double)ri;
        }
        store_vec(x, i, n, xv);
        store_vec(r, i, n, rv);
        store_vec(z, i, n, zv);
        i += (int64_t)gridDim.x * kThreads * kVec<XT>;
        load();
    }
    write_partials<2>(acc, part);
}

// Learned preconditioner M = G^T G: the update and the first half of the application in one pass.
// alpha = r.z / p.q; x += alpha p; r -= alpha q; y = G r is kept by the same recurrence,
// y -= alpha G q, so the pass gathers q, which needs no alpha, and r.z of the new iterate is y.y.
// (y is formed anew from r wherever r is: at the start and at every reliable update. In between it drifts from
// G r by the vectors' rounding, with the trained factor of 8^3 to 20^3 to |y - G r| / |y| = 5e-4 to 8e-4 at the end of
// an FP32 segment of 1e-4, 2e-8 and 2e-4 at the end of an FP64 solve to 1e-8 and 1e-12; iterations and residuals are
// those of y formed anew each time, to 1e-15.) Against an
// update and a product of their own this saves a launch and its chain of loads per iteration, and
// the entries are in flight beside the sums: 64^3, FP32: 10.9 + 24.2 -> 29.8 us (24.9 with
// the present rounds of loads).
// Partials: y.y and r.r of the stored values.
template <typename XT, int U>
__global__ void __launch_bounds__(kThreads) k_cg_update_g(int32_t n, int32_t ns, const SellCols S,
                                                          const uint32_t *__restrict__ pk, XT *__restrict__ x,
                                                          XT *__restrict__ r, XT *__restrict__ y,
                                                          const XT *__restrict__ p, const XT *__restrict__ q,
                                                          const double *__restrict__ qpart, int m,
                                                          double *__restrict__ yy_part, double *__restrict__ rr_part,
                                                          const double *scal, const int32_t *flags, int32_t par) {
    __shared__ double sh[2][kThreads / 64];
    __shared__ int stopped;
    const SellRange sr = sell_range(ns);
    const int32_t lane = (int32_t)(threadIdx.x & 63);
    if (threadIdx.x == 0) stopped = flags[0];
    double pq[1] = {load_partials(qpart, m)};
    const double rz = scal[S_RZ + (par ^ 1)];
    double xi = 0.0, ri = 0.0, yi = 0.0, pi = 0.0, qi = 0.0, u = 0.0;
    auto load = [&](int32_t s) {
        const int32_t row = s * kSlice + lane;
        if (row < n) {
            xi = (double)x[row];
            ri = (double)r[row];
            yi = (double)y[row];
            pi = (double)p[row];
            qi = (double)q[row];
        }
        u = sell_dot<U>(S, pk, q, s);
    };
    if (sr.begin < sr.end) load(sr.begin);
    block_sums<1>(pq, sh);
    if (stopped) return;
    const double alpha = rz / pq[0];
    double acc[2] = {0.0, 0.0};
    for (int32_t s = sr.begin; s < sr.end; s += sr.step) {
        if (s > sr.begin) load(s);
        const int32_t row = s * kSlice + lane;
        if (row < n) {
            x[row] = (XT)(xi + alpha * pi);
            const XT rn = (XT)(ri - alpha * qi), yn = (XT)(yi - alpha * u);
            r[row] = rn;
            y[row] = yn;
            acc[0] += (double)yn * (double)yn;
            acc[1] += (double)rn * (double)rn;
        }
    }
    __syncthreads();  // every wave has read the first sums
    block_sums<2>(acc, sh);
    if (threadIdx.x == 0) {
        yy_part[blockIdx.x] = acc[0];
        rr_part[blockIdx.x] = acc[1];
    }
}

// ||b - A x||^2 and ||b||^2 (partials). STORE: also r = b - A x (the mixed-precision solve's
// reliable updates).
template <bool STORE, int U>
__global__ void __launch_bounds__(kThreads) k_residual(int32_t n, int32_t ns, const SellCols S,
                                                       const double *__restrict__ val, const double *__restrict__ x,
                                                       const double *__restrict__ b, double *__restrict__ r,
                                                       double *__restrict__ part) {
    double acc[2] = {0.0, 0.0};
    sell_rows<U>(n, ns, S, val, x, [&](int32_t row, double s) {
        const double bb = b[row];
        const double ri = bb - s;
        if (STORE) r[row] = ri;
        acc[0] += ri * ri;
        acc[1] += bb * bb;
    });
    write_partials<2>(acc, part);
}

// Mixed-precision solve. Start: the FP32 system A d = r0 / s, s = ||r0|| (a unit right-hand
// side), from d = 0: r32 = r0 / s, d = p = 0, with Jacobi z = D^-1 r32; partials of r.z (Jacobi),
// r.r. rr: ||r0||^2 on the device; s is kept in scal[S_SCALE] for the solve.
template <bool JAC>
__global__ void __launch_bounds__(kThreads) k_inner_init(int32_t n, const double *__restrict__ r, const double *rr,
                                                         double *scal, float *__restrict__ r32,
                                                         float *__restrict__ x32, float *__restrict__ z32,
                                                         float *__restrict__ p32, const double *__restrict__ dinv,
                                                         float *__restrict__ dinv32, double *__restrict__ part) {
    const double s = sqrt(*rr), inv = 1.0 / s;
    if (blockIdx.x == 0 && threadIdx.x == 0) scal[S_SCALE] = s;
    double acc[2] = {0.0, 0.0};
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kThreads) {
        const float ri = (float)(r[i] * inv);
        r32[i] = ri;
        x32[i] = 0.0f;
        p32[i] = 0.0f;
        if (JAC) {
            const float di = (float)dinv[i];
            dinv32[i] = di;
            const float zi = (float)((double)ri * (double)di);
            z32[i] = zi;
            acc[0] += (double)ri * (double)zi;
        }
        acc[1] += (double)ri * (double)ri;
    }
    write_partials<2>(acc, part);
}

// Reliable update, first half: x += s d in FP64 and d = 0. A batch that met non-finite values is not
// applied.
__global__ void k_refine(int32_t n, double *__restrict__ x, float *__restrict__ d, const double *scal,
                         const int32_t *flags) {
    if (flags[0] == CG_NONFINITE) return;
    const double s = scal[S_SCALE];
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        x[i] += s * (double)d[i];
        d[i] = 0.0f;
    }
}

// Reliable update, second half (after r = b - A x in FP64): the recurrence's residual replaced by
// r32 = r / s, with Jacobi z = D^-1 r32, and the partials of r.z (Jacobi) and r.r written where
// the update kernel writes them, so the iteration continues with the next product (its beta
// from the new r.z), the stop flag is cleared and thr2 is the next segment's target. The stall rule's history of r.r goes on: the
// replaced residual differs from the recurrence's by its FP32 drift only, far below the rule's
// 10 % over ten iterations while the solve converges, and a stalled solve stays stalled.
template <bool JAC>
__global__ void __launch_bounds__(kThreads) k_replace(int32_t n, const double *__restrict__ r, double *scal,
                                                      float *__restrict__ r32, float *__restrict__ z32,
                                                      const float *__restrict__ dinv32, double *__restrict__ part,
                                                      int32_t *flags, double thr2) {
    const double inv = 1.0 / scal[S_SCALE];
    double acc[2] = {0.0, 0.0};
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kThreads) {
        const float ri = (float)(r[i] * inv);
        r32[i] = ri;
        if (JAC) {
            const float zi = (float)((double)ri * (double)dinv32[i]);
            z32[i] = zi;
            acc[0] += (double)ri * (double)zi;
        }
        acc[1] += (double)ri * (double)ri;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        flags[0] = CG_RUNNING;
        scal[S_THR2] = thr2;
    }
    write_partials<2>(acc, part);
}

// A whole solve in one launch, for systems of at most 32 slices (2048 rows; 24 slices, 1536 rows, with
// the learned preconditioner): one block of sixteen waves, each with its slices' x, r, p, q in registers
// and the gathered vectors in LDS, so an iteration costs two block barriers (three with the learned
// preconditioner) instead of as many launches with their chains of cold loads, and the host waits
// once. FP64 throughout (also for mixed-precision solves: the matrix is cached, so FP32 saves nothing
// here). The same recurrences, tests and restarts as the launches.
// The limits are where one CU stops being faster than the chip. A step with 70-90 edge iterations, one
// launch against many: Jacobi 7^3 925 against 1018 us, 8^3 1495 against 1049; learned 7^3 812 against
// 696 (6^3: 562).
constexpr int kSmallWaves = 16, kSmallThreads = 64 * kSmallWaves;
constexpr int kRestarts = 2;  // from the iterate, when the recomputed residual misses the target

inline bool small_system(const DevSell &M, bool learned) { return M.ns <= (learned ? 24 : 32); }

template <int NV>
__device__ __forceinline__ void small_sums(double (&v)[NV], double (*sh)[kSmallWaves]) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        v[k] = wave_sum(v[k]);
        if (lane == 0) sh[k][wid] = v[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < kSmallWaves; ++w) t += sh[k][w];
        v[k] = t;
    }
}

// RES (Jacobi, one slice per wave, rows of at most 20 entries): the entries stay in registers from
// iteration to iteration (with the learned factor they do not fit: 182 registers spilled).
constexpr int kResA = 20;
template <bool LEARNED, int NS, bool RES>
__global__ void __launch_bounds__(kSmallThreads) k_solve_small(
    int32_t n, int32_t ns, const SellCols S, const double *__restrict__ val, const SellCols SG,
    const uint32_t *__restrict__ gpk, const SellCols ST, const uint32_t *__restrict__ tpk, double *__restrict__ xg,
    const double *__restrict__ b, const double *__restrict__ dinv, double tol2, const double *abs_thr2, int max_it,
    HostResults *host) {
    constexpr int UA = LEARNED ? 4 : 10, UG = 4;  // entries in flight per lane, within 128 registers
    static_assert(!RES || (NS == 1 && !LEARNED), "resident entries: Jacobi, one slice per wave");
    extern __shared__ double lds[];  // two vectors of ns slices
    __shared__ double sh_a[3][kSmallWaves], sh_b[1][kSmallWaves], sh_c[2][kSmallWaves];
    __shared__ double hist[kHist];
    const int lane = threadIdx.x & 63;
    const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    double *va = lds, *vb = lds + ns * kSlice;
    double x[NS], r[NS], p[NS], q[NS], d[NS], z[NS], y[NS];  // d: D^-1 (Jacobi); y = G r (learned)
#pragma unroll
    for (int j = 0; j < NS; ++j) {
        const int row = (wid + j * kSmallWaves) * kSlice + lane;
        x[j] = r[j] = p[j] = q[j] = d[j] = z[j] = y[j] = 0.0;
        if (row < n) {
            x[j] = xg[row];
            if (!LEARNED) d[j] = dinv[row];
        }
    }
    // resident entries: FP64 values with two 16-bit columns to a word
    double av[RES ? kResA : 1];
    uint32_t ac[RES ? kResA / 2 : 1];
    if (RES && wid < ns) {
        int32_t c[kResA];
        const int32_t o0 = wid * S.width;
        const int64_t e0 = (int64_t)o0 * kSlice + lane;
#pragma unroll
        for (int u = 0; u < kResA; ++u) {  // at most 1024 unknowns: 16-bit columns
            av[u] = u < S.width ? val[e0 + u * kSlice] : 0.0;
            c[u] = u < S.width ? S.base[o0 + u] + (int32_t)S.c16[e0 + u * kSlice] : 0;
        }
#pragma unroll
        for (int u = 0; u < kResA / 2; ++u) ac[u] = (uint32_t)c[2 * u] | (uint32_t)c[2 * u + 1] << 16;
    }
    auto prod_a = [&](const double *v, int sl) {
        if constexpr (RES) {
            double acc = 0.0;
#pragma unroll
            for (int u = 0; u < kResA; ++u)
                if (u < S.width) acc = fma(av[u], v[u & 1 ? ac[u / 2] >> 16 : ac[u / 2] & 0xffffu], acc);
            return acc;
        } else {
            return sell_dot<UA>(S, val, v, sl);
        }
    };
    // each(f): f(j, slice, row) for this wave's slices; f's row may lie past n (vectors hold 0 there)
    auto each = [&](auto &&f) {
#pragma unroll
        for (int j = 0; j < NS; ++j) {
            const int sl = wid + j * kSmallWaves;
            if (sl < ns) f(j, sl, sl * kSlice + lane);
        }
    };
    double thr2 = 0.0, rr0 = 0.0, bb0 = 0.0, res2 = 0.0, bb2 = 0.0;
    int it = 0, state = CG_RUNNING;
    for (int restart = 0;; ++restart) {
        each([&](int j, int, int row) { va[row] = x[j]; });
        __syncthreads();
        double sa[3] = {0.0, 0.0, 0.0};  // r.z, r.r, b.b
        each([&](int j, int sl, int row) {
            const double ax = prod_a(va, sl), bi = row < n ? b[row] : 0.0;
            r[j] = row < n ? bi - ax : 0.0;
            p[j] = q[j] = 0.0;
            z[j] = r[j] * d[j];
            sa[0] += r[j] * z[j];
            sa[1] += r[j] * r[j];
            sa[2] += bi * bi;
        });
        if (LEARNED) {
            each([&](int j, int, int row) { vb[row] = r[j]; });
            __syncthreads();
            each([&](int j, int sl, int row) {
                y[j] = row < n ? sell_dot<UG>(SG, gpk, vb, sl) : 0.0;
                sa[0] += y[j] * y[j];
            });
            __syncthreads();
            each([&](int j, int, int row) { vb[row] = y[j]; });
            __syncthreads();
            each([&](int j, int sl, int row) { z[j] = row < n ? sell_dot<UG>(ST, tpk, vb, sl) : 0.0; });
        }
        small_sums<3>(sa, sh_a);
        double rz = sa[0], rr = sa[1];
        if (restart == 0) {
            thr2 = abs_thr2 ? *abs_thr2 : tol2 * sa[2];
            rr0 = rr;
            bb0 = sa[2];
        }
        state = cg_state(rr, rz, thr2, LEARNED ? 1 : 0, 0, nullptr);
        if (threadIdx.x == 0) hist[0] = rr;
        each([&](int j, int, int row) { va[row] = z[j]; });
        __syncthreads();
        double beta = 0.0;
        for (int k = 1; !state && it < max_it; ++k) {
            double sb[1] = {0.0};
            each([&](int j, int sl, int row) {
                const double w = prod_a(va, sl);
                p[j] = z[j] + beta * p[j];
                q[j] = row < n ? w + beta * q[j] : 0.0;
                sb[0] += p[j] * q[j];
                if (LEARNED) vb[row] = q[j];
            });
            small_sums<1>(sb, sh_b);  // z is no longer read, q is there for all
            const double alpha = rz / sb[0];
            double sc[2] = {0.0, 0.0};  // r.z, r.r
            each([&](int j, int sl, int row) {
                x[j] += alpha * p[j];
                r[j] -= alpha * q[j];
                if (LEARNED) {
                    const double u = sell_dot<UG>(SG, gpk, vb, sl);
                    y[j] = row < n ? y[j] - alpha * u : 0.0;
                    va[row] = y[j];
                    sc[0] += y[j] * y[j];
                } else {
                    z[j] = r[j] * d[j];
                    va[row] = z[j];
                    sc[0] += r[j] * z[j];
                }
                sc[1] += r[j] * r[j];
            });
            small_sums<2>(sc, sh_c);
            if (LEARNED) {  // z = G^T y into the other vector
                each([&](int j, int sl, int row) {
                    z[j] = row < n ? sell_dot<UG>(ST, tpk, va, sl) : 0.0;
                    vb[row] = z[j];
                });
                __syncthreads();
                double *t = va;
                va = vb;
                vb = t;
            }
            ++it;
            beta = sc[0] / rz;
            rz = sc[0];
            rr = sc[1];
            state = cg_state(rr, rz, thr2, LEARNED ? 1 : 0, k, hist);
            if (threadIdx.x == 0) hist[k & (kHist - 1)] = rr;  // read ten iterations on
        }
        // true residual, recomputed
        __syncthreads();
        each([&](int j, int, int row) { va[row] = x[j]; });
        __syncthreads();
        double st[3] = {0.0, 0.0, 0.0};
        each([&](int, int sl, int row) {
            const double ax = prod_a(va, sl);
            const double bi = row < n ? b[row] : 0.0, ri = row < n ? bi - ax : 0.0;
            st[0] += ri * ri;
            st[1] += bi * bi;
        });
        small_sums<3>(st, sh_a);
        res2 = st[0];
        bb2 = st[1];
        __syncthreads();
        if (state != CG_CONVERGED || res2 <= thr2 || it >= max_it || restart == kRestarts) break;
    }
    each([&](int j, int, int row) {
        if (row < n) xg[row] = x[j];
    });
    if (threadIdx.x == 0) {
        host->flags[0] = state;
        host->flags[1] = it;
        host->thr2 = thr2;
        host->rr0 = rr0;
        host->bb = bb0;
        host->res[0] = res2;
        host->res[1] = bb2;
    }
}

template <typename S, typename D>
__global__ void k_convert(int64_t n, const S *__restrict__ in, D *__restrict__ out) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        out[i] = (D)in[i];
}

// one block, after a batch: finish the last update's convergence test; the verdict goes to the host
__global__ void __launch_bounds__(kThreads) k_cg_check(const double *__restrict__ upart, int m, double *scal,
                                                       int32_t *flags, int32_t k, HostResults *host) {
    __shared__ double sh[1][kThreads / 64];
    double rr = sum_partials(upart + kMaxBlocks, m, sh);
    if (threadIdx.x == 0) {
        int state = flags[0], it = flags[1];
        if (!state) {
            scal[S_RR] = rr;
            flags[1] = it = k;
            // convergence or a non-finite residual; the stall rule waits for the next product
            // kernel, which also has r.z
            state = cg_state(rr, 1.0, scal[S_THR2], 0, k, nullptr);
            if (state) flags[0] = state;
        }
        host->flags[0] = state;
        host->flags[1] = it;
        host->rr = scal[S_RR];
    }
}

__global__ void k_diag_inv(int32_t n, const SellCols S, const double *__restrict__ val, double *__restrict__ dinv) {
    const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    const int32_t s = __builtin_amdgcn_readfirstlane(i / kSlice), l = i % kSlice;
    if (i >= n) return;
    double d = 0.0;
    int32_t o0, w;
    sell_extent(S, s, o0, w);
    if (w > 0) {
        const SellScalars base = sell_bases(S, o0);
        const bool wide = base[0] < 0;
        const int64_t e0 = (int64_t)o0 * kSlice + l;
        auto take = [&](int32_t k) {
            const double v = val[e0 + (int64_t)k * kSlice];
            if (v != 0.0) d = v;  // padding holds zeros
        };
        if (wide) {
            for (int32_t k = 0; k < w; ++k)
                if (S.c32[e0 + (int64_t)k * kSlice] == i) take(k);
        } else {
            const uint16_t *cp = S.c16 + e0;
            int32_t k = 0;
            for (; k + 4 <= w; k += 4) {  // four columns' loads in flight
                uint32_t c[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) c[u] = cp[(int64_t)(k + u) * kSlice];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (base[k + u] + (int32_t)c[u] == i) take(k + u);
            }
            for (; k < w; ++k)
                if (base[k] + (int32_t)cp[(int64_t)k * kSlice] == i) take(k);
        }
    }
    dinv[i] = d != 0.0 ? 1.0 / d : 0.0;
}

// A = [*eps] + tau S on the CSR pattern
__global__ void k_axpy_vals(int64_t n, const double *__restrict__ a, const double *__restrict__ s, double tau,
                            double *__restrict__ out) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = a[i] + tau * s[i];
}

// CSR values on slices (src: CSR entry, -1: padding)
__global__ void k_to_slices(int64_t len, const int32_t *__restrict__ src, const double *__restrict__ a,
                            double *__restrict__ out) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < len) out[i] = src[i] >= 0 ? a[src[i]] : 0.0;
}

// A = [*eps] + tau S and the right-hand-side matrix [*eps] - tau S on the slices, from both there: a
// change of dt streams four arrays of A's size. (From the CSR values through src instead, every lane
// another row, and the CSR copy of A filled beside them: 395 + 121 us at 64^3.)
__global__ void k_axpy_slices(int64_t len, const double *__restrict__ a, const double *__restrict__ s, double tau,
                              double *__restrict__ out, double *__restrict__ out_m) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= len) return;
    const double ae = a[i], se = s[i];
    out[i] = ae + tau * se;
    out_m[i] = ae - tau * se;
}

__global__ void k_renumber(int64_t n, const int32_t *__restrict__ idx, const double *__restrict__ in,
                           double *__restrict__ out) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = in[idx[i]];
}

// Edge right-hand side in two passes over the edge unknowns:
//   rhs_i = sum_j ([*eps] - tau S)_ij e_j - u_q g[int_edge_i]          (k_edge_rhs_e)
//   rhs_i += dt u_b sum_f (C^T [*mu^-1])_if b_f                          (k_edge_rhs_b)
// The second takes its rows in interior-edge order (pos: their place in rhs): face fluxes are kept
// by face number, a dozen per node, and the edges of one node share most of them. Rows in device
// numbering gather 96 bytes apart (both passes, us: 48^3 75.9 against 74.4, 64^3 195 against 187), but they are
// taken (pos null) where interior-edge order has no 16-bit columns, as of 74^3 (96^3: 601 against 630),
// and where the device numbering follows a curve in space (48^3 numbered at random: 87.5 against 129).
template <int U>
__global__ void __launch_bounds__(kThreads) k_edge_rhs_e(int32_t n, int32_t ns, const SellCols S,
                                                         const double *__restrict__ mval,
                                                         const double *__restrict__ e,
                                                         const int64_t *__restrict__ g,
                                                         const int32_t *__restrict__ int_edges, double u_q,
                                                         double *__restrict__ rhs) {
    const SellRange r = sell_range(ns);
    for (int32_t s = r.begin; s < r.end; s += r.step) {
        const int32_t row = s * kSlice + (int32_t)(threadIdx.x & 63);
        const double a = sell_dot<U>(S, mval, e, s);
        if (row < n) rhs[row] = a - u_q * (double)g[int_edges[row]];
    }
}

template <int U>
__global__ void __launch_bounds__(kThreads) k_edge_rhs_b(int32_t n, int32_t ns, const SellCols S,
                                                         const double *__restrict__ cval,
                                                         const int64_t *__restrict__ b, double dtub,
                                                         const int32_t *__restrict__ pos, double *__restrict__ rhs) {
    const SellRange r = sell_range(ns);
    for (int32_t s = r.begin; s < r.end; s += r.step) {
        const int32_t row = s * kSlice + (int32_t)(threadIdx.x & 63);
        const double t = sell_dot<U>(S, cval, b, s);
        if (row < n) {
            double *d = rhs + (pos ? pos[row] : row);
            *d += dtub * t;
        }
    }
}

// Gauss residual rg = rho - G^T [*eps] e on interior nodes, rho = u_q (Q_bg - Q);
// threshold thr2 = (tol_n (||rho|| + || |G^T [*eps]| |e| ||))^2: the residual is measured
// against the size of the terms that cancel in G^T [*eps] e (normwise backward error), so
// the tolerance stays above the FP64 rounding floor when the charge is small against E.
// Rows are few and long (about 50 entries: every edge of the tets around the node), so the eight
// waves of a block share each slice, a part of its entries each: one wave per slice would leave
// most of the chip idle behind seven dependent rounds of loads (25^3: 5.2 us a launch; eight lanes per row of a
// CSR matrix took 6.8).
__global__ void __launch_bounds__(kThreads) k_gauss_rhs(int32_t n, int32_t ns, const SellCols S,
                                                        const double *__restrict__ val,
                                                        const double *__restrict__ e,
                                                        const int64_t *__restrict__ Qbg,
                                                        const int64_t *__restrict__ Q,
                                                        const int32_t *__restrict__ int_nodes, double u_q,
                                                        const double *__restrict__ dbnd,
                                                        double *__restrict__ rg, double *__restrict__ rho_out,
                                                        double *__restrict__ x0, double *__restrict__ part) {
    __shared__ double part_s[kSellWaves][kSlice], part_a[kSellWaves][kSlice];
    const int32_t lane = (int32_t)(threadIdx.x & 63);
    const int32_t wid = __builtin_amdgcn_readfirstlane((int32_t)(threadIdx.x >> 6));
    // one contiguous span of slices per XCD, as sell_range
    const int32_t per_x = (int32_t)gridDim.x / 8, span = (ns + 7) / 8, xcd = (int32_t)blockIdx.x & 7;
    const int32_t end = (xcd + 1) * span < ns ? (xcd + 1) * span : ns;
    double acc[3] = {0.0, 0.0, 0.0};
    for (int32_t sl = xcd * span + ((int32_t)blockIdx.x >> 3); sl < end; sl += per_x) {
        double s = 0.0, sa = 0.0;
        sell_each<kU64>(S, val, e, sl, [&](double v, double x) {
            const double t = v * x;
            s += t;
            sa += fabs(t);
        }, wid, kSellWaves);
        part_s[wid][lane] = s;
        part_a[wid][lane] = sa;
        __syncthreads();
        const int32_t row = sl * kSlice + lane;
        if (wid == 0 && row < n) {
            s = sa = 0.0;
#pragma unroll
            for (int w = 0; w < kSellWaves; ++w) {
                s += part_s[w][lane];
                sa += part_a[w][lane];
            }
            int32_t gn = int_nodes[row];
            // charge, plus the normal flux a plane wave brought in through a natural boundary
            double rho = u_q * (double)(Qbg[gn] - Q[gn]) + (dbnd ? dbnd[gn] : 0.0);
            double res = rho - s;
            rg[row] = res;
            x0[row] = 0.0;  // the node solve starts from zero
            if (rho_out) rho_out[row] = rho;
            acc[0] += rho * rho;
            acc[1] += sa * sa;
            acc[2] += res * res;
        }
        __syncthreads();
    }
    write_partials<3>(acc, part);
}

// one block: out[0] = (tol_n scale)^2, out[1] = scale, out[2] = ||r||^2, out[3] = ||rho||, also to the host
__global__ void __launch_bounds__(kThreads) k_gauss_finish(const double *__restrict__ part, int m, double *out,
                                                           double tol_n, HostResults *host) {
    __shared__ double sh[1][kThreads / 64];
    double a = sum_partials(part, m, sh);
    double b = sum_partials(part + kMaxBlocks, m, sh);
    double c = sum_partials(part + 2 * kMaxBlocks, m, sh);
    if (threadIdx.x == 0) {
        double scale = sqrt(a) + sqrt(b);
        const double v[4] = {tol_n * tol_n * scale * scale, scale, c, sqrt(a)};
        for (int q = 0; q < 4; ++q) out[q] = host->gauss[q] = v[q];
    }
}

// Item of this thread in kernels that gather from another numbering than the one they run over: the
// blocks of an XCD (which gets every eighth) take one contiguous span, since the edges at 256 nodes are
// seven runs of 256 by kind in the device numbering and interleaved by edge number, so neighbouring blocks
// gather the same lines and one L2 serves them. Grids (xcd_grid) are multiples of 8, or blocks share items.
inline unsigned xcd_grid(int64_t n) { return (unsigned)(((n + 255) / 256 + 7) / 8 * 8); }
__device__ __forceinline__ int32_t xcd_item() {
    const int32_t block = ((int32_t)blockIdx.x & 7) * ((int32_t)gridDim.x >> 3) + ((int32_t)blockIdx.x >> 3);
    return block * 256 + (int32_t)threadIdx.x;
}

// e_i += delta[head] - delta[tail] (wall nodes carry 0); keep: the uncorrected e (or null). ends: the edge's
// tail and head among the unknown nodes, -1: wall (through the edge's number and its nodes' numbers, three
// dependent gathers, 19.3 us at 64^3 and 60 at 96^3; now 12.8 and 39).
__global__ void k_gauss_apply(int32_t n, const int2 *__restrict__ ends, const double *__restrict__ delta,
                              double *__restrict__ e, double *__restrict__ keep) {
    const int32_t i = xcd_item();
    if (i >= n) return;
    const int2 v = ends[i];
    const double d = (v.y >= 0 ? delta[v.y] : 0.0) - (v.x >= 0 ? delta[v.x] : 0.0);
    const double ei = e[i];
    if (keep) keep[i] = ei;
    e[i] = ei + d;
}

// u = round((dt/2)(e_new + e_old)/u_b) per interior edge; e (global) <- e_new. edge_of: the edge of item i,
// pos_of: its position (null: i). In edge order it gathers e and writes u in order (over the device numbering,
// with scattered writes, 21.3 us at 64^3 and 61 at 96^3; so 14.5 and 39.5); where the device numbering follows
// a curve in space the gathers are the worse (48^3 numbered at random, with k_faraday_b: 33.4 against 26.5),
// and the items are the positions.
__global__ void k_faraday_u(int32_t n, const int32_t *__restrict__ edge_of, const int32_t *__restrict__ pos_of,
                            const double *__restrict__ enew, const double *__restrict__ eold, double half_dt_over_ub,
                            int64_t *__restrict__ u, double *__restrict__ eglob) {
    const int32_t i = xcd_item();
    if (i >= n) return;
    const int32_t ge = edge_of[i], p = pos_of ? pos_of[i] : i;
    const double en = enew[p];
    u[ge] = (int64_t)llrint(half_dt_over_ub * (en + eold[p]));
    eglob[ge] = en;
}

// b_f -= u_bc - u_ac + u_ab
__global__ void k_faraday_b(int64_t nf, const int32_t *__restrict__ fe, const int64_t *__restrict__ u,
                            int64_t *__restrict__ b) {
    int64_t f = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (f >= nf) return;
    b[f] -= u[fe[3 * f + 2]] - u[fe[3 * f + 1]] + u[fe[3 * f]];
}

__global__ void __launch_bounds__(kThreads) k_sum2(const double *__restrict__ part, int m, double *out,
                                                   HostResults *host) {
    __shared__ double sh[1][kThreads / 64];
    double a = sum_partials(part, m, sh);
    double b = sum_partials(part + kMaxBlocks, m, sh);
    if (threadIdx.x == 0) {
        out[0] = host->res[0] = a;
        out[1] = host->res[1] = b;
    }
}

// Right-hand side of the wave-equation update (eq. wave_cont, Newmark beta = 1/4, gamma = 1/2)
// on the interior edges:
//   rhs = 2 ([*eps] - tau S) e^n - ([*eps] + tau S) e^{n-1} - u_q (g^{n+1/2} - g^{n-1/2}).
template <int U>
__global__ void __launch_bounds__(kThreads) k_wave_rhs(int32_t n, int32_t ns, const SellCols S,
                                                       const double *__restrict__ arhs,
                                                       const double *__restrict__ aval,
                                                       const double *__restrict__ e,
                                                       const double *__restrict__ e_prev,
                                                       const int64_t *__restrict__ g,
                                                       const int64_t *__restrict__ g_prev,
                                                       const int32_t *__restrict__ int_edges, double u_q,
                                                       double *__restrict__ rhs) {
    const SellRange r = sell_range(ns);
    for (int32_t s = r.begin; s < r.end; s += r.step) {
        const int32_t row = s * kSlice + (int32_t)(threadIdx.x & 63);
        const double a = sell_dot<U>(S, arhs, e, s);
        const double ap = sell_dot<U>(S, aval, e_prev, s);
        if (row < n) {
            const int32_t ge = int_edges[row];
            rhs[row] = (2.0 * a - u_q * (double)(g[ge] - g_prev[ge])) - ap;
        }
    }
}

// Plane wave through the natural boundary. s'(tau) of the modulated Gaussian s(u) =
// exp(-(u - t0)^2 / (2 sig^2)) cos(2 pi f0 (u - t0)).
__device__ __forceinline__ double pw_ds(double tau, double f0, double sig, double t0) {
    const double u = tau - t0, om = 2.0 * M_PI * f0;
    const double env = exp(-u * u / (2.0 * sig * sig));
    return env * (-(u / (sig * sig)) * cos(om * u) - om * sin(om * u));
}

// s'(t - x/c) at the step's three times for each distinct x of the rule points.
__global__ void k_pw_table(int32_t nu, const double *__restrict__ xs, double f0, double sig, double t0, double c0,
                           double t_prev, double t_n, double t_next, double *__restrict__ tab) {
    const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nu) return;
    const double ret = xs[i] / c0;
    tab[3 * i] = pw_ds(t_prev - ret, f0, sig, t0);
    tab[3 * i + 1] = pw_ds(t_n - ret, f0, sig, t0);
    tab[3 * i + 2] = pw_ds(t_next - ret, f0, sig, t0);
}

// Boundary term h_i(t) = sum over the edge's rule points of coef * (E0/eta) s'(t - x/c), at the
// step's times (s' from the table); adds the update's share to the right-hand side
// (trapezoidal: dt/2 (h^n + h^{n+1}); wave equation: dt/2 (h^{n+1} - h^{n-1})) and keeps
// dt/2 (h^n + h^{n+1}) for the Gauss-law target.
__global__ void k_plane_wave(int32_t nb, const int32_t *__restrict__ ptr, const int32_t *__restrict__ edge,
                             const double *__restrict__ coef, const int32_t *__restrict__ xi,
                             const double *__restrict__ tab, double amp, double half_dt, int wave,
                             double *__restrict__ rhs, double *__restrict__ hsum) {
    const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nb) return;
    double hp = 0.0, hn = 0.0, hx = 0.0;
    for (int32_t k = ptr[i]; k < ptr[i + 1]; ++k) {
        const double w = coef[k];
        const double *s = tab + 3 * xi[k];
        hn += w * s[1];
        hx += w * s[2];
        if (wave) hp += w * s[0];
    }
    const double hs = half_dt * amp * (hn + hx);
    hsum[i] = hs;
    rhs[edge[i]] += wave ? half_dt * amp * (hx - hp) : hs;
}

// dbnd += G^T hsum on the boundary nodes (edge a -> b: +1 at b, -1 at a), one thread per node in
// a fixed order.
__global__ void k_boundary_flux(int32_t nn, const int32_t *__restrict__ nptr, const int32_t *__restrict__ nlist,
                                const int32_t *__restrict__ node, const double *__restrict__ hsum,
                                double *__restrict__ dbnd) {
    const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nn) return;
    double s = 0.0;
    for (int32_t k = nptr[i]; k < nptr[i + 1]; ++k) {
        const int32_t v = nlist[k];
        s += (v & 1) ? -hsum[v >> 1] : hsum[v >> 1];
    }
    dbnd[node[i]] += s;
}

}  // namespace

int qh_cg_alloc(qh_ctx *c, CgWork &w, int32_t n) {
    w.n = n;
    int rc;
    if ((rc = qh_alloc(c, &w.x, n)) || (rc = qh_alloc(c, &w.r, n)) || (rc = qh_alloc(c, &w.z, n)) ||
        (rc = qh_alloc(c, &w.q, n)) || (rc = qh_alloc(c, &w.p0, n)) || (rc = qh_alloc(c, &w.p1, n)) ||
        (rc = qh_alloc(c, &w.dinv, n)) || (rc = qh_alloc(c, &w.b, n)) ||
        (rc = qh_alloc(c, &w.partial, 9 * kMaxBlocks)) || (rc = qh_alloc(c, &w.scal, S_NSCAL)) ||
        (rc = qh_alloc(c, &w.counter, 4)) || (rc = qh_alloc(c, &w.flags, 4)))
        return rc;
    QH_HIP(c, hipMemsetAsync(w.counter, 0, 4 * sizeof(unsigned int), c->stream));
    QH_HIP(c, hipMemsetAsync(w.x, 0, n * sizeof(double), c->stream));
    QH_HIP(c, hipMemsetAsync(w.scal, 0, S_NSCAL * sizeof(double), c->stream));
    return QH_OK;
}

hipError_t launch_diag_inv(qh_ctx *c, const DevSell &M, double *dinv) {
    if (M.n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_diag_inv, dim3((M.n + 255) / 256), dim3(256), 0, c->stream, M.n, M.cols(), M.val, dinv);
    return hipGetLastError();
}

hipError_t launch_renumber(qh_ctx *c, int64_t n, const int32_t *idx, const double *in, double *out) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_renumber, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, c->stream, n, idx, in, out);
    return hipGetLastError();
}

template <typename T>
static void launch_update_g(qh_ctx *c, T *x, T *r, T *y, const T *p, const T *q, const double *qpart, int m,
                            double *yy_part, double *rr_part, const double *scal, const int32_t *flags, int32_t par) {
    const LearnedPrec &L = c->lp;
    hipLaunchKernelGGL((L.gs.width > 0 ? k_cg_update_g<T, kUPrecAll> : k_cg_update_g<T, kUPrec>),
                       dim3(sell_grid(L.gs.ns)), dim3(kThreads), 0, c->stream, L.n, L.gs.ns, L.gs.cols(),
                       (const uint32_t *)L.gpk, x, r, y, p, q, qpart, m, yy_part, rr_part, scal, flags, par);
}

// The one-launch solve of a small system, from w.x; fills `out`.
static int solve_small(qh_ctx *c, const DevSell &M, CgWork &w, double tol, int max_it, SolveResult &out,
                       const double *abs_thr2_dev, int timer, bool learned) {
    const LearnedPrec &L = c->lp;
    if (learned) QH_HIP(c, launch_prec_pack(c));
    const size_t bytes = sizeof(double) * 2 * kSlice * (size_t)M.ns;
    int t0 = qh_tbeg(c);
    auto run = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(1), dim3(kSmallThreads), bytes, c->stream, w.n, M.ns, M.cols(),
                           (const double *)M.val, L.gs.cols(), (const uint32_t *)L.gpk, L.ts.cols(),
                           (const uint32_t *)L.tpk, w.x, (const double *)w.b, (const double *)w.dinv, tol * tol,
                           abs_thr2_dev, max_it, c->host);
    };
    const int per = (M.ns + kSmallWaves - 1) / kSmallWaves;
    const bool res = per == 1 && M.width > 0 && M.width <= kResA;
    if (learned) {
        if (per == 1) run(k_solve_small<true, 1, false>);
        else run(k_solve_small<true, 2, false>);
    } else {
        if (res) run(k_solve_small<false, 1, true>);
        else if (per == 1) run(k_solve_small<false, 1, false>);
        else run(k_solve_small<false, 2, false>);
    }
    qh_tend(c, t0, timer);
    QH_HIP(c, hipGetLastError());
    QH_HIP(c, hipStreamSynchronize(c->stream));
    volatile const HostResults *H = c->host;
    const double res2 = H->res[0], bb2 = H->res[1], thr2 = H->thr2;
    out.flag = H->flags[0];
    out.iters = H->flags[1];
    out.res = bb2 > 0 ? sqrt(res2 / bb2) : 0.0;
    out.true_ok = res2 == res2 && res2 <= thr2;
    out.converged = out.flag == CG_CONVERGED && out.true_ok;
    return QH_OK;
}

// Iterations until r.r has fallen by `factor` more, from the reduction so far (rr0 -> rr in k
// iterations); 0 if there was none.
static int iterations_for(double rr0, double rr, int k, double factor) {
    const double drop = rr > 0 && rr0 > 0 && k > 0 ? std::log(rr / rr0) / k : 0.0;
    if (!(drop < 0) || !(factor > 0) || factor >= 1) return 0;
    return (int)std::min(1e6, std::ceil(std::log(factor) / drop));
}

// The same from the mean rate so far (rr0 in k iterations) or the last batch's (rr_last in `batch`),
// whichever promises it sooner, and at most twice the iterations done: a residual often falls little at
// first (a smooth or a local right-hand side) and a mean over that asks for many times what is needed. On
// the node system of 44^3 to 1e-12, a constant right-hand side, 136 iterations: 1449 launched by the mean
// alone (10.3 ms), 136 so (1.6 ms); white noise, 198 iterations: 204 and 202 (2.2 ms each).
static int iterations_ahead(double rr0, int k, double rr_last, int batch, double rr, double factor) {
    const int mean = iterations_for(rr0, rr, k, factor), last = iterations_for(rr_last, rr, batch, factor);
    const int soon = mean > 0 && last > 0 ? std::min(mean, last) : std::max(mean, last);
    return (int)std::min<int64_t>(soon, 2 * (int64_t)k);
}

int qh_cg_solve(qh_ctx *c, const DevSell &M, CgWork &w, double tol, int max_it, int check_every,
                SolveResult &out, const double *abs_thr2_dev, bool node_system, bool learned) {
    const int k_spmv = node_system ? QK_NODE_SPMV : QK_CG_SPMV;
    const int k_upd = node_system ? QK_NODE_UPDATE : QK_CG_UPDATE;
    out = SolveResult();
    if (w.n == 0) {
        out.converged = true;
        out.flag = CG_CONVERGED;
        return QH_OK;
    }
    if (small_system(M, learned)) {
        int rc = solve_small(c, M, w, tol, max_it, out, abs_thr2_dev, k_spmv, learned);
        if (rc) return rc;
        if (out.converged) w.last_iters[learned ? 1 : 0] = out.iters;
        return QH_OK;
    }
    // partials: [0, 4K) init / update (slot 0 r.z with Jacobi, 1 r.r, 2 b.b), [4K, 5K) products,
    // [5K, 6K) r.z of the learned preconditioner, [6K, 8K) the true residual's, taken ahead
    double *upart = w.partial, *qpart = w.partial + 4 * kMaxBlocks, *ppart = w.partial + 5 * kMaxBlocks;
    const unsigned ge = grid_elems<double>(w.n), gt = sell_grid(M.ns);
    const unsigned gp = learned ? qh_prec_grid(c) : 0;
    const int stall = learned ? 1 : 0;
    volatile const HostResults *H = c->host;
    if (check_every <= 0) check_every = 8;
    // iterations after convergence return at once on the device; sizing the first batch from
    // the previous solve avoids most of them and most host reads of the flag
    int first = w.last_iters[learned ? 1 : 0];
    if (first > 0) ++first;  // one idle launch when the count repeats, no second batch when it grows by one
    int it = 0;
    // true residual, recomputed with a fresh FP64 product
    auto residual = [&]() -> int {
        int tr = qh_tbeg(c);
        hipLaunchKernelGGL((M.width > 0 ? k_residual<false, kUAll> : k_residual<false, kU64>), dim3(gt), dim3(kThreads), 0, c->stream, w.n, M.ns, M.cols(), M.val, w.x,
                           w.b, (double *)nullptr, upart);
        hipLaunchKernelGGL(k_sum2, dim3(1), dim3(kThreads), 0, c->stream, upart, (int)gt, w.scal + S_RES, c->host);
        qh_tend(c, tr, QK_TRUE_RES);
        QH_HIP(c, hipGetLastError());
        return QH_OK;
    };
    // Recurrence residuals drift from the true one; a solve whose recurrence converged but whose
    // recomputed residual misses the target restarts from its iterate (at most kRestarts times)
    for (int restart = 0;; ++restart) {
        int t0 = qh_tbeg(c);
        hipLaunchKernelGGL((M.width > 0 ? k_cg_init<kUAll> : k_cg_init<kU64>), dim3(gt), dim3(kThreads), 0, c->stream, w.n, M.ns, M.cols(), M.val,
                           w.x, w.b, w.dinv, w.r, w.z, w.p0, upart);
        if (learned) QH_HIP(c, launch_prec_apply(c, w.r, w.z, ppart));
        hipLaunchKernelGGL(k_cg_start, dim3(1), dim3(kThreads), 0, c->stream, upart, (int)gt,
                           learned ? (const double *)ppart : (const double *)upart, learned ? (int)gp : (int)gt,
                           w.scal, w.flags, tol * tol, abs_thr2_dev, stall, 0, c->host);
        qh_tend(c, t0, QK_CG_INIT);
        QH_HIP(c, hipGetLastError());
        // the start's verdict is read on the host only when the last solve needed no iteration
        // (or there was none); otherwise the first batch is launched at once, its launches return
        // at once if the start already stopped the iteration, and the true residual follows it
        // before the host looks
        const bool ahead = first > 0 && restart == 0;
        int stopped = 0, done = 0;  // this run's flag and iterations
        bool have_res = false, at_start = false;
        double rr_start = 0.0, rr_last = 0.0;  // r.r at the start and at the last read
        int m_up = (int)gt;
        if (!ahead) {
            QH_HIP(c, hipStreamSynchronize(c->stream));
            stopped = H->flags[0];
            at_start = stopped == CG_CONVERGED;
            rr_start = rr_last = H->rr;
        }
        const int it0 = it;  // the device counts this run's iterations from 0
        int batch = ahead ? first : check_every;
        while (it < max_it && !stopped) {
            batch = std::min(batch, max_it - it);
            for (int k = it - it0; k < it - it0 + batch; ++k) {
                int par = k & 1;
                int ta = qh_tbeg(c);
                hipLaunchKernelGGL((M.width > 0 ? k_cg_spmv<double, double, kUAll> : k_cg_spmv<double, double, kU64>),
                                   dim3(gt), dim3(kThreads), 0, c->stream, w.n, M.ns, M.cols(), M.val, w.z, w.p0, w.q,
                                   learned ? (const double *)ppart : (const double *)upart, learned ? (int)gp : m_up,
                                   upart + kMaxBlocks, m_up, qpart, w.scal, w.flags, k, par, stall);
                qh_tend(c, ta, k_spmv);
                int tb = qh_tbeg(c);
                if (learned) {
                    launch_update_g<double>(c, w.x, w.r, c->lp.y, w.p0, w.q, qpart, (int)gt, ppart, upart + kMaxBlocks,
                                            w.scal, w.flags, par);
                    qh_tend(c, tb, k_upd);
                    m_up = (int)gp;
                    int tp = qh_tbeg(c);
                    QH_HIP(c, launch_prec_gt(c, w.z, w.flags));
                    qh_tend(c, tp, QK_PREC);
                } else {
                    hipLaunchKernelGGL(k_cg_update<double>, dim3(ge), dim3(kThreads), 0, c->stream, w.n, w.x, w.r, w.z,
                                       w.p0, w.q, w.dinv, qpart, upart, (int)gt, w.scal, w.flags, par);
                    qh_tend(c, tb, k_upd);
                    m_up = (int)ge;
                }
            }
            const bool last_guess = ahead && it == it0;
            it += batch;
            hipLaunchKernelGGL(k_cg_check, dim3(1), dim3(kThreads), 0, c->stream, upart, m_up, w.scal, w.flags,
                               it - it0, c->host);
            QH_HIP(c, hipGetLastError());
            // the residual's partials take the update's place, which a continued run still needs
            have_res = last_guess;
            if (last_guess) {
                double *keep = upart;
                upart = w.partial + 6 * kMaxBlocks;
                int rc = residual();
                upart = keep;
                if (rc) return rc;
            }
            QH_HIP(c, hipStreamSynchronize(c->stream));
            stopped = H->flags[0];
            done = H->flags[1];
            // the next read after most of the iterations that the present rate leaves to do
            if (last_guess) rr_start = rr_last = H->rr0;
            const double rr = H->rr;
            const int next = 3 * (int64_t)iterations_ahead(rr_start, it - it0, rr_last, batch, rr, H->thr2 / rr) / 4;
            rr_last = rr;
            batch = std::max(check_every, next);
        }
        it = it0 + done;
        out.iters = it;
        out.flag = stopped;
        if (at_start) {
            // r = b - A x was formed anew at the start: its norm is the true residual
            const double rr = H->rr, bb = H->bb;
            out.res = bb > 0 ? sqrt(rr / bb) : 0.0;
            out.true_ok = true;
        } else {
            if (!have_res || !stopped) {
                int rc = residual();
                if (rc) return rc;
                QH_HIP(c, hipStreamSynchronize(c->stream));
            }
            const double res2 = H->res[0], bb2 = H->res[1], thr2 = H->thr2;
            out.res = bb2 > 0 ? sqrt(res2 / bb2) : 0.0;
            out.true_ok = res2 == res2 && res2 <= thr2;
        }
        out.converged = out.flag == CG_CONVERGED && out.true_ok;
        if (out.converged || out.flag != CG_CONVERGED || it >= max_it || restart == kRestarts) break;
    }
    if (out.converged) w.last_iters[learned ? 1 : 0] = out.iters;
    return QH_OK;
}

// FP32 buffers of a CgWork for n unknowns (kept when large enough)
int qh_cg_alloc32(qh_ctx *c, CgWork &w, int32_t n) {
    if (w.n32 >= n) return QH_OK;
    int rc;
    if ((rc = qh_alloc(c, &w.x32, n)) || (rc = qh_alloc(c, &w.r32, n)) || (rc = qh_alloc(c, &w.z32, n)) ||
        (rc = qh_alloc(c, &w.p32, n)) || (rc = qh_alloc(c, &w.q32, n)) || (rc = qh_alloc(c, &w.dinv32, n)))
        return rc;
    w.n32 = n;
    return QH_OK;
}

// Mixed-precision solve: PCG in FP32 (the FP32 copy of A's values, FP32 vectors, FP64 products
// and dot products, the same preconditioner) on A d = r0 / s from the FP64 residual r0 = b - A x0,
// s = ||r0||, with reliable updates: at the end of each batch of iterations x += s d in FP64,
// r = b - A x is recomputed in FP64 (the convergence test: ||r|| <= tol ||b||, the FP64 solve's
// stopping rule) and, unless it is met, replaces the recurrence's residual, which then continues
// without a restart (its Krylov space and convergence rate are kept). A segment between updates
// may reduce the residual by about 1e-4 at most (the FP32 correction d holds the FP64 solution's
// change only to FP32 accuracy): its length comes from the last solve's rate of convergence, and
// the last batch ends at the last solve's iteration count (from the second segment on, taking in
// a remainder of at most an eighth of a segment), where the FP64 residual usually meets the
// target already (the recurrence aims a little lower), so a step of the benchmark takes two
// reliable updates. Without a history, a first batch of check_every iterations, then what this
// solve's own rate gives for the segment or for the rest, whichever is less (iterations_ahead). These are
// estimates: the device ends a segment that has reduced the residual by 3e-5 (kSegment2), which takes less
// than the batch where the residual falls faster than before. The host reads once per update: the verdict
// of the batch and the recomputed residual. A batch that meets non-finite values is not applied
// (flag 3); one stopped by the stall rule is applied and the solve returns (flag 2).
int qh_cg_solve_mixed(qh_ctx *c, DevSell &M, CgWork &w, double tol, int max_it, int check_every,
                      SolveResult &out, bool learned) {
    out = SolveResult();
    const int32_t n = w.n;
    if (n == 0) {
        out.converged = out.true_ok = true;
        out.flag = CG_CONVERGED;
        return QH_OK;
    }
    int rc;
    if (small_system(M, learned)) {
        rc = solve_small(c, M, w, tol, max_it, out, nullptr, QK_CG_SPMV, learned);
        // one FP64 residual after the start, the final one, unless the start met the target
        out.refinements = out.flag == CG_NONFINITE || (out.converged && out.iters == 0) ? 0 : 1;
        return rc;
    }
    if ((rc = qh_cg_alloc32(c, w, n))) return rc;
    // FP32 copy of the matrix values once per time step size
    if (!M.val32 || M.val32_tau != c->tau_assembled) {
        if (!M.val32 && (rc = qh_alloc(c, &M.val32, (size_t)M.len))) return rc;
        const unsigned gc = (unsigned)std::min<int64_t>((M.len + 255) / 256, 8192);
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_convert<double, float>), dim3(gc), dim3(256), 0, c->stream, M.len, M.val,
                           M.val32);
        M.val32_tau = c->tau_assembled;
    }
    QH_HIP(c, hipGetLastError());
    double *upart = w.partial, *qpart = w.partial + 4 * kMaxBlocks, *ppart = w.partial + 5 * kMaxBlocks;
    const unsigned ge = grid_elems<float>(n), gt = sell_grid(M.ns);
    const unsigned gp = learned ? qh_prec_grid(c) : 0;
    const int stall = learned ? 1 : 0;
    volatile const HostResults *H = c->host;
    if (check_every <= 0) check_every = 8;
    // r = b - A x in FP64 with ||r||^2 and ||b||^2
    auto fp64_residual = [&]() -> int {
        int tr = qh_tbeg(c);
        hipLaunchKernelGGL((M.width > 0 ? k_residual<true, kUAll> : k_residual<true, kU64>), dim3(gt), dim3(kThreads), 0, c->stream, n, M.ns, M.cols(), M.val, w.x, w.b,
                           w.r, upart);
        hipLaunchKernelGGL(k_sum2, dim3(1), dim3(kThreads), 0, c->stream, upart, (int)gt, w.scal + S_RES, c->host);
        qh_tend(c, tr, QK_TRUE_RES);
        QH_HIP(c, hipGetLastError());
        return QH_OK;
    };
    if ((rc = fp64_residual())) return rc;
    int t0 = qh_tbeg(c);
    hipLaunchKernelGGL((learned ? k_inner_init<false> : k_inner_init<true>), dim3(ge), dim3(kThreads), 0, c->stream, n, w.r,
                       w.scal + S_RES, w.scal, w.r32, w.x32, w.z32, w.p32, w.dinv, w.dinv32, upart);
    if (learned) QH_HIP(c, launch_prec_apply32(c, w.r32, w.z32, ppart));
    hipLaunchKernelGGL(k_cg_start, dim3(1), dim3(kThreads), 0, c->stream, upart, (int)ge,
                       learned ? (const double *)ppart : (const double *)upart, learned ? (int)gp : (int)ge,
                       w.scal, w.flags, tol * tol, (const double *)nullptr, stall, 1, c->host);
    qh_tend(c, t0, QK_CG_INIT);
    QH_HIP(c, hipGetLastError());
    const int prev = w.last_mixed[learned ? 1 : 0];     // iterations of the last converged solve
    const int seg = w.last_segment[learned ? 1 : 0];    // its iterations per 1e-4 of reduction
    int m_up = (int)ge;  // blocks that left the last partials of r.r
    int k = 0, flag = CG_RUNNING, batch_next = check_every;
    double rr0 = 0.0, rr = 0.0, rr_last = 0.0;
    for (int update = 0;; ++update) {
        // a batch: to the next segment end, at most to the last solve's iteration count (from
        // the second segment on, a last remainder of at most an eighth of a segment joins the
        // one before it), then as this solve's rate says
        int target = 0;
        if (prev > 0 && seg > 0) {
            target = std::min((update + 1) * seg, prev);
            if (update > 0 && prev - target <= seg / 8) target = prev;
        }
        const int batch = std::max(0, std::min(target > k ? target - k : batch_next, max_it - k));
        for (int kk = k; kk < k + batch; ++kk) {
            const int par = kk & 1;
            int ta = qh_tbeg(c);
            hipLaunchKernelGGL((M.width > 0 ? k_cg_spmv<float, float, kUAll> : k_cg_spmv<float, float, kU32>), dim3(gt),
                               dim3(kThreads), 0, c->stream, n, M.ns, M.cols(), (const float *)M.val32,
                               (const float *)w.z32, w.p32, w.q32, learned ? (const double *)ppart : (const double *)upart,
                               learned ? (int)gp : (int)ge, upart + kMaxBlocks, m_up, qpart, w.scal, w.flags, kk, par,
                               stall);
            qh_tend(c, ta, QK_CG_SPMV);
            int tb = qh_tbeg(c);
            if (learned) {
                launch_update_g<float>(c, w.x32, w.r32, c->lp.y32, w.p32, w.q32, qpart, (int)gt, ppart, upart + kMaxBlocks,
                                       w.scal, w.flags, par);
                qh_tend(c, tb, QK_CG_UPDATE);
                m_up = (int)gp;
                int tp = qh_tbeg(c);
                QH_HIP(c, launch_prec_gt32(c, w.z32, w.flags));
                qh_tend(c, tp, QK_PREC);
            } else {
                hipLaunchKernelGGL(k_cg_update<float>, dim3(ge), dim3(kThreads), 0, c->stream, n, w.x32, w.r32, w.z32,
                                   (const float *)w.p32, (const float *)w.q32, (const float *)w.dinv32, qpart, upart,
                                   (int)gt, w.scal, w.flags, par);
                qh_tend(c, tb, QK_CG_UPDATE);
            }
        }
        if (batch > 0)
            hipLaunchKernelGGL(k_cg_check, dim3(1), dim3(kThreads), 0, c->stream, upart, m_up, w.scal, w.flags, k + batch,
                               c->host);
        // reliable update: x += s d, r = b - A x in FP64
        int tf = qh_tbeg(c);
        hipLaunchKernelGGL(k_refine, dim3(ge), dim3(kThreads), 0, c->stream, n, w.x, w.x32, (const double *)w.scal,
                           (const int32_t *)w.flags);
        qh_tend(c, tf, QK_TRUE_RES);
        QH_HIP(c, hipGetLastError());
        if ((rc = fp64_residual())) return rc;
        QH_HIP(c, hipStreamSynchronize(c->stream));
        const int stopped = H->flags[0];
        const double bb = H->bb, thr2 = H->thr2;
        rr0 = H->rr0;
        // the start decided: r0 is not finite (an overflowing ||b||^2 makes its target infinite too),
        // or meets its target
        const bool finite0 = rr0 <= 1.7976931348623157e308;
        if (update == 0 && (!finite0 || rr0 <= thr2)) {
            out.res = bb > 0 ? sqrt(rr0 / bb) : 0.0;
            flag = finite0 ? CG_CONVERGED : CG_NONFINITE;
            break;
        }
        const int k_last = k;
        k = stopped ? H->flags[1] : k + batch;
        if (stopped == CG_NONFINITE) {
            flag = CG_NONFINITE;  // the batch is not applied: x keeps the last reliable update
            if (update == 0) out.res = bb > 0 ? sqrt(rr0 / bb) : 0.0;
            break;
        }
        out.refinements = update + 1;
        rr_last = update == 0 ? rr0 : rr;
        rr = H->res[0];
        out.res = bb > 0 ? sqrt(rr / bb) : 0.0;
        if (rr == rr && rr <= thr2) {
            flag = CG_CONVERGED;
            break;
        }
        if (!(rr == rr) || rr > 1.7976931348623157e308) {
            flag = CG_NONFINITE;
            break;
        }
        if (stopped == CG_STALLED) {
            flag = CG_STALLED;
            break;
        }
        if (k >= max_it) break;
        batch_next = std::max(check_every, iterations_ahead(rr0, k, rr_last, k - k_last, rr, std::max(1e-8, 0.81 * thr2 / rr)));
        // the recurrence continues from the FP64 residual
        int tq = qh_tbeg(c);
        hipLaunchKernelGGL((learned ? k_replace<false> : k_replace<true>), dim3(ge), dim3(kThreads), 0, c->stream, n,
                           (const double *)w.r, w.scal, w.r32, w.z32, (const float *)w.dinv32, upart, w.flags,
                           std::max(0.81 * thr2, kSegment2 * rr) / rr0);
        m_up = (int)ge;
        if (learned) QH_HIP(c, launch_prec_apply32(c, w.r32, w.z32, ppart));
        qh_tend(c, tq, QK_CG_INIT);
        QH_HIP(c, hipGetLastError());
    }
    out.iters = k;
    out.flag = flag;
    out.converged = out.true_ok = flag == CG_CONVERGED;
    if (out.converged) {
        w.last_mixed[learned ? 1 : 0] = k;
        // iterations per 1e-4 of residual reduction (1e-8 of r.r), at least check_every
        const int per = iterations_for(rr0, rr, k, 1e-8);
        w.last_segment[learned ? 1 : 0] = per > 0 ? std::max(check_every, per) : 0;
    }
    return QH_OK;
}

hipError_t launch_A_to_slices(qh_ctx *c) {
    const int64_t len = c->As.len;
    if (len == 0) return hipSuccess;
    const dim3 grid((unsigned)((len + 255) / 256));
    hipLaunchKernelGGL(k_to_slices, grid, dim3(256), 0, c->stream, len, c->As.src, c->A.val2, c->As_eps);
    hipLaunchKernelGGL(k_to_slices, grid, dim3(256), 0, c->stream, len, c->As.src, c->A_S, c->As_S);
    return hipGetLastError();
}

hipError_t launch_assemble_A(qh_ctx *c, double tau) {
    const int64_t len = c->As.len;
    if (len == 0) return hipSuccess;
    hipLaunchKernelGGL(k_axpy_slices, dim3((unsigned)((len + 255) / 256)), dim3(256), 0, c->stream, len, c->As_eps,
                       c->As_S, tau, c->As.val, c->A_rhs);
    return hipGetLastError();
}

hipError_t launch_assemble_A_csr(qh_ctx *c, double tau) {
    const int64_t nnz = c->A.nnz;
    if (nnz == 0) return hipSuccess;
    hipLaunchKernelGGL(k_axpy_vals, dim3((unsigned)((nnz + 255) / 256)), dim3(256), 0, c->stream, nnz, c->A.val2,
                       c->A_S, tau, c->A.val);
    return hipGetLastError();
}

hipError_t launch_edge_rhs(qh_ctx *c) {
    const DevSell &A = c->As, &C = c->CMb;
    hipLaunchKernelGGL((A.width > 0 ? k_edge_rhs_e<kUAll> : k_edge_rhs_e<kU64>), dim3(sell_grid(A.ns)), dim3(kThreads), 0,
                       c->stream, A.n, A.ns, A.cols(), c->A_rhs, c->cge.x, c->g, c->int_edges, c->phys.u_q, c->cge.b);
    hipLaunchKernelGGL((C.width > 0 ? k_edge_rhs_b<kUAll> : k_edge_rhs_b<kU64>), dim3(sell_grid(C.ns)), dim3(kThreads), 0,
                       c->stream, C.n, C.ns, C.cols(), C.val, c->b, c->phys.dt * c->phys.u_b, c->CMb_pos, c->cge.b);
    return hipGetLastError();
}

hipError_t launch_wave_rhs(qh_ctx *c) {
    const DevSell &A = c->As;
    hipLaunchKernelGGL((A.width > 0 ? k_wave_rhs<kUAll> : k_wave_rhs<kU64>), dim3(sell_grid(A.ns)), dim3(kThreads), 0, c->stream, A.n, A.ns, A.cols(), c->A_rhs,
                       A.val, c->cge.x, c->e_prev, c->g, c->g_prev, c->int_edges, c->phys.u_q, c->cge.b);
    return hipGetLastError();
}

hipError_t launch_plane_wave(qh_ctx *c, bool wave) {
    const double dt = c->phys.dt, tn = (double)c->step_index * dt;
    hipLaunchKernelGGL(k_pw_table, dim3((c->pw_nu + 255) / 256), dim3(256), 0, c->stream, c->pw_nu, c->pw_xs, c->pw_f0,
                       c->pw_sig, c->pw_t0, c->pw_c, tn - dt, tn, tn + dt, c->pw_tab);
    hipLaunchKernelGGL(k_plane_wave, dim3((c->pw_nb + 255) / 256), dim3(256), 0, c->stream, c->pw_nb, c->pw_ptr,
                       c->pw_edge, c->pw_coef, c->pw_xi, c->pw_tab, c->pw_amp, 0.5 * dt, wave ? 1 : 0, c->cge.b,
                       c->pw_hsum);
    hipLaunchKernelGGL(k_boundary_flux, dim3((c->pw_nn + 255) / 256), dim3(256), 0, c->stream, c->pw_nn, c->pw_nptr,
                       c->pw_nlist, c->pw_node, c->pw_hsum, c->dbnd);
    return hipGetLastError();
}

static unsigned gauss_grid(int32_t ns) {
    const int32_t b = (ns + 7) / 8 * 8;
    return (unsigned)(b < 8 ? 8 : b < kMaxBlocks ? b : kMaxBlocks);
}

hipError_t launch_gauss_rhs(qh_ctx *c, double *out3, double tol_n) {
    const DevSell &M = c->GtM;
    const unsigned gr = gauss_grid(M.ns);
    hipLaunchKernelGGL(k_gauss_rhs, dim3(gr), dim3(kThreads), 0, c->stream, M.n, M.ns, M.cols(), M.val, c->cge.x,
                       c->Q_bg, c->Q, c->int_nodes, c->phys.u_q, (const double *)c->dbnd, c->cgn.b, c->rho,
                       c->cgn.x, c->cgn.partial);
    hipLaunchKernelGGL(k_gauss_finish, dim3(1), dim3(kThreads), 0, c->stream, c->cgn.partial, (int)gr, out3, tol_n,
                       c->host);
    return hipGetLastError();
}

// Quasi-Helmholtz split: cgn.b = -G^T [*eps] e (the Gauss-law right-hand side with no charge
// and no boundary flux), with the node solve's threshold in out3 as for the correction.
hipError_t launch_div_e(qh_ctx *c, double *out3, double tol_n) {
    const DevSell &M = c->GtM;
    const unsigned gr = gauss_grid(M.ns);
    hipLaunchKernelGGL(k_gauss_rhs, dim3(gr), dim3(kThreads), 0, c->stream, M.n, M.ns, M.cols(), M.val, c->cge.x,
                       (const int64_t *)c->Q, (const int64_t *)c->Q, c->int_nodes, 0.0, (const double *)nullptr,
                       c->cgn.b, (double *)nullptr, c->cgn.x, c->cgn.partial);
    hipLaunchKernelGGL(k_gauss_finish, dim3(1), dim3(kThreads), 0, c->stream, c->cgn.partial, (int)gr, out3, tol_n,
                       c->host);
    return hipGetLastError();
}

// e_int += G delta (interior edge values; delta on the unknown nodes)
hipError_t launch_grad_add(qh_ctx *c, const double *delta, double *e_int) {
    int32_t n = c->A.n;
    hipLaunchKernelGGL(k_gauss_apply, dim3(xcd_grid(n)), dim3(256), 0, c->stream, n, c->edge_ends, delta, e_int,
                       (double *)nullptr);
    return hipGetLastError();
}

hipError_t launch_gauss_apply(qh_ctx *c, bool delta) {
    int32_t n = c->A.n;
    if (n == 0) return hipSuccess;
    if (!delta)
        return hipMemcpyAsync(c->e_star, c->cge.x, sizeof(double) * n, hipMemcpyDeviceToDevice, c->stream);
    hipLaunchKernelGGL(k_gauss_apply, dim3(xcd_grid(n)), dim3(256), 0, c->stream, n, c->edge_ends, c->cgn.x,
                       c->cge.x, c->e_star);
    return hipGetLastError();
}

hipError_t launch_faraday(qh_ctx *c) {
    int32_t n = c->A.n;
    const bool by_pos = c->hm.in_space;
    hipLaunchKernelGGL(k_faraday_u, dim3(xcd_grid(n)), dim3(256), 0, c->stream, n, by_pos ? c->int_edges : c->edge_of,
                       by_pos ? (const int32_t *)nullptr : c->pos_of, c->cge.x, c->e_old, 0.5 * c->phys.dt / c->phys.u_b, c->u_int, c->e);
    int64_t nf = c->hm.Nf;
    hipLaunchKernelGGL(k_faraday_b, dim3((unsigned)((nf + 255) / 256)), dim3(256), 0, c->stream, nf, c->face_edges,
                       c->u_int, c->b);
    return hipGetLastError();
}
