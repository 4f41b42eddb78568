// Multi-right-hand-side kernels: the same V-cycle and Krylov steps applied to
// W = 4, 8 or 16 (at most kW) independent right-hand sides at once.
//
// Vectors are n x W, row-major, in hierarchical order: with W = 16 the values
// of a row are one 128-byte (FP64) or 64-byte (FP32) line, so every gathered
// neighbour is one line and every matrix entry is read once per 16 columns.
// The width is a launch argument (lw = log2 W): a batch of few right-hand sides
// moves few columns.  A row is handled by a group of W/CPL lanes, each lane owning
// CPL adjacent columns.  Per column the arithmetic is a fixed sequence (entries in CSR
// order, members in order), independent of the unroll depth U, of CPL and
// of the other columns: a column's result does not depend on what else is
// in the batch.  Reductions are per-workgroup partials combined in a fixed
// order by single-workgroup finalize kernels, one recurrence per column.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "kernels.hpp"

namespace pamg {

constexpr int kW = 16;   // right-hand sides per batch

struct BatchCol {
    double beta, alpha, rho, rho_old, delta_old, rnorm, bnorm, tol;
    int iter, done, status, first, maxit, fixed_iters, active, pad;
};

struct BatchState {
    BatchCol col[kW];
    int all_done, krylov, pad0, pad1;
};

// ---------------------------------------------------------------- helpers

template <typename T, int C>
struct Vec {
    T v[C];
};

template <typename T, int C>
__device__ __forceinline__ Vec<T, C> vload(const T* p) {
    Vec<T, C> r;
    if constexpr (C == 1) {
        r.v[0] = p[0];
    } else if constexpr (C == 2) {
        using V2 = typename std::conditional<std::is_same<T, double>::value, double2, float2>::type;
        const V2 t = *reinterpret_cast<const V2*>(p);
        r.v[0] = t.x;
        r.v[1] = t.y;
    } else if constexpr (std::is_same<T, float>::value) {
        static_assert(C == 4, "1, 2 or 4 columns per lane");
        const float4 t = *reinterpret_cast<const float4*>(p);
        r.v[0] = t.x; r.v[1] = t.y; r.v[2] = t.z; r.v[3] = t.w;
    } else {
        static_assert(C == 4, "1, 2 or 4 columns per lane");
        const double2 t0 = *reinterpret_cast<const double2*>(p);
        const double2 t1 = *reinterpret_cast<const double2*>(p + 2);
        r.v[0] = t0.x; r.v[1] = t0.y; r.v[2] = t1.x; r.v[3] = t1.y;
    }
    return r;
}

template <typename T, int C>
__device__ __forceinline__ void vstore(T* p, const Vec<T, C>& a) {
    if constexpr (C == 1) {
        p[0] = a.v[0];
    } else if constexpr (C == 2) {
        using V2 = typename std::conditional<std::is_same<T, double>::value, double2, float2>::type;
        V2 t;
        t.x = a.v[0];
        t.y = a.v[1];
        *reinterpret_cast<V2*>(p) = t;
    } else if constexpr (std::is_same<T, float>::value) {
        float4 t;
        t.x = a.v[0]; t.y = a.v[1]; t.z = a.v[2]; t.w = a.v[3];
        *reinterpret_cast<float4*>(p) = t;
    } else {
        double2 t0, t1;
        t0.x = a.v[0]; t0.y = a.v[1];
        t1.x = a.v[2]; t1.y = a.v[3];
        *reinterpret_cast<double2*>(p) = t0;
        *reinterpret_cast<double2*>(p + 2) = t1;
    }
}

// The row group of this thread and its first column: W / CPL lanes a group.
template <int CPL>
struct LaneGroup {
    static constexpr int kLog = CPL == 4 ? 2 : CPL == 2 ? 1 : 0;
    int g, col0, gpb;
    __device__ __forceinline__ explicit LaneGroup(int lw)
        : g((int)threadIdx.x >> (lw - kLog)), col0(((int)threadIdx.x & ((1 << (lw - kLog)) - 1)) * CPL),
          gpb((int)blockDim.x >> (lw - kLog)) {}
};

// Units (rows or coarse rows) handled by one row group: first, +stride, < end;
// units are split into contiguous per-XCD chunks as in tile_walk.
__device__ __forceinline__ TileWalk unit_walk(int nunits, int gpb, int g) {
    const int G = gridDim.x, b = blockIdx.x;
    TileWalk w;
    if (G < kXcds) {
        w.first = b * gpb + g;
        w.stride = G * gpb;
        w.end = nunits;
        return w;
    }
    const int x = b % kXcds, j = b / kXcds;
    const int gx = G / kXcds + (x < G % kXcds ? 1 : 0);
    w.first = (int)((long long)nunits * x / kXcds) + j * gpb + g;
    w.end = (int)((long long)nunits * (x + 1) / kXcds);
    w.stride = gx * gpb;
    return w;
}

inline int unit_grid(long long nunits, int gpb) {
    long long g = (nunits + gpb - 1) / gpb;
    if (g > kMaxGrid) g = kMaxGrid;
    return g < 1 ? 1 : (int)g;
}

// s[q] += the next U entries of a row, in entry order, of a_k x[c_k][col0 + q],
// all their loads in flight together; TAIL: only the first rem of them (the
// others repeat the last one's loads and are left out of the sum).
template <int U, bool TAIL, int ST, int CPL, typename T, typename XT, bool APART = false>
__device__ __forceinline__ void entries_accumulate(int o, int rem, const int* __restrict__ ci,
                                                   const T* __restrict__ av, const XT* __restrict__ x, int lw,
                                                   int col0, T (&s)[CPL]) {
    int c[U];
    T a[U];
#pragma unroll
    for (int u = 0; u < U; ++u) c[u] = ci[o + (TAIL ? min(u, rem - 1) : u) * ST];
#pragma unroll
    for (int u = 0; u < U; ++u) a[u] = av[o + (TAIL ? min(u, rem - 1) : u) * ST];
    Vec<XT, CPL> xv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) xv[u] = vload<XT, CPL>(x + ((size_t)c[u] << lw) + col0);
    if constexpr (APART) __builtin_amdgcn_sched_barrier(0);   // every gather is issued before the first sum
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int q = 0; q < CPL; ++q) {
            const T t = s[q] + a[u] * (T)xv[u].v[q];
            s[q] = !TAIL || u < rem ? t : s[q];
        }
}

// The last rem < U entries of a row, one trip to memory for the columns and one
// for the values: the smallest power of two of loads that holds them.  (One
// entry after the other before: rows of 7 at unroll 8 were a chain of 7 trips;
// the Krylov pass over 227 thousand such rows, FP64, 8 columns, 28.7 us, now
// 20.6, level 0's up-sweep 20.0 and 15.4.)
template <int U, int ST, int CPL, typename T, typename XT>
__device__ __forceinline__ void tail_accumulate(int o, int rem, const int* __restrict__ ci,
                                                const T* __restrict__ av, const XT* __restrict__ x, int lw, int col0,
                                                T (&s)[CPL]) {
    if constexpr (U == 1) {
        if (rem > 0) entries_accumulate<1, false, ST, CPL, T, XT>(o, 1, ci, av, x, lw, col0, s);
    } else {
        if (rem > U / 2)
            entries_accumulate<U, true, ST, CPL, T, XT>(o, rem, ci, av, x, lw, col0, s);
        else
            tail_accumulate<U / 2, ST, CPL, T, XT>(o, rem, ci, av, x, lw, col0, s);
    }
}

// s[q] += sum over row i's entries, in entry order, of a_k x[c_k][col0 + q], U
// entries at a time.  (The lanes of a group load the same index and value;
// plain loads keep the line in L2 for the group's next entries: non-temporal
// loads made the 16-column engine 1.6x slower.)
// APART keeps the compiler from moving sums in between the gathers to save
// registers.
template <int U, int CPL, typename T, typename XT, bool APART = false, class ROWS>
__device__ __forceinline__ void row_accumulate(const ROWS& R, int i, const int* __restrict__ ci,
                                               const T* __restrict__ av, const XT* __restrict__ x, int lw, int col0,
                                               T (&s)[CPL]) {
    constexpr int ST = ROWS::kStride;
    const int len = R.len(i);
    int o = R.start(i), k = 0;
    for (; k + U <= len; k += U, o += U * ST)
        entries_accumulate<U, false, ST, CPL, T, XT, APART>(o, U, ci, av, x, lw, col0, s);
    tail_accumulate<U, ST, CPL, T, XT>(o, len - k, ci, av, x, lw, col0, s);
}

// Two rows at once (i and the next one): s0 and s1 as row_accumulate computes
// them, H entries of each in flight together.  For long sliced rows: entry k of
// two neighbouring rows shares a line of columns and of values, and the rows of
// an aggregate share most of the lines they gather, which then are still in L1
// (128^3 trilinear, 16 columns, level 0: FP32 403 us one row after the other,
// 326 in pairs, FP64 639 and 596; level 1: 222 and 191, 387 and 345).  Short
// rows share little (1.33 million rows of 7, FP64: 140 and 151), and with a
// row's entries contiguous a pair only widens the spread of the loads (550
// thousand rows, FP32: 100 and 120; 227 thousand rows of 7, FP64: 21 and 27).
constexpr int kPairRow = 16;                            // mean entries per row
template <int H, int CPL, typename T, typename XT, class ROWS>
__device__ __forceinline__ void row_pair_accumulate(const ROWS& R, int i, const int* __restrict__ ci,
                                                    const T* __restrict__ av, const XT* __restrict__ x, int lw,
                                                    int col0, T (&s0)[CPL], T (&s1)[CPL]) {
    constexpr int st = ROWS::kStride;
    const int len0 = R.len(i), len1 = R.len(i + 1);
    const int o0 = R.start(i), o1 = R.start(i + 1);
    const int most = max(len0, len1);
    for (int k = 0; k < most; k += H) {
        int c0[H], c1[H];
        T a0[H], a1[H];
#pragma unroll
        for (int u = 0; u < H; ++u) {
            const int k0 = min(k + u, len0 - 1), k1 = min(k + u, len1 - 1);
            c0[u] = ci[o0 + k0 * st];
            c1[u] = ci[o1 + k1 * st];
            a0[u] = av[o0 + k0 * st];
            a1[u] = av[o1 + k1 * st];
        }
        Vec<XT, CPL> x0[H], x1[H];
#pragma unroll
        for (int u = 0; u < H; ++u) {
            x0[u] = vload<XT, CPL>(x + ((size_t)c0[u] << lw) + col0);
            x1[u] = vload<XT, CPL>(x + ((size_t)c1[u] << lw) + col0);
        }
#pragma unroll
        for (int u = 0; u < H; ++u)
#pragma unroll
            for (int q = 0; q < CPL; ++q) {
                const T t0 = s0[q] + a0[u] * (T)x0[u].v[q], t1 = s1[q] + a1[u] * (T)x1[u].v[q];
                s0[q] = k + u < len0 ? t0 : s0[q];
                s1[q] = k + u < len1 ? t1 : s1[q];
            }
    }
}

// ---------------------------------------------------------------- V-cycle

// Down-sweep: rc[I] = sum_{m in G_I} p_m (r_m - (A D^-1 r)_m), per column.
// PAIR: two members at a time (row_pair_accumulate).
template <int U, int CPL, bool PAIR, typename T, typename RT, class ROWS>
static __global__ __launch_bounds__(kBlock) void kb_down(int nc, int lw, ROWS rows, const int* __restrict__ ci,
                                                  const T* __restrict__ vd, const RT* __restrict__ r,
                                                  const T* __restrict__ p, const int* __restrict__ aggptr,
                                                  T* __restrict__ rc, const int* __restrict__ done) {
    if (*done) return;
    const LaneGroup<CPL> lg(lw);
    const int col0 = lg.col0;
    const TileWalk w = unit_walk(nc, lg.gpb, lg.g);
    for (int I = w.first; I < w.end; I += w.stride) {
        const int m0 = aggptr[I], m1 = aggptr[I + 1];
        T acc[CPL];
#pragma unroll
        for (int q = 0; q < CPL; ++q) acc[q] = 0;
        int m = m0;
        if constexpr (PAIR && U > 1)
            for (; m + 1 < m1; m += 2) {
                T s0[CPL], s1[CPL];
#pragma unroll
                for (int q = 0; q < CPL; ++q) s0[q] = s1[q] = 0;
                const Vec<RT, CPL> rm0 = vload<RT, CPL>(r + ((size_t)m << lw) + col0);
                const Vec<RT, CPL> rm1 = vload<RT, CPL>(r + ((size_t)(m + 1) << lw) + col0);
                const T p0 = p[m], p1 = p[m + 1];
                row_pair_accumulate<U / 2, CPL, T, RT>(rows, m, ci, vd, r, lw, col0, s0, s1);
#pragma unroll
                for (int q = 0; q < CPL; ++q) acc[q] += p0 * ((T)rm0.v[q] - s0[q]);
#pragma unroll
                for (int q = 0; q < CPL; ++q) acc[q] += p1 * ((T)rm1.v[q] - s1[q]);
            }
        for (; m < m1; ++m) {
            T s[CPL];
#pragma unroll
            for (int q = 0; q < CPL; ++q) s[q] = 0;
            row_accumulate<U, CPL, T, RT>(rows, m, ci, vd, r, lw, col0, s);
            const Vec<RT, CPL> rm = vload<RT, CPL>(r + ((size_t)m << lw) + col0);
            const T pm = p[m];
#pragma unroll
            for (int q = 0; q < CPL; ++q) acc[q] += pm * ((T)rm.v[q] - s[q]);
        }
        Vec<T, CPL> o;
#pragma unroll
        for (int q = 0; q < CPL; ++q) o.v[q] = acc[q];
        vstore<T, CPL>(rc + ((size_t)I << lw) + col0, o);
    }
}

// Up-sweep at level l > 0: z = zp + D^-1 (r - A zp), prolongated into level
// l-1: zp_f[m] = dinv_f[m] r_f[m] + p_f[m] z for the members m of row i.
template <int U, int CPL, typename T, typename RT, typename RTF, class ROWS>
static __global__ __launch_bounds__(kBlock) void kb_up(int n, int lw, ROWS rows, const int* __restrict__ ci,
                                                const T* __restrict__ av, const T* __restrict__ zp,
                                                const RT* __restrict__ r, const T* __restrict__ dinv,
                                                const int* __restrict__ aggptr_f, const RTF* __restrict__ r_f,
                                                const T* __restrict__ dinv_f, const T* __restrict__ p_f,
                                                T* __restrict__ zp_f, const int* __restrict__ done) {
    if (*done) return;
    const LaneGroup<CPL> lg(lw);
    const int col0 = lg.col0;
    const TileWalk w = unit_walk(n, lg.gpb, lg.g);
    for (int i = w.first; i < w.end; i += w.stride) {
        T s[CPL];
#pragma unroll
        for (int q = 0; q < CPL; ++q) s[q] = 0;
        row_accumulate<U, CPL, T, T>(rows, i, ci, av, zp, lw, col0, s);
        const Vec<T, CPL> zpi = vload<T, CPL>(zp + ((size_t)i << lw) + col0);
        const Vec<RT, CPL> ri = vload<RT, CPL>(r + ((size_t)i << lw) + col0);
        const T di = dinv[i];
        T z[CPL];
#pragma unroll
        for (int q = 0; q < CPL; ++q) z[q] = zpi.v[q] + di * ((T)ri.v[q] - s[q]);
        for (int m = aggptr_f[i]; m < aggptr_f[i + 1]; ++m) {
            const Vec<RTF, CPL> rf = vload<RTF, CPL>(r_f + ((size_t)m << lw) + col0);
            const T df = dinv_f[m], pf = p_f[m];
            Vec<T, CPL> o;
#pragma unroll
            for (int q = 0; q < CPL; ++q) o.v[q] = prolong_value(df, (T)rf.v[q], pf, z[q]);
            vstore<T, CPL>(zp_f + ((size_t)m << lw) + col0, o);
        }
    }
}

// Level-0 up-sweep: z = zp + D^-1 (r - A zp), with per-column partials of
// z . dv.  Fixed shape, whatever the tuning and the width (its partial sums
// must not depend on them): kFixedRows rows a workgroup, four lanes a row
// (W / 4 columns per lane, one 16-byte load in FP32 at W = 16, two in FP64),
// unroll 8.  z is written in the cycle's precision T: with the FP32 cycle z is
// a float (exactly its FP64 widening), so the Krylov pass gathers half lines.
constexpr int kFixedLanes = 4;
constexpr int kFixedRows = kBlock / kFixedLanes;

template <int CPL, typename T, class ROWS>
static __global__ __launch_bounds__(kBlock) void kb_up0(int n, ROWS rows, const int* __restrict__ ci,
                                                 const T* __restrict__ av, const T* __restrict__ zp,
                                                 const T* __restrict__ r, const T* __restrict__ dinv,
                                                 T* __restrict__ z_out, const double* __restrict__ dv,
                                                 double* __restrict__ partial, const int* __restrict__ done) {
    if (*done) return;
    constexpr int lw = CPL == 4 ? 4 : CPL == 2 ? 3 : 2, W = 1 << lw;
    __shared__ double s_dot[kFixedRows][W];
    const int g = threadIdx.x / kFixedLanes, col0 = (threadIdx.x % kFixedLanes) * CPL;
    const TileWalk w = unit_walk(n, kFixedRows, g);
    double dot[CPL];
#pragma unroll
    for (int q = 0; q < CPL; ++q) dot[q] = 0.0;
    for (int i = w.first; i < w.end; i += w.stride) {
        T s[CPL];
#pragma unroll
        for (int q = 0; q < CPL; ++q) s[q] = 0;
        row_accumulate<8, CPL, T, T>(rows, i, ci, av, zp, lw, col0, s);
        const size_t e = ((size_t)i << lw) + col0;
        const Vec<T, CPL> zv = vload<T, CPL>(zp + e);
        const T di = dinv[i];
#pragma unroll
        for (int q = 0; q < CPL; ++q) {
            const T z = zv.v[q] + di * (r[e + q] - s[q]);
            z_out[e + q] = z;
            dot[q] += (double)z * dv[e + q];
        }
    }
#pragma unroll
    for (int q = 0; q < CPL; ++q) s_dot[g][col0 + q] = dot[q];
    __syncthreads();
    if (threadIdx.x < W) {
        double t = 0.0;
        for (int q = 0; q < kFixedRows; ++q) t += s_dot[q][threadIdx.x];
        partial[(size_t)blockIdx.x * W + threadIdx.x] = t;
    }
}

// Coarsest level: Z = A_L^-1 R (nL x nL times nL x W), then prolongation
// into level L-1 or (single level) z out with per-column partials of z . dv.
// FP64 uses the matrix cores: v_mfma_f64_16x16x4_f64 on 16-row blocks, one
// wave per block.  Z goes through the scratch zc (nL x W).
template <typename T, typename RT, typename RTF, bool OUT>
static __global__ __launch_bounds__(kCoarseThreads) void kb_coarse(
    int nL, int lw, const T* __restrict__ ainv, const RT* __restrict__ r, T* __restrict__ zc,
    const int* __restrict__ aggptr_f, const RTF* __restrict__ r_f, const T* __restrict__ dinv_f,
    const T* __restrict__ p_f, T* __restrict__ zp_f, double* __restrict__ z_out, const double* __restrict__ dv,
    double* __restrict__ partial, const int* __restrict__ done) {
    if (*done) return;
    const int tid = threadIdx.x, wave = tid / 64, l = tid % 64;
    constexpr int kWaves = kCoarseThreads / 64;
    const int W = 1 << lw;
    if constexpr (std::is_same<T, double>::value) {
        // A tile (16 x 4): lane l holds A[l % 16][l / 16]; B tile (4 x 16):
        // lane l holds B[l / 16][l % 16]; D (16 x 16): result register i of
        // lane l holds row 4 i + l / 16 of column l % 16 (one-row groups for
        // the FP64 instruction).
        using d4 = __attribute__((__vector_size__(4 * sizeof(double)))) double;
        for (int rb = wave; rb * 16 < nL; rb += kWaves) {
            d4 acc = {0.0, 0.0, 0.0, 0.0};
            const int m = rb * 16 + (l % 16);
            for (int k0 = 0; k0 < nL; k0 += 4) {
                const int k = k0 + l / 16;
                const double a = (m < nL && k < nL) ? ainv[(size_t)m * nL + k] : 0.0;
                const double b = (k < nL && l % 16 < W) ? (double)r[((size_t)k << lw) + (l % 16)] : 0.0;
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc, 0, 0, 0);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = rb * 16 + 4 * i + (l / 16);
                if (row < nL && l % 16 < W) zc[((size_t)row << lw) + (l % 16)] = acc[i];
            }
        }
    } else {
        for (int e = tid; e < nL << lw; e += kCoarseThreads) {
            const int I = e >> lw, c = e & (W - 1);
            T s = 0;
            for (int j = 0; j < nL; ++j) s += ainv[(size_t)I * nL + j] * (T)r[((size_t)j << lw) + c];
            zc[e] = s;
        }
    }
    __threadfence_block();
    __syncthreads();
    if constexpr (OUT) {
        // thread t: column t mod W, rows t / W + 64 i (64 rows at every width,
        // so that a column's dot product is the same bits at each)
        __shared__ double s_dot[kCoarseThreads];
        const int stride = (kCoarseThreads / kW) << lw;
        double dot = 0.0;
        if (tid < stride)
            for (int e = tid; e < nL << lw; e += stride) {
                const T z = zc[e];
                z_out[e] = (double)z;
                dot += (double)z * dv[e];
            }
        s_dot[tid] = dot;
        __syncthreads();
        if (tid < W) {
            double t = 0.0;
            for (int q = tid; q < stride; q += W) t += s_dot[q];
            partial[tid] = t;
        }
    } else {
        for (int e = tid; e < nL << lw; e += kCoarseThreads) {
            const int I = e >> lw, c = e & (W - 1);
            const T z = zc[e];
            for (int m = aggptr_f[I]; m < aggptr_f[I + 1]; ++m)
                zp_f[((size_t)m << lw) + c] = prolong_value(dinv_f[m], (T)r_f[((size_t)m << lw) + c], p_f[m], z);
        }
    }
}

// Large coarsest level (L >= 1): the product and the prolongation into level
// L-1 spread over many workgroups of 256 threads that own 16 rows each (OUT: the
// product is written to z_out instead, n_L x W in FP64, for the per-operator
// parity check).  FP64: the workgroup's four waves split the columns j in four
// ranges on the matrix cores, the four tiles meeting in LDS in range order.
// FP32: its threads split the columns j in 16 fixed ranges (one row and all W
// right-hand sides per thread), meeting in LDS in a fixed order.  Both are bound
// by the chain of their loads (a few MB from L2), so several steps' loads are
// issued together: FP64 at 1096 rows 120 us with one wave over all columns and a
// load per step, now 16; FP32 18.4 us with a load per step, now 12.5.
constexpr int kCoarseBlockRows = 16;
// Coarsest sizes from which the many-workgroup kernel replaces the single
// workgroup, whose time is its chain of n_L / 4 loads: FP64 at 210 rows 26.9 us
// against 5.2, so below 64 rows (8 us by that chain) there is little to split.
template <typename T>
constexpr int coarse_rows_min_b() { return std::is_same<T, double>::value ? 64 : 32; }
inline int coarse_rows_grid_b(int nL) { return (nL + kCoarseBlockRows - 1) / kCoarseBlockRows; }

// The FP32 ranges of kb_coarse_rows: row I's products over columns [j0, j1), one
// after the other, for W right-hand sides in registers; the loads of U columns
// are in flight together.
template <int W, typename T, typename RT>
static __device__ void coarse_range(int nL, int I, int j0, int j1, const T* __restrict__ ainv, const RT* __restrict__ r,
                                    T* __restrict__ out) {
    constexpr int U = 4;
    T acc[W];
#pragma unroll
    for (int c = 0; c < W; ++c) acc[c] = 0;
    if (I < nL) {
        int j = j0;
        for (; j + U <= j1; j += U) {
            T a[U], v[U][W];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                a[u] = ainv[(size_t)(j + u) * nL + I];
#pragma unroll
                for (int c = 0; c < W; ++c) v[u][c] = (T)r[(size_t)(j + u) * W + c];
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int c = 0; c < W; ++c) acc[c] += a[u] * v[u][c];
        }
        for (; j < j1; ++j) {
            const T a = ainv[(size_t)j * nL + I];
#pragma unroll
            for (int c = 0; c < W; ++c) acc[c] += a * (T)r[(size_t)j * W + c];
        }
    }
#pragma unroll
    for (int c = 0; c < W; ++c) out[c] = acc[c];
}

template <typename T, typename RT, typename RTF, bool OUT = false>
static __global__ __launch_bounds__(kBlock) void kb_coarse_rows(
    int nL, int lw, const T* __restrict__ ainv, const RT* __restrict__ r,
    const int* __restrict__ aggptr_f, const RTF* __restrict__ r_f, const T* __restrict__ dinv_f,
    const T* __restrict__ p_f, T* __restrict__ zp_f, double* __restrict__ z_out, const int* __restrict__ done) {
    if (*done) return;
    constexpr int R = kCoarseBlockRows, G = std::is_same<T, double>::value ? kBlock / 64 : kBlock / R;
    __shared__ T s_part[G][R][kW + 1];
    const int tid = threadIdx.x, W = 1 << lw;
    if constexpr (std::is_same<T, double>::value) {
        using d4 = __attribute__((__vector_size__(4 * sizeof(double)))) double;
        constexpr int U = 8;                                // k steps whose loads are in flight together
        const int wave = tid / 64, l = tid % 64, col = l % 16;
        const int m = min((int)blockIdx.x * R + col, nL - 1);       // rows past the end repeat the last: not stored
        const int steps = (nL + 3) / 4;
        const int s0 = steps * wave / G, s1 = steps * (wave + 1) / G;
        d4 acc = {0.0, 0.0, 0.0, 0.0};
        for (int t = s0; t < s1; t += U) {
            double a[U], b[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = 4 * (t + u) + l / 16;
                const bool in = t + u < s1 && k < nL;
                a[u] = in ? ainv[(size_t)m * nL + k] : 0.0;
                b[u] = in && col < W ? (double)r[((size_t)k << lw) + col] : 0.0;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], b[u], acc, 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) s_part[wave][4 * i + l / 16][col] = acc[i];
    } else {
        const int g = tid / R, lt = tid % R;
        const int I = blockIdx.x * R + lt;
        const int j0 = (int)((long long)nL * g / G), j1 = (int)((long long)nL * (g + 1) / G);
        if (lw == 2)
            coarse_range<4>(nL, I, j0, j1, ainv, r, s_part[g][lt]);
        else if (lw == 3)
            coarse_range<8>(nL, I, j0, j1, ainv, r, s_part[g][lt]);
        else
            coarse_range<16>(nL, I, j0, j1, ainv, r, s_part[g][lt]);
    }
    __syncthreads();
    for (int e = tid; e < R << lw; e += kBlock) {
        const int row = e >> lw, c = e & (W - 1);
        const int II = blockIdx.x * R + row;
        if (II >= nL) continue;
        T z = s_part[0][row][c];
        for (int q = 1; q < G; ++q) z += s_part[q][row][c];
        if constexpr (OUT) {
            z_out[((size_t)II << lw) + c] = (double)z;
            continue;
        }
        for (int mm = aggptr_f[II]; mm < aggptr_f[II + 1]; ++mm)
            zp_f[((size_t)mm << lw) + c] = prolong_value(dinv_f[mm], (T)r_f[((size_t)mm << lw) + c], p_f[mm], z);
    }
}

// FP64 -> FP32 copy of cnt values (the FP32 cycle's level-0 right-hand side, for
// the debug entry point and after widening; in the iteration every writer of R
// also writes R32).
static __global__ __launch_bounds__(kBlock) void kb_narrow(long long cnt, const double* __restrict__ src,
                                                    float* __restrict__ dst, const int* __restrict__ done) {
    if (*done) return;
    const long long stride = (long long)gridDim.x * kBlock;
    for (long long i = (long long)blockIdx.x * kBlock + threadIdx.x; i < cnt; i += stride) dst[i] = (float)src[i];
}

// Rows of 2^from values to rows of 2^to (more): each column at its place, zeros in
// the new ones.  cnt: the values written.
static __global__ __launch_bounds__(kBlock) void kb_widen(long long cnt, int from, int to,
                                                          const double* __restrict__ src, double* __restrict__ dst) {
    const long long stride = (long long)gridDim.x * kBlock;
    for (long long i = (long long)blockIdx.x * kBlock + threadIdx.x; i < cnt; i += stride) {
        const int c = (int)(i & ((1 << to) - 1));
        dst[i] = c < 1 << from ? src[((i >> to) << from) + c] : 0.0;
    }
}

// ---------------------------------------------------------------- Krylov

// p = z + beta_c p_old (p = z on a column's first iteration), q = A p as
// A z + beta_c q_old (the same vector in exact arithmetic: only z is
// gathered, one line per entry instead of two), and per-column partials of
// p.q and p.r.  A column on its first iteration, or finished, takes q = A z
// (an idle column's q stays bounded).  q holds q_old on entry; each element
// is read before it is overwritten, by the same lane.  Fixed shape, as kb_up0.
// Bound by the gathered rows of z.  With four columns a lane eight gathers take
// 64 registers, and the compiler put sums between them to stay within 128: one
// to three gathers in flight, 907 us (128^3 trilinear, 16 columns, FP64 z; FP32
// 629); kept apart 132 registers, all eight in flight, 755 us (590).
template <int CPL, typename ZT, class ROWS>
static __global__ __launch_bounds__(kBlock) void kb_krylov_pq(int n, ROWS rows, const int* __restrict__ ci,
                                                       const double* __restrict__ av, const ZT* __restrict__ z,
                                                       const double* __restrict__ p_old, double* __restrict__ p_new,
                                                       double* __restrict__ q, const double* __restrict__ r,
                                                       const BatchState* __restrict__ st, double* __restrict__ partial,
                                                       const int* __restrict__ done) {
    if (*done) return;
    constexpr int lw = CPL == 4 ? 4 : CPL == 2 ? 3 : 2, W = 1 << lw, GPB = kFixedRows;
    __shared__ double s_pq[GPB][W], s_pr[GPB][W];
    const int g = threadIdx.x / kFixedLanes, col0 = (threadIdx.x % kFixedLanes) * CPL;
    bool first[CPL], fresh[CPL];
    double beta[CPL], pq[CPL], pr[CPL];
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        const BatchCol& C = st->col[col0 + c];
        first[c] = C.first != 0;
        fresh[c] = first[c] || C.done != 0;
        beta[c] = C.beta;
        pq[c] = 0.0;
        pr[c] = 0.0;
    }
    const TileWalk w = unit_walk(n, GPB, g);
    for (int i = w.first; i < w.end; i += w.stride) {
        double s[CPL];
#pragma unroll
        for (int c = 0; c < CPL; ++c) s[c] = 0.0;
        row_accumulate<8, CPL, double, ZT, CPL == 4>(rows, i, ci, av, z, lw, col0, s);
        const size_t e = ((size_t)i << lw) + col0;
        const Vec<ZT, CPL> zi = vload<ZT, CPL>(z + e);
        const Vec<double, CPL> po = vload<double, CPL>(p_old + e);
        const Vec<double, CPL> qo = vload<double, CPL>(q + e), ri = vload<double, CPL>(r + e);
        Vec<double, CPL> pn, qn;
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            const double zc = (double)zi.v[c];
            pn.v[c] = first[c] ? zc : zc + beta[c] * po.v[c];
            qn.v[c] = fresh[c] ? s[c] : s[c] + beta[c] * qo.v[c];
            pq[c] += pn.v[c] * qn.v[c];
            pr[c] += pn.v[c] * ri.v[c];
        }
        vstore<double, CPL>(p_new + e, pn);
        vstore<double, CPL>(q + e, qn);
    }
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        s_pq[g][col0 + c] = pq[c];
        s_pr[g][col0 + c] = pr[c];
    }
    __syncthreads();
    if (threadIdx.x < W) {
        double a = 0.0, b = 0.0;
        for (int t = 0; t < GPB; ++t) { a += s_pq[t][threadIdx.x]; b += s_pr[t][threadIdx.x]; }
        partial[((size_t)blockIdx.x * W + threadIdx.x) * 2] = a;
        partial[((size_t)blockIdx.x * W + threadIdx.x) * 2 + 1] = b;
    }
}

// The vector kernels below take kRowGroups rows a workgroup, one lane per
// column (kRowGroups W threads), whatever the width.
constexpr int kRowGroups = kBlock / kW;

// x += alpha_c p, r -= alpha_c q for the active columns; partials of r.r.
// r32 (the FP32 cycle): r rounded to FP32 beside it, the cycle's level-0
// right-hand side.
static __global__ __launch_bounds__(kBlock) void kb_update(int n, int lw, double* __restrict__ x, double* __restrict__ r,
                                                    float* __restrict__ r32, const double* __restrict__ p,
                                                    const double* __restrict__ q, const BatchState* __restrict__ st,
                                                    double* __restrict__ partial, const int* __restrict__ done) {
    if (*done) return;
    constexpr int GPB = kRowGroups;
    const int W = 1 << lw;
    __shared__ double s_rr[GPB][kW];
    const int g = threadIdx.x >> lw, lane = threadIdx.x & (W - 1);
    const bool live = st->col[lane].done == 0;
    const double alpha = st->col[lane].alpha;
    double rr = 0.0;
    const int stride = gridDim.x * GPB;
    for (int i = blockIdx.x * GPB + g; i < n; i += stride) {
        const size_t e = ((size_t)i << lw) + lane;
        double ri = r[e];
        if (live) {
            x[e] += alpha * p[e];
            ri -= alpha * q[e];
            r[e] = ri;
            if (r32) r32[e] = (float)ri;
        }
        rr += ri * ri;
    }
    s_rr[g][lane] = rr;
    __syncthreads();
    if ((int)threadIdx.x < W) {
        double t = 0.0;
        for (int q2 = 0; q2 < GPB; ++q2) t += s_rr[q2][threadIdx.x];
        partial[(size_t)blockIdx.x * W + threadIdx.x] = t;
    }
}

// Fixed-order per-column sums of `count` partials (partial gi of column c at
// ((gi * W + c) * stride + off)) by one workgroup of kFinParts W threads: thread
// t takes column t mod W and the partials gi = t / W, + kFinParts, ...
// (neighbouring threads read neighbouring columns of one partial), four loads
// in flight; the kFinParts part sums of a column then meet in LDS in part
// order.  The result is valid in threads 0 .. W-1 (thread c: column c).
constexpr int kFinParts = 64;
constexpr int kFinThreads = kFinParts * kW;

__device__ __forceinline__ double col_sum(const double* __restrict__ partial, int count, int stride, int off, int lw,
                                          double (*s_part)[kW]) {
    const int c = threadIdx.x & ((1 << lw) - 1), part = threadIdx.x >> lw;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    int gi = part;
    const auto at = [&](int g) { return partial[(((size_t)g << lw) + c) * stride + off]; };
    for (; gi + 3 * kFinParts < count; gi += 4 * kFinParts) {
        s0 += at(gi);
        s1 += at(gi + kFinParts);
        s2 += at(gi + 2 * kFinParts);
        s3 += at(gi + 3 * kFinParts);
    }
    for (; gi < count; gi += kFinParts) s0 += at(gi);
    s_part[part][c] = (s0 + s1) + (s2 + s3);
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x < (1u << lw))
        for (int q = 0; q < kFinParts; ++q) t += s_part[q][threadIdx.x];
    __syncthreads();
    return t;
}

// all_done = no active column left running (read after the barrier, which
// orders this workgroup's global writes).
__device__ __forceinline__ void update_all_done(BatchState* st) {
    __syncthreads();
    if (threadIdx.x == 0) {
        int all = 1;
        for (int c = 0; c < kW; ++c)
            if (st->col[c].active && !st->col[c].done) all = 0;
        st->all_done = all;
    }
}

// beta (and rho for PCG) from the partials of z.dv.
static __global__ __launch_bounds__(kFinThreads) void kb_fin_beta(int lw, BatchState* __restrict__ st,
                                                                  const double* __restrict__ partial, int count) {
    if (st->all_done) return;
    __shared__ double s_part[kFinParts][kW];
    const int c = threadIdx.x;
    const double d = col_sum(partial, count, 1, 0, lw, s_part);
    if (c < 1 << lw) {
        BatchCol& C = st->col[c];
        if (C.active && !C.done) {
            if (st->krylov == PAMG_KRYLOV_CG) {
                C.rho = d;
                C.beta = C.first ? 0.0 : d / C.rho_old;
            } else {
                C.beta = C.first ? 0.0 : -d / C.delta_old;
            }
        }
    }
}

static __global__ __launch_bounds__(kFinThreads) void kb_fin_alpha(int lw, BatchState* __restrict__ st,
                                                                   const double* __restrict__ partial, int count) {
    if (st->all_done) return;
    __shared__ double s_part[kFinParts][kW];
    const int c = threadIdx.x;
    const double pq = col_sum(partial, count, 2, 0, lw, s_part);
    const double pr = col_sum(partial, count, 2, 1, lw, s_part);
    if (c < 1 << lw) {
        BatchCol& C = st->col[c];
        if (C.active && !C.done) {
            if (!(pq > 0.0)) {
                C.status = (pq != pq) ? PAMG_E_NUMERIC : PAMG_E_NOT_SPD;
                C.done = 1;
                C.alpha = 0.0;
            } else {
                const double num = (st->krylov == PAMG_KRYLOV_CG) ? C.rho : pr;
                C.alpha = num / pq;
                if (st->krylov == PAMG_KRYLOV_CG) C.rho_old = C.rho;
                C.delta_old = pq;
                C.first = 0;
            }
        }
    }
    update_all_done(st);
}

static __global__ __launch_bounds__(kFinThreads) void kb_fin_norm(int lw, BatchState* __restrict__ st,
                                                                  const double* __restrict__ partial, int count) {
    if (st->all_done) return;
    __shared__ double s_part[kFinParts][kW];
    const int c = threadIdx.x;
    const double rr = col_sum(partial, count, 1, 0, lw, s_part);
    if (c < 1 << lw) {
        BatchCol& C = st->col[c];
        if (C.active && !C.done) {
            const double rn = sqrt(rr);
            C.rnorm = rn;
            const int it = C.iter + 1;
            C.iter = it;
            if (rn != rn) {
                C.status = PAMG_E_NUMERIC;
                C.done = 1;
            } else if (C.fixed_iters > 0) {
                if (it >= C.fixed_iters) { C.status = PAMG_OK; C.done = 1; }
            } else if (rn <= C.tol * C.bnorm) {
                C.status = PAMG_OK;
                C.done = 1;
            } else if (it >= C.maxit) {
                C.status = PAMG_NOT_CONVERGED;
                C.done = 1;
            }
        }
    }
    update_all_done(st);
}

// Start (or restart) the columns in `mask`: ||b|| and ||r|| from partials
// (bb_count == 0: keep bnorm), first iteration next, stopping state.
static __global__ __launch_bounds__(kFinThreads) void kb_fin_init(int lw, BatchState* __restrict__ st,
                                                                  const double* __restrict__ bb_part, int bb_count,
                                                                  const double* __restrict__ rr_part, int rr_count,
                                                                  int mask) {
    __shared__ double s_part[kFinParts][kW];
    const int c = threadIdx.x;
    const double bb = bb_count > 0 ? col_sum(bb_part, bb_count, 1, 0, lw, s_part) : 0.0;
    const double rr = col_sum(rr_part, rr_count, 1, 0, lw, s_part);
    if (c < 1 << lw && ((mask >> c) & 1)) {
        BatchCol& C = st->col[c];
        if (bb_count > 0) C.bnorm = sqrt(bb);
        C.rnorm = sqrt(rr);
        C.first = 1;
        C.done = 0;
        C.active = 1;
        C.status = PAMG_NOT_CONVERGED;
        if (C.bnorm == 0.0) {
            C.status = PAMG_OK;
            C.done = 2;   // zero right-hand side: x = 0
        } else if (C.fixed_iters <= 0 && C.rnorm <= C.tol * C.bnorm) {
            C.status = PAMG_OK;
            C.done = 1;
        } else if (C.rnorm != C.rnorm) {
            C.status = PAMG_E_NUMERIC;
            C.done = 1;
        }
    }
    update_all_done(st);
}

// Load columns from caller buffers (src[c] != nullptr: column c of b in the
// caller's numbering): B[:, c] = b_c (hierarchical order), R[:, c] = B[:, c],
// X[:, c] = 0; per-column partials of b.b (also r.r).
static __global__ __launch_bounds__(kBlock) void kb_load(int n, int lw, const int* __restrict__ iperm,
                                                  const double* const* __restrict__ src, double* __restrict__ B,
                                                  double* __restrict__ R, float* __restrict__ R32,
                                                  double* __restrict__ X, double* __restrict__ partial) {
    constexpr int GPB = kRowGroups;
    const int W = 1 << lw;
    __shared__ double s_bb[GPB][kW];
    const int g = threadIdx.x >> lw, lane = threadIdx.x & (W - 1);
    const double* sc = src[lane];
    double bb = 0.0;
    const int stride = gridDim.x * GPB;
    for (int i = blockIdx.x * GPB + g; i < n; i += stride) {
        const size_t e = ((size_t)i << lw) + lane;
        if (sc) {
            const double v = sc[iperm[i]];
            B[e] = v;
            R[e] = v;
            if (R32) R32[e] = (float)v;
            X[e] = 0.0;
            bb += v * v;
        }
    }
    s_bb[g][lane] = bb;
    __syncthreads();
    if ((int)threadIdx.x < W) {
        double t = 0.0;
        for (int q = 0; q < GPB; ++q) t += s_bb[q][threadIdx.x];
        partial[(size_t)blockIdx.x * W + threadIdx.x] = t;
    }
}

// Store columns (dst[c] != nullptr): dst_c[i] = X[perm[i], c] (caller order);
// a column whose right-hand side was zero gets x = 0.
static __global__ __launch_bounds__(kBlock) void kb_store(int n, int lw, const int* __restrict__ perm, double* const* __restrict__ dst,
                                                   const double* __restrict__ X, const BatchState* __restrict__ st) {
    constexpr int GPB = kRowGroups;
    const int W = 1 << lw;
    const int g = threadIdx.x >> lw, lane = threadIdx.x & (W - 1);
    double* dc = dst[lane];
    if (!dc) return;
    const bool zero = st->col[lane].done == 2;
    const int stride = gridDim.x * GPB;
    for (int i = blockIdx.x * GPB + g; i < n; i += stride) dc[i] = zero ? 0.0 : X[((size_t)perm[i] << lw) + lane];
}

// Y = B - A X (all columns) and per-column partials of y.y; with `commit`
// set, columns in `mask` also take Y as their recurrence residual R.
template <class ROWS>
static __global__ __launch_bounds__(kBlock) void kb_resid(int n, int lw, ROWS rows, const int* __restrict__ ci,
                                                   const double* __restrict__ av, const double* __restrict__ X,
                                                   const double* __restrict__ B, double* __restrict__ Y,
                                                   double* __restrict__ R, float* __restrict__ R32, int mask,
                                                   double* __restrict__ partial) {
    constexpr int GPB = kRowGroups;
    const int W = 1 << lw;
    __shared__ double s_yy[GPB][kW];
    const int g = threadIdx.x >> lw, lane = threadIdx.x & (W - 1);
    const TileWalk w = unit_walk(n, GPB, g);
    double yy = 0.0;
    const bool commit = R != nullptr && ((mask >> lane) & 1);
    for (int i = w.first; i < w.end; i += w.stride) {
        double s[1] = {0.0};
        row_accumulate<4, 1, double, double>(rows, i, ci, av, X, lw, lane, s);
        const size_t e = ((size_t)i << lw) + lane;
        const double y = B[e] - s[0];
        Y[e] = y;
        if (commit) {
            R[e] = y;
            if (R32) R32[e] = (float)y;
        }
        yy += y * y;
    }
    s_yy[g][lane] = yy;
    __syncthreads();
    if ((int)threadIdx.x < W) {
        double t = 0.0;
        for (int q = 0; q < GPB; ++q) t += s_yy[q][threadIdx.x];
        partial[(size_t)blockIdx.x * W + threadIdx.x] = t;
    }
}

// 16 caller vectors (column c at src + c*n, canonical order) into the
// hierarchical n x 16 layout, and back.
template <typename D>
static __global__ __launch_bounds__(kBlock) void kb_cols_in(int n, const int* __restrict__ iperm,
                                                            const double* __restrict__ src, D* __restrict__ dst) {
    const long long total = (long long)n * kW;
    const long long stride = (long long)gridDim.x * kBlock;
    for (long long e = (long long)blockIdx.x * kBlock + threadIdx.x; e < total; e += stride) {
        const int i = (int)(e / kW), c = (int)(e % kW);
        dst[e] = (D)src[(size_t)c * n + iperm[i]];
    }
}

template <typename S>
static __global__ __launch_bounds__(kBlock) void kb_cols_out(int n, const int* __restrict__ perm,
                                                             const S* __restrict__ src, double* __restrict__ dst) {
    const long long total = (long long)n * kW;
    const long long stride = (long long)gridDim.x * kBlock;
    for (long long e = (long long)blockIdx.x * kBlock + threadIdx.x; e < total; e += stride) {
        const int c = (int)(e / n), i = (int)(e % n);
        dst[e] = (double)src[(size_t)perm[i] * kW + c];
    }
}

// Gather a level's n x 16 block from canonical into hierarchical order (and back).
template <typename S, typename D>
static __global__ __launch_bounds__(kBlock) void kb_permute(int n, const int* __restrict__ idx, const S* __restrict__ src,
                                                     D* __restrict__ dst) {
    const long long total = (long long)n * kW;
    const long long stride = (long long)gridDim.x * kBlock;
    for (long long e = (long long)blockIdx.x * kBlock + threadIdx.x; e < total; e += stride) {
        const int i = (int)(e / kW), c = (int)(e % kW);
        dst[e] = (D)src[(size_t)idx[i] * kW + c];
    }
}

}  // namespace pamg
