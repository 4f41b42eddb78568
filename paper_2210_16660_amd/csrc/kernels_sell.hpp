// Kernels of the large levels (gfx950, wave64) on sliced rows.
//
// The level's rows (hierarchical order) are cut into tiles of at most 256
// consecutive rows, whole aggregates, one row per thread of a workgroup; inside
// a tile the rows are sorted by length and their entries stored step by step
// (entry k of all rows is contiguous), padded to the longest row.  Lanes past
// their row's end do not load the padding.  A wave streams its 64 rows with no
// communication at all, each lane summing its own row in column order; the
// sums then go through LDS back to row order, so that every other vector is
// read and written coalesced whatever the sort did.
//
// The vector is gathered once per tile, at the tile's distinct columns (its
// dictionary), into LDS; an entry reads its value through a 16-bit position.
// These passes are bound by HBM traffic, the matrix stream and the gathers that
// miss L2 (counters: 6.4 GB a Krylov pass of 16.9 M rows and 453 M entries, 6.9 GB
// in the dictionary tiles of the smaller levels): in those, 4096 entries are staged
// through LDS as products, so about 150 rows of the 27-point operator share a
// dictionary, 4.9 gathers a row; 256 rows take 4.1.  Without the products the
// kernels need 80 registers and 18 KB of LDS, six workgroups per CU in place of
// four.  16.9 M rows, FP64: Krylov pass 1369 -> 1278 us, down-sweep 1185 ->
// 1108, up-sweep 1302 -> 1217; 2.1 M rows, FP32: 102 -> 83 and 95 -> 85 us.
//
// Tried without gain: tiles of 512 rows (3.3 gathers a row, but the stream of
// six such tiles a CU is slower: within 1 %), four or five workgroups per CU
// with longer batches, seven or eight (spills), every load one batch ahead.
//
// Where it is used (sell_applies, sell_fits): levels of at least two rounds of
// the chip (786,432 rows) whose padding stays within 1.4 times the entries.  A
// tile waits on memory for its gather, its stream and its finish one after the
// other, and only other tiles hide that.  Down- and up-sweep, dictionary tiles
// -> sliced rows, us: 27-point rows, 1.05 million, FP64 65 -> 60 and 68 -> 64,
// FP32 51 -> 43 and 49 -> 45; 528 thousand 34 -> 36 and 39 -> 41, FP32 24 -> 25
// and 27 -> 30; 7-point rows, 1.06 million 29 -> 24 and 31 -> 25, FP32 24 -> 20
// and 24 -> 20; 531 thousand 11 -> 13 and 16 -> 19, FP32 8 -> 11 and 12 -> 15.
#pragma once

#include "kernels.hpp"

namespace pamg {

static_assert(kSellDict <= kDictSlots * kBlock, "dictionary longer than the gather slots");
static_assert(kSlice == kBlock, "one thread per row of a tile");
static_assert(kSellGrid <= kMaxGrid, "one partial per workgroup");

// tiles: two int4 per tile, {first row, end row, first entry, first dictionary
// entry} and {dictionary length, first coarse row, end coarse row, 0}.
// xcd: the tiles of XCD x are xcd[x] .. xcd[x + 1] - 1, equal shares of the
// level's rows (shares of the tiles, whose size varies where dictionaries had
// to be cut, left up to 30 % of the chip idle).  slot[p]: the row (offset in
// its tile, low 16 bits) and length (high 16 bits) of sorted position p.
struct SellView {
    const int4* tiles;
    int ntiles;
    int xcd[kXcds + 1];
    const uint32_t* slot;
    const int* col;
    const uint16_t* loc;
};

// Workgroups of a launch: as many as the chip holds at once (each takes a fixed
// share of the tiles, so one that had to wait for a slot would double the time).
inline int sell_grid(int ntiles) { return ntiles < kSellGrid ? ntiles : kSellGrid; }

// The tiles of this workgroup, as tile_walk with the level's XCD shares.
__device__ __forceinline__ TileWalk sell_tiles_of(const SellView& V) {
    const int G = gridDim.x, b = blockIdx.x;
    if (G < kXcds) return {b, G, V.ntiles};
    const int x = b % kXcds, j = b / kXcds;
    return {V.xcd[x] + j, G / kXcds + (x < G % kXcds ? 1 : 0), V.xcd[x + 1]};
}

// Dynamic LDS: the dictionary values.
template <typename T>
inline size_t sell_lds_bytes(int dmax) { return (size_t)dmax * sizeof(T); }

// Sum of the lane's row: kSellStep steps at a time, their value and position
// loads issued together.  all: steps every lane of the wave has; max: steps of
// its longest row (the first lane's).  Past `all`, a lane repeats its own last
// entry and drops it.
template <typename T>
__device__ __forceinline__ T sell_row(const T* __restrict__ av, const uint16_t* __restrict__ loc, int len, int all,
                                      int max, const T* s_x) {
    constexpr int U = kSellStep, R = 4;
    T s = 0;
    int k = 0;
    for (; k + U <= all; k += U) {
        uint16_t li[U];
        T a[U];
#pragma unroll
        for (int u = 0; u < U; ++u) li[u] = ld_stream(&loc[(k + u) * kSlice]);
#pragma unroll
        for (int u = 0; u < U; ++u) a[u] = ld_stream(&av[(k + u) * kSlice]);
#pragma unroll
        for (int u = 0; u < U; ++u) s += a[u] * s_x[li[u]];
    }
    for (; k < max; k += R) {
        uint16_t li[R];
        T a[R];
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const int e = min(k + u, len - 1) * kSlice;
            li[u] = ld_stream(&loc[e]);
            a[u] = ld_stream(&av[e]);
        }
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const T t = s + a[u] * s_x[li[u]];
            s = k + u < len ? t : s;
        }
    }
    return s;
}

// The tiles of this workgroup.  gather(c): the vector value at column c;
// finish(d, e): called with the tile's descriptor once its row sums are in
// s_sum (row d.x + j at s_sum[j]).  The next tile's descriptor and dictionary
// columns are loaded while a tile streams, so that a tile starts with the
// gather itself.
template <typename T, class Gather, class Finish>
__device__ __forceinline__ void sell_walk(const SellView& V, const T* __restrict__ av, T* s_x, T* s_sum, Gather gather,
                                          Finish finish) {
    const TileWalk w = sell_tiles_of(V);
    const int wave = threadIdx.x >> 6;
    int4 nd{}, ne{};
    int nc[kDictSlots];
    const auto cols = [&]() {
#pragma unroll
        for (int s = 0; s < kDictSlots; ++s) {
            const int j = s * kBlock + (int)threadIdx.x;
            if (s * kBlock < ne.x) nc[s] = V.col[nd.w + (j < ne.x ? j : ne.x - 1)];
        }
    };
    if (w.first < w.end) {
        nd = V.tiles[2 * w.first];
        ne = V.tiles[2 * w.first + 1];
        cols();
    }
    for (int t = w.first; t < w.end; t += w.stride) {
        const int4 d = nd, e = ne;
        const int rows = d.y - d.x;
        T x[kDictSlots];
#pragma unroll
        for (int s = 0; s < kDictSlots; ++s)
            if (s * kBlock < e.x) x[s] = gather(nc[s]);
        if (t + w.stride < w.end) {
            nd = V.tiles[2 * (t + w.stride)];
            ne = V.tiles[2 * (t + w.stride) + 1];
        }
        const int j = min((int)threadIdx.x, rows - 1);      // threads past the tile repeat its last row
        const uint32_t q = V.slot[d.x + j];
#pragma unroll
        for (int s = 0; s < kDictSlots; ++s) {
            const int jj = s * kBlock + (int)threadIdx.x;
            if (s * kBlock < e.x && jj < e.x) s_x[jj] = x[s];
        }
        if (t + w.stride < w.end) cols();
        __syncthreads();                    // dictionary values in LDS
        if (wave * 64 < rows) {
            const int len = (int)(q >> 16);
            const int max = __builtin_amdgcn_readfirstlane(len);
            const int all = __builtin_amdgcn_readlane(len, 63);
            const size_t o = (size_t)d.z + j;
            const T sum = sell_row<T>(av + o, V.loc + o, len, all, max, s_x);
            if ((int)threadIdx.x < rows) s_sum[q & 0xffff] = sum;
        }
        __syncthreads();                    // sums in LDS; s_x is free
        finish(d, e);
        // no barrier here: the next tile writes s_x (free since the barrier
        // above) and s_sum only after its own dictionary barrier
    }
}

// ----------------------------------------------------------------------------
// k_down on sliced rows.
template <typename T, typename RT, typename GT>
static __global__ __launch_bounds__(kBlock, kSellWaves) void ks_down(
    const T* __restrict__ ad, const RT* __restrict__ r, const GT* __restrict__ g, const T* __restrict__ p,
    const int* __restrict__ aggptr, SellView V, T* __restrict__ rc, const int* __restrict__ done) {
    if (*done) return;
    extern __shared__ __align__(16) unsigned char s_dyn[];
    T* s_x = reinterpret_cast<T*>(s_dyn);
    __shared__ T s_sum[kBlock];
    const int tid = threadIdx.x;
    sell_walk<T>(
        V, ad, s_x, s_sum, [&](int c) { return (T)g[c]; },
        [&](const int4& d, const int4& e) {
            // thread j finishes fine row d.x + j, u_m = p_m (r_m - s_m), then
            // sums the members of coarse row e.y + j in order
            const int m = d.x + tid, I = e.y + tid;
            int a0 = 0, a1 = 0;
            if (I < e.z) {
                a0 = aggptr[I] - d.x;
                a1 = aggptr[I + 1] - d.x;
            }
            if (m < d.y) s_sum[tid] = p[m] * ((T)r[m] - s_sum[tid]);
            __syncthreads();
            if (I < e.z) {
                T acc = s_sum[a0];
                for (int j = a0 + 1; j < a1; ++j) acc += s_sum[j];
                rc[I] = acc;
            }
        });
}

// ----------------------------------------------------------------------------
// k_up on sliced rows (modes and outputs as there).
template <typename T, typename RT, typename RTF, int MODE, typename ZO = double>
static __global__ __launch_bounds__(kBlock, kSellWaves) void ks_up(
    const T* __restrict__ av, const T* __restrict__ zp, const RT* __restrict__ r, const T* __restrict__ dinv,
    SellView V, const int* __restrict__ aggptr_f, const RTF* __restrict__ r_f, const T* __restrict__ dinv_f,
    const T* __restrict__ p_f, T* __restrict__ zp_f, ZO* __restrict__ z_out, const double* __restrict__ dv,
    double* __restrict__ partial, const int* __restrict__ done) {
    if (*done) return;
    extern __shared__ __align__(16) unsigned char s_dyn[];
    T* s_x = reinterpret_cast<T*>(s_dyn);
    __shared__ T s_sum[kBlock];
    __shared__ double s_redd[kBlock / 64];
    __shared__ uint8_t s_own[MODE == kUpWide ? kBlock << kMaxAggSteps : 1];
    const int tid = threadIdx.x;
    double dot = 0.0;
    sell_walk<T>(
        V, av, s_x, s_sum, [&](int c) { return zp[c]; },
        [&](const int4& d, const int4&) {
            const int i = d.x + tid;
            const bool own = i < d.y;
            T z = 0;
            if (own) z = zp[i] + dinv[i] * ((T)r[i] - s_sum[tid]);
            if constexpr (MODE == kUpOut) {
                if (own) {
                    z_out[i] = (ZO)z;
                    dot += (double)z * dv[i];
                }
            } else if constexpr (MODE == kUpPair) {
                // aggregates of one or two rows
                if (own) {
                    const int a0 = aggptr_f[i], m1 = aggptr_f[i + 1] - 1;
                    const T v0 = prolong_value(dinv_f[a0], (T)r_f[a0], p_f[a0], z);
                    const T v1 = prolong_value(dinv_f[m1], (T)r_f[m1], p_f[m1], z);
                    zp_f[a0] = v0;
                    if (m1 > a0) zp_f[m1] = v1;
                }
            } else {
                // the tile's fine rows F0..F1, one per thread
                const int F0 = aggptr_f[d.x], F1 = aggptr_f[d.y];
                s_sum[tid] = z;
                if (own)
                    for (int m = aggptr_f[i]; m < aggptr_f[i + 1]; ++m) s_own[m - F0] = (uint8_t)tid;
                __syncthreads();
                for (int m = F0 + tid; m < F1; m += kBlock)
                    zp_f[m] = prolong_value(dinv_f[m], (T)r_f[m], p_f[m], s_sum[s_own[m - F0]]);
            }
        });
    if constexpr (MODE == kUpOut) {
        dot = block_sum(dot, s_redd);
        if (tid == 0) partial[blockIdx.x] = dot;
    }
}

// ----------------------------------------------------------------------------
// k_spmv on sliced rows: y = A x, y = b - A x (with the partial of y . y), or
// the l1-Jacobi step (kSpmvSmooth).
template <typename T, typename XT, typename YT, typename BT = double, int EPI = kSpmvPlain>
static __global__ __launch_bounds__(kBlock, kSellWaves) void ks_spmv(
    const T* __restrict__ av, const XT* __restrict__ xv, const BT* __restrict__ b, const T* __restrict__ dscale,
    YT* __restrict__ y, SellView V, double* __restrict__ partial, const int* __restrict__ done) {
    static_assert(EPI == kSpmvPlain || EPI == kSpmvSmooth, "epilogues of a level's own matrix");
    if (done && *done) return;
    extern __shared__ __align__(16) unsigned char s_dyn[];
    T* s_x = reinterpret_cast<T*>(s_dyn);
    __shared__ T s_sum[kBlock];
    __shared__ double s_redd[kBlock / 64];
    const int tid = threadIdx.x;
    double nrm = 0.0;
    sell_walk<T>(
        V, av, s_x, s_sum, [&](int c) { return (T)xv[c]; },
        [&](const int4& d, const int4&) {
            const int i = d.x + tid;
            if (i >= d.y) return;
            const T s = s_sum[tid];
            if constexpr (EPI == kSpmvSmooth) {
                const T t = (T)((double)b[i] - (double)s);
                y[i] = (YT)((T)xv[i] + dscale[i] * t);
            } else {
                const double v = b ? (double)b[i] - (double)s : (double)s;
                y[i] = (YT)v;
                nrm += v * v;
            }
        });
    if (partial) {
        nrm = block_sum(nrm, s_redd);
        if (tid == 0) partial[blockIdx.x] = nrm;
    }
}

// ----------------------------------------------------------------------------
// k_krylov_pq on sliced rows.
template <typename ZT = double>
static __global__ __launch_bounds__(kBlock, kSellWaves) void ks_krylov_pq(
    const double* __restrict__ av, const ZT* __restrict__ z, const double* __restrict__ p_old,
    double* __restrict__ p_new, double* __restrict__ q, const double* __restrict__ r, SellView V,
    SolveState* __restrict__ st, const double* __restrict__ zpart, int zcount, double* __restrict__ partial,
    const int* __restrict__ done) {
    if (*done) return;
    extern __shared__ __align__(16) unsigned char s_dyn[];
    double* s_x = reinterpret_cast<double*>(s_dyn);
    __shared__ double s_sum[kBlock];
    __shared__ double s_red[kBlock / 64];
    const int tid = threadIdx.x;
    const bool first = st->first != 0;
    const double beta = krylov_beta(st, zpart, zcount, s_red);
    double pq = 0.0, pr = 0.0;
    sell_walk<double>(
        V, av, s_x, s_sum, [&](int c) { return (double)z[c]; },
        [&](const int4& d, const int4&) {
            const int i = d.x + tid;
            if (i >= d.y) return;
            const double s = s_sum[tid], zi = (double)z[i], po = p_old[i], qo = q[i], ri = r[i];
            const double pi = first ? zi : zi + beta * po;
            const double qi = first ? s : s + beta * qo;
            p_new[i] = pi;
            q[i] = qi;
            pq += pi * qi;
            pr += pi * ri;
        });
    pq = block_sum(pq, s_red);
    __syncthreads();
    pr = block_sum(pr, s_red);
    if (tid == 0) {
        partial[2 * blockIdx.x] = pq;
        partial[2 * blockIdx.x + 1] = pr;
    }
}

// ----------------------------------------------------------------------------
// A level's entries (values, columns, positions) into its sliced rows: entry k
// of row i is src[rp[i] + k], or src[idx[rp[i] + k]] (IDX: values in another
// order).  The padding is not written.  A wave takes 64 sorted rows of a tile: a
// whole row at a time (kFillStep entries of a longer one) is read by 8, 16 or 32
// lanes, so that its entries, neighbours in src, cost their lines once; they
// turn in LDS and are written step by step, coalesced.  With idx, 56.6 million
// FP64 values: 1010 us step by step over the whole level with an index per stored
// entry, 430 to 480 with 8 or 16 entries of 256 rows at a time (a row's lines are
// gone from L2 by its next step), now 265.
constexpr int kFillStep = 32;
inline int sell_fill_grid(int ntiles) {
    const long long waves = (long long)kSlice / 64 * ntiles;
    return (int)(waves < 16 * kMaxGrid ? waves : 16 * kMaxGrid);
}

template <typename E, bool IDX>
static __global__ __launch_bounds__(64) void ks_fill(SellView V, const int* __restrict__ rp,
                                                     const int* __restrict__ idx, const E* __restrict__ src,
                                                     E* __restrict__ dst) {
    constexpr int W = kSlice / 64, U = 8;
    __shared__ E s_v[kFillStep][64 + 1];
    const int lane = threadIdx.x;
    for (int w = blockIdx.x; w < W * V.ntiles; w += gridDim.x) {
        const int4 d = V.tiles[2 * (w / W)];
        const int p0 = w % W * 64, m = min(64, d.y - d.x - p0);
        if (m <= 0) continue;
        const uint32_t q = V.slot[d.x + p0 + min(lane, m - 1)];                 // lanes past the rows repeat the last
        const int len = (int)(q >> 16), b = rp[d.x + (int)(q & 0xffff)];
        const int longest = __builtin_amdgcn_readfirstlane(len);
        const int lg = longest > 16 ? 5 : longest > 8 ? 4 : 3, rows = 64 >> lg;
        const int u = lane & ((1 << lg) - 1), g = lane >> lg;
        for (int k0 = 0; k0 < longest; k0 += kFillStep) {
            for (int r0 = g; r0 < 64; r0 += U * rows) {
                int c[U], n[U];
                E x[U];
#pragma unroll
                for (int y = 0; y < U; ++y) {
                    n[y] = __shfl(len, r0 + y * rows);
                    c[y] = __shfl(b, r0 + y * rows) + min(k0 + u, n[y] - 1);
                    if constexpr (IDX) c[y] = idx[c[y]];
                }
#pragma unroll
                for (int y = 0; y < U; ++y) x[y] = src[c[y]];
#pragma unroll
                for (int y = 0; y < U; ++y)
                    if (k0 + u < n[y]) s_v[u][r0 + y * rows] = x[y];
            }
            __syncthreads();
            for (int k = 0; k < min(kFillStep, longest - k0); ++k)
                if (lane < m && k0 + k < len) dst[(size_t)d.z + (size_t)(k0 + k) * kSlice + p0 + lane] = s_v[k][lane];
            __syncthreads();
        }
    }
}

}  // namespace pamg
