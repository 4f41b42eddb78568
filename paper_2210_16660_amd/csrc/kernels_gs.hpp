// Hybrid forward/backward Gauss-Seidel smoother (arXiv 2210.16660, Sec. 3.1)
// and the V-cycle kernels that go with it.
//
// The smoother is x <- x + M^-1 (r - A x) with M = blockdiag(omega (L_pp +
// D_pp)): the level's rows (hierarchical order, which is the nested-aggregate
// order) are cut into blocks of nb <= 256 consecutive rows; within a block
// the correction d solves (L_pp + D_pp) d = (r - A x)_p by substitution
// (forward: earlier rows; backward, M^T: later rows) and x += d / omega.
// Blocks are independent (block Jacobi between them), one workgroup each.
// Inside a block the substitution runs by depth: a row's depth is one more
// than the deepest earlier (later) row of the block it couples to, so rows of
// one depth only need results of smaller depths (schedule built at setup).
// The residual of the old iterate, r - A x_old, comes from the row-tile SpMV
// (coalesced, like every other pass over A); the sweep kernel then reads
// only each row's in-block entries, which are consecutive in the sorted row
// (their range is part of the schedule).
#pragma once

#include "kernels.hpp"

namespace pamg {

constexpr int kGsMaxBlock = kBlock;   // largest block (one workgroup of kBlock threads)
constexpr int kGsSmallBlock = 64;     // blocks of <= 64 rows run one wave per workgroup
constexpr int kGsFresh = 16;          // in-block entries of a row held in registers
static_assert(kGsFresh % 4 == 0, "the substitution reads its slots in groups of four");
constexpr int kGsBatch = 8;           // entries past those loaded together in a depth step
// Levels whose blocks are inverted (gs_dense_level; the figures are at k_hgs_dense):
// rows of kGsDenseRow entries or more on average, and before a row in its block
// kGsDenseInBlock on average, or m < kGsDenseInBlock where the inverses of a
// direction take at most 4^(m - 3) MB (m = 5: 16 MB, 6: 64 MB).
constexpr int kGsDenseRow = 64;
constexpr double kGsDenseInBlock = 8.0;

// One sweep from t = r - A x_old (ZERO: x_old = 0 and t = r, the first
// pre-smoothing sweep).  Row i of the block: d_i = (t_i - sum_{fresh j}
// a_ij d_j) / a_ii with fresh = in the block and earlier (forward) / later
// (backward), in column order; x_new = x_old + d / omega.
template <int MAXB, typename T, typename TT, bool BACKWARD, bool ZERO, class ROWS>
static __global__ __launch_bounds__(MAXB) void k_hgs(
    int n, int nb, ROWS R, const int* __restrict__ ci, const T* __restrict__ av, const int2* __restrict__ fr,
    const T* __restrict__ ainv, const uint8_t* __restrict__ depth, const int* __restrict__ maxd,
    const TT* __restrict__ tin, const T* __restrict__ x_old, T* __restrict__ x_new, T omega_inv,
    const int* __restrict__ done) {
    if (*done) return;
    __shared__ T s_d[MAXB];
    const int p = blockIdx.x, t = threadIdx.x;
    const int b0 = p * nb, b1 = min(n, b0 + nb);
    const int i = b0 + t;
    const bool own = t < nb && i < b1;
    constexpr int st = ROWS::kStride;
    int dep = -1, nf = 0, kf = 0;
    T ti = 0, xi = 0, ai = 0;
    if (own) {
        const int2 f = fr[i];
        const int before = f.y & 0xff, after = (f.y >> 8) & 0xff, diag = (f.y >> 16) & 1;
        nf = BACKWARD ? after : before;
        kf = R.entry(i, f.x + (BACKWARD ? before + diag : 0));     // in-block entries: kf, kf + st, ...
        ti = (T)tin[i];
        ai = ainv[i];
        dep = depth[i];
        if constexpr (!ZERO) xi = x_old[i];
    }
    // the row's first kGsFresh in-block entries: every load issued at once
    // (indices clamped into the row's range; entry 0 for a row with none),
    // the conditions applied afterwards, so no load waits for another
    T fa[kGsFresh];
    int fq[kGsFresh];
    const int kb = nf > 0 ? kf : 0, kl = nf > 0 ? nf - 1 : 0;
#pragma unroll
    for (int u = 0; u < kGsFresh; ++u) {
        const int k = kb + min(u, kl) * st;
        fa[u] = av[k];
        fq[u] = ci[k];
    }
#pragma unroll
    for (int u = 0; u < kGsFresh; ++u) {
        fa[u] = u < nf ? fa[u] : T(0);
        fq[u] = u < nf ? fq[u] - b0 : 0;
    }
    // every value a slot can read is finite from the start, so a slot past
    // the row's count (coefficient 0 at column 0) adds exactly +0
    s_d[t] = T(0);
    __syncthreads();
    const int md = maxd[2 * p + (BACKWARD ? 1 : 0)];
    for (int d = 0; d <= md; ++d) {
        if (dep == d) {
            // slots in groups of four: a group's LDS reads are issued
            // together, and a group no row at this depth reaches is skipped
            T fresh = 0;
#pragma unroll
            for (int g = 0; g < kGsFresh; g += 4) {
                if (g == 0 || nf > g) {
                    T dj[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) dj[u] = s_d[fq[g + u]];
#pragma unroll
                    for (int u = 0; u < 4; ++u) fresh += fa[g + u] * dj[u];
                }
            }
            // entries past the registers: kGsBatch at a time, loaded together
            // at clamped indices, added in order, a branch per entry (it
            // holds the level-0 kernels' registers down)
            for (int k0 = kGsFresh; k0 < nf; k0 += kGsBatch) {
                T ab[kGsBatch];
                int cb[kGsBatch];
#pragma unroll
                for (int u = 0; u < kGsBatch; ++u) {
                    const int k = kf + min(k0 + u, nf - 1) * st;
                    ab[u] = av[k];
                    cb[u] = ci[k] - b0;
                }
#pragma unroll
                for (int u = 0; u < kGsBatch; ++u)
                    if (k0 + u < nf) fresh += ab[u] * s_d[cb[u]];
            }
            s_d[t] = (ti - fresh) * ai;
        }
        __syncthreads();
    }
    if (own) x_new[i] = xi + s_d[t] * omega_inv;
}

// ----------------------------------------------------------------------------
// Levels with long rows (smoothed Galerkin levels, wide stencils).  The rows of a
// block of 256 then hold tens of entries in it (23, 42 and 104 before a row on
// the three levels of the 56^3 trilinear operator's smoothed hierarchy), so its
// substitution is a chain of some 200 steps, each waiting on memory for the
// row's entries: 417, 592 and 1516 us a sweep on those levels of 23,032, 2,912
// and 369 rows (FP64, with the residual's pass).  The triangles are inverted
// instead, once at setup: W = (L_pp + D_pp)^-1 (backward: (U_pp + D_pp)^-1), and
// a sweep is one product d = W t, with no chain (a row of W holds at most its
// position in the block: 160 values on average): 17, 12 and 8 us there, the
// inversion 0.49 ms per direction.
// On levels with short rows the substitution stays: level 0 of the
// 27-point operator holds 3 to 4 in-block entries a row, so W would be twice
// the whole matrix (45 us a sweep there, against 47 us for W's bytes alone).
//
// Where the line lies (gs_dense_level).  The chain costs with the entries a row
// has in its block, once they are more than the registers hold; W costs with
// its tiles, which a block of less than 64 rows fills badly (32 KB a block, 4 KB
// a row at nb = 8).  A sweep, substitution -> product, us (both with the
// residual's pass), m the mean entries before a row in its block:
//   2,912 rows of 339:    nb 8, m 3.1, 12 -> 11; nb 16, m 5.6, 13 -> 11;
//                         nb 32, m 10, 28 -> 10
//   23,032 rows of 121:   nb 16, m 5.4, FP64 16 -> 19, FP32 14 -> 12;
//                         nb 24, m 7.5, 21 -> 15; nb 64, m 15, 76 -> 13
//   262 thousand of 118:  nb 8, m 2.7, 105 -> 238; nb 24, m 6.7, 95 -> 127;
//                         nb 32, m 8.3, 101 -> 108, FP32 83 -> 68;
//                         nb 48, m 10.5, 126 -> 91; nb 256, m 22, 564 -> 137
//   1.33 million of 121:  nb 8, 537 -> 1205; nb 24, m 6.7, 549 -> 634;
//                         nb 32, m 8.2, 574 -> 560, FP32 443 -> 319;
//                         nb 48, m 10.5, 652 -> 488; nb 256, 2346 -> 679
//   100 thousand of 81, columns anywhere: nb 256, m 1.3, 62 -> 73.
// With m >= 8 (blocks of 17 rows or more) W holds at most 241 values a row.
//
// W is stored in 64 x 64 tiles, column-major inside a tile, so that the 64
// lanes of a wave (one row each) read 512 consecutive bytes per column; only
// the tiles on and below (backward: above) the diagonal are kept.
constexpr int kGsTile = 64;
constexpr int kGsInvCols = 16;        // columns of W one wave computes

inline int gs_strips(int nb) { return (nb + kGsTile - 1) / kGsTile; }
inline long long gs_dense_block(int nb) {            // values of W per block and direction
    const long long ns = gs_strips(nb);
    return ns * (ns + 1) / 2 * kGsTile * kGsTile;
}
// First value of tile (row strip s, column strip q) inside a block's W.
template <bool BACKWARD>
__device__ __forceinline__ int gs_tile_offset(int ns, int s, int q) {
    return (BACKWARD ? s * ns - s * (s - 1) / 2 + (q - s) : s * (s + 1) / 2 + q) * (kGsTile * kGsTile);
}

// Columns c0 .. c0 + 15 of W for block p (grid: blocks x 16-column groups, one
// wave each): substitution on columns of the identity, rows in order, the
// wave's four 16-lane groups taking every fourth in-block entry of a row and
// meeting in a fixed butterfly.  Rows and columns past the block are zero.
template <bool BACKWARD>
static __global__ __launch_bounds__(64) void k_gs_invert(int n, int nb, int ns, RowIdx R, const int* __restrict__ ci,
                                                         const double* __restrict__ av, const int2* __restrict__ fr,
                                                         const double* __restrict__ ainv, double* __restrict__ W) {
    __shared__ double S[kGsMaxBlock][kGsInvCols + 1];
    const int groups = ns * (kGsTile / kGsInvCols);
    const int p = blockIdx.x / groups, c0 = (blockIdx.x % groups) * kGsInvCols;
    const int lane = threadIdx.x, c = lane % kGsInvCols, part = lane / kGsInvCols;
    const int b0 = p * nb, m = min(n - b0, nb);
    for (int e = lane; e < ns * kGsTile * kGsInvCols; e += 64) S[e / kGsInvCols][e % kGsInvCols] = 0.0;
    __syncthreads();
    // forward: rows from the group's first column down; backward: from its last column up
    const int first = BACKWARD ? min(c0 + kGsInvCols, m) - 1 : c0;
    const int count = BACKWARD ? first + 1 : m - c0;
    for (int u = 0; u < count; ++u) {
        const int i = BACKWARD ? first - u : first + u;
        const int2 f = fr[b0 + i];
        const int before = f.y & 0xff, after = (f.y >> 8) & 0xff, diag = (f.y >> 16) & 1;
        const int o = R.start(b0 + i) + (f.x - R.rp[b0 + i] + (BACKWARD ? before + diag : 0)) * R.stride();
        const int nf = BACKWARD ? after : before;
        double s = 0.0;
#pragma unroll 4
        for (int u4 = part; u4 < nf; u4 += 4) {
            const int k = o + u4 * R.stride();
            s += av[k] * S[ci[k] - b0][c];
        }
        s += __shfl_xor(s, 16, 64);
        s += __shfl_xor(s, 32, 64);
        if (part == 0) S[i][c] = ((i == c0 + c ? 1.0 : 0.0) - s) * ainv[b0 + i];
        __syncthreads();
    }
    double* Wp = W + (size_t)p * (ns * (ns + 1) / 2 * kGsTile * kGsTile);
    const int q = c0 / kGsTile;
    for (int s = BACKWARD ? 0 : q; s < (BACKWARD ? q + 1 : ns); ++s) {
        double* T = Wp + gs_tile_offset<BACKWARD>(ns, s, q) + (c0 % kGsTile) * kGsTile;
        for (int cc = 0; cc < kGsInvCols; ++cc) T[cc * kGsTile + lane] = S[s * kGsTile + lane][cc];
    }
}

// One sweep with the inverted blocks from t = r - A x_old (ZERO: x_old = 0,
// t = r): x_new = x_old + (W t) / omega.  One workgroup per 64-row strip of a
// block (90 blocks of 256 rows fill the chip four ways); wave g takes columns
// g, g + 4, ... of each tile, the 16 loads of a tile issued together and the
// next tile's before this one is used; the four waves' sums meet in LDS in a
// fixed order.
template <typename T, typename TT, bool BACKWARD, bool ZERO>
static __global__ __launch_bounds__(kBlock) void k_hgs_dense(int n, int nb, int ns, const T* __restrict__ W,
                                                             const TT* __restrict__ tin, const T* __restrict__ x_old,
                                                             T* __restrict__ x_new, T omega_inv,
                                                             const int* __restrict__ done) {
    if (*done) return;
    constexpr int G = kBlock / 64, C = kGsTile / G;
    __shared__ T s_t[kGsMaxBlock];
    __shared__ T s_part[G][kGsTile];
    const int p = blockIdx.x / ns, s = blockIdx.x % ns;
    const int b0 = p * nb, m = min(n - b0, nb);
    const int lane = threadIdx.x & 63, g = threadIdx.x >> 6;
    const int q0 = BACKWARD ? s : 0, q1 = BACKWARD ? ns : s + 1;
    const T* __restrict__ Wp = W + (size_t)p * (ns * (ns + 1) / 2 * kGsTile * kGsTile) +
                               gs_tile_offset<BACKWARD>(ns, s, q0) + g * kGsTile + lane;
    T a[C];
#pragma unroll
    for (int u = 0; u < C; ++u) a[u] = Wp[u * G * kGsTile];
    s_t[threadIdx.x] = (int)threadIdx.x < m ? (T)tin[b0 + threadIdx.x] : T(0);
    const int i = s * kGsTile + lane;
    const bool own = g == 0 && i < m;
    T xi = 0;
    if constexpr (!ZERO) xi = own ? x_old[b0 + i] : T(0);
    __syncthreads();
    T acc = 0;
    for (int q = q0; q < q1; ++q) {
        T cur[C];
#pragma unroll
        for (int u = 0; u < C; ++u) cur[u] = a[u];
        Wp += kGsTile * kGsTile;
        if (q + 1 < q1) {
#pragma unroll
            for (int u = 0; u < C; ++u) a[u] = Wp[u * G * kGsTile];
        }
#pragma unroll
        for (int u = 0; u < C; ++u) acc += cur[u] * s_t[q * kGsTile + u * G + g];
    }
    s_part[g][lane] = acc;
    __syncthreads();
    if (own) {
        T d = s_part[0][lane];
#pragma unroll
        for (int u = 1; u < G; ++u) d += s_part[u][lane];
        x_new[b0 + i] = xi + d * omega_inv;
    }
}

// Dense coarsest solve e = A_L^-1 r: one wave per row of the symmetric
// inverse (row I read along its length, 64 consecutive columns per load),
// the lanes' partial sums met in a wave butterfly (fixed order); grid
// ceil(nL / 4) workgroups of four waves.
template <typename T, typename RT>
static __global__ __launch_bounds__(kBlock) void k_gs_coarse(int nL, const T* __restrict__ ainv,
                                                      const RT* __restrict__ r, T* __restrict__ e,
                                                      const int* __restrict__ done) {
    if (*done) return;
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    const int I = blockIdx.x * (kBlock / 64) + wave;
    T s = 0;
    if (I < nL) {
        const T* __restrict__ row = ainv + (size_t)I * nL;
#pragma unroll 4
        for (int j = lane; j < nL; j += 64) s += row[j] * (T)r[j];
    }
    s = wave_sum(s);
    if (I < nL && lane == 0) e[I] = s;
}

// z_m += p_m e_I for the members m of every coarse row I.
template <typename T>
static __global__ __launch_bounds__(kBlock) void k_gs_prolong(int nc, const int* __restrict__ aggptr,
                                                       const T* __restrict__ p, const T* __restrict__ e,
                                                       T* __restrict__ z, const int* __restrict__ done) {
    if (*done) return;
    const int stride = gridDim.x * kBlock;
    for (int I = blockIdx.x * kBlock + threadIdx.x; I < nc; I += stride) {
        const T eI = e[I];
        for (int m = aggptr[I]; m < aggptr[I + 1]; ++m) z[m] = z[m] + p[m] * eI;
    }
}

// Level-0 output: z_out = z (FP64) and per-workgroup partials of z . dv.
template <typename T>
static __global__ __launch_bounds__(kBlock) void k_gs_out(int n, const T* __restrict__ z, double* __restrict__ z_out,
                                                   const double* __restrict__ dv, double* __restrict__ partial,
                                                   const int* __restrict__ done) {
    if (*done) return;
    __shared__ double s_red[kBlock / 64];
    const int stride = gridDim.x * kBlock;
    double dot = 0.0;
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += stride) {
        const double zi = (double)z[i];
        z_out[i] = zi;
        dot += zi * dv[i];
    }
    dot = block_sum(dot, s_red);
    if (threadIdx.x == 0) partial[blockIdx.x] = dot;
}

}  // namespace pamg
