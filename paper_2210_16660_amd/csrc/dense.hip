// Coarsest level: dense Cholesky factorization A_L = L L^T and the explicit
// inverse A_L^{-1} = L^{-T} L^{-1}, computed once at setup on the device
// (Sec. 3.1 solves the coarsest system directly).  The V-cycle then applies
// the inverse as one matrix-vector (or, for 16 right-hand sides, one
// matrix-matrix) product.
//
// Blocked algorithms on 64 x 64 tiles of the zero-padded N x N matrix
// (N = n rounded up to 64; the padding carries an identity diagonal, so the
// factor and the inverse of the padded matrix are block-diagonal with the
// wanted ones in the top-left corner):
//   for each block column k, two launches:
//            panel L_ik = A_ik L_kk^{-T} and block row k of
//            X = L^{-1} (X_kc = L_kk^{-1} X_kc, the block forward substitution
//            on the identity); trailing update A_ij -= L_ik L_jk^T (j <= i)
//            and X_mc -= L_mk X_kc (m > k), and in it the Cholesky factor of
//            the next diagonal tile and its triangular inverse, in registers;
//   then     A^{-1} = X^T X on the lower block triangle, mirrored.
// The two halves need the same panel, so they share its launches (with five
// launches a block column the substitution alone took 34 us of them).
// n = 2675: 8.7 -> 1.9 ms (a block column: panel 5.9 us, update 32.5 us, of
// which the next diagonal tile's serial factorization is the longer part).
// Every tile product runs on the matrix cores (v_mfma_f64_16x16x4_f64): one
// wave per 16-row strip of the 64 x 64 output tile, four 16-column tiles.
// All sums have a fixed order, so the result is deterministic.
#include <hip/hip_runtime.h>

#include <cmath>

#include "hier.hpp"

namespace pamg {
namespace {

constexpr int kT = 64;             // tile edge
constexpr int kTP = kT + 1;        // padded LDS row (bank spread)
constexpr int kDenseThreads = 256; // four waves

using d4 = __attribute__((__vector_size__(4 * sizeof(double)))) double;

// acc[ct] += A(strip rows, 0..63) * B(0..63, tile ct columns) for this wave's
// 16-row strip.  MFMA operand layout (16x16x4, FP64): the A fragment lane l
// holds A[l % 16][l / 16], the B fragment lane l holds B[l / 16][l % 16]; the
// result register i of lane l is row 4 i + l / 16, column l % 16.
template <class FA, class FB>
__device__ __forceinline__ void strip_product(d4 (&acc)[4], int wave, int lane, FA a_at, FB b_at) {
    const int ar = 16 * wave + (lane % 16);
    const int kq = lane / 16;
    const int bc = lane % 16;
#pragma unroll 4
    for (int k0 = 0; k0 < kT; k0 += 4) {
        const double a = a_at(ar, k0 + kq);
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) acc[ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b_at(k0 + kq, 16 * ct + bc), acc[ct], 0, 0, 0);
    }
}

__device__ __forceinline__ void zero(d4 (&acc)[4]) {
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) acc[ct] = d4{0.0, 0.0, 0.0, 0.0};
}

// (row, col) inside the 64 x 64 tile of result register i, column tile ct
__device__ __forceinline__ int res_row(int wave, int lane, int i) { return 16 * wave + 4 * i + lane / 16; }
__device__ __forceinline__ int res_col(int lane, int ct) { return 16 * ct + lane % 16; }

// Two tiles into LDS, all loads (two values each: tiles and their rows are 16-byte
// aligned) in flight before the first is stored.  A load and its store at a time,
// a launch waited on memory 32 times over: n = 2675, panel 13.3 us, now 5.9, update
// with the diagonal tile 38, now 32.5, X^T X 512, now 211 (its flops take 185 at
// the rate of a large FP64 product).
__device__ __forceinline__ void load_tiles(double (*S0)[kTP], const double* __restrict__ g0, int ld0,
                                           double (*S1)[kTP], const double* __restrict__ g1, int ld1) {
    constexpr int P = kT * kT / 2 / kDenseThreads;
    double2 x[P], y[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int e = 2 * ((int)threadIdx.x + p * kDenseThreads), r = e / kT, c = e % kT;
        x[p] = *reinterpret_cast<const double2*>(g0 + (size_t)r * ld0 + c);
        y[p] = *reinterpret_cast<const double2*>(g1 + (size_t)r * ld1 + c);
    }
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int e = 2 * ((int)threadIdx.x + p * kDenseThreads), r = e / kT, c = e % kT;
        S0[r][c] = x[p].x;
        S0[r][c + 1] = x[p].y;
        S1[r][c] = y[p].x;
        S1[r][c + 1] = y[p].y;
    }
}

// M = 0 beforehand; scatter the CSR of the coarsest level, identity padding
__global__ __launch_bounds__(kDenseThreads) void k_dense_scatter(int n, int N, const int* __restrict__ rp,
                                                                 const int* __restrict__ ci,
                                                                 const double* __restrict__ v, double* __restrict__ M) {
    const int i = blockIdx.x * kDenseThreads + threadIdx.x;
    if (i >= N) return;
    if (i >= n) {
        M[(size_t)i * N + i] = 1.0;
        return;
    }
    for (int k = rp[i]; k < rp[i + 1]; ++k) M[(size_t)i * N + ci[k]] = v[k];
}

__global__ __launch_bounds__(kDenseThreads) void k_dense_eye(int N, double* __restrict__ X) {
    const int i = blockIdx.x * kDenseThreads + threadIdx.x;
    if (i < N) X[(size_t)i * N + i] = 1.0;
}

// Diagonal tile kb: Cholesky factor (written back with zeros above the
// diagonal) and its triangular inverse into Dinv[kb].  A pivot that is not
// positive sets *bad and is replaced by 1 so that the rest stays finite; the
// host then reports the matrix as not positive definite.
//
// This tile is the serial part of the factorization (one workgroup, one after
// the other), so it is bound by the latency of its 64 column steps.  A thread
// of the 16 x 16 grid holds 4 x 4 entries of the tile and of the inverse in
// registers (rows ty + 16 a, columns tx + 16 b); two steps exchange only their
// two columns and two rows of the inverse through LDS (two buffers, one barrier;
// every thread makes the second step's column and row from the first's itself),
// and both triangles are eliminated together: A_ic -= (a_ij / d_j) a_cj and
// T_i -= (a_ij / d_j) T_j.  The square roots of the pivots stay out of the chain
// and scale L and T at the end.  In LDS with three barriers a step, and the
// inverse afterwards by one thread per column, the tile took 126 us (5.3 of the
// 8.7 ms of n = 2675); in registers with a barrier a step 28, now 22, and the
// update that contains it 32.5.
__device__ __forceinline__ void potrf_tile(double* M, int N, int kb, double* Dinv, int* bad) {
    __shared__ double s_col[2][2][kT];  // columns j and j + 1 of the tile
    __shared__ double s_row[2][2][kT];  // rows j and j + 1 of the inverse
    __shared__ double s_piv[kT];
    const int tx = threadIdx.x % 16, ty = threadIdx.x / 16;
    double* G = M + (size_t)kb * kT * N + (size_t)kb * kT;
    double A[4][4], T[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int r = ty + 16 * a, c = tx + 16 * b;
            A[a][b] = G[(size_t)r * N + c];
            T[a][b] = r == c ? 1.0 : 0.0;
        }
#pragma unroll
    for (int J = 0; J < 4; ++J) {
#pragma unroll 1                        // (unrolled, the code outgrows the instruction cache)
        for (int jj = 0; jj < 16; jj += 2) {
            const int j = 16 * J + jj, buf = (jj >> 1) & 1;
            if ((tx & ~1) == jj) {
#pragma unroll
                for (int a = 0; a < 4; ++a) s_col[buf][tx & 1][ty + 16 * a] = A[a][J];
            }
            if ((ty & ~1) == jj) {
#pragma unroll
                for (int b = 0; b < 4; ++b) s_row[buf][ty & 1][tx + 16 * b] = T[J][b];
            }
            __syncthreads();
            // step j, and what it makes of the pivot of step j + 1
            double d0 = s_col[buf][0][j], d1 = s_col[buf][1][j + 1];
            const double m = s_col[buf][0][j + 1];
            double r0[4], r1[4], c0[4], c1[4], t0[4], t1[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                r0[u] = s_col[buf][0][ty + 16 * u];
                r1[u] = s_col[buf][1][ty + 16 * u];
                c0[u] = s_col[buf][0][tx + 16 * u];
                c1[u] = s_col[buf][1][tx + 16 * u];
                t0[u] = s_row[buf][0][tx + 16 * u];
                t1[u] = s_row[buf][1][tx + 16 * u];
            }
            const bool spd0 = d0 > 0.0;
            if (!spd0) d0 = 1.0;
            const double rd0 = 1.0 / d0, lm = m * rd0;
            d1 -= lm * m;
            const bool spd1 = d1 > 0.0;
            if (!spd1) d1 = 1.0;
            const double rd1 = 1.0 / d1;
            if (threadIdx.x == 0) {
                s_piv[j] = d0;
                s_piv[j + 1] = d1;
                if (!spd0 || !spd1) *bad = 1;
            }
            // columns and rows j + 1 after step j; an entry past its range
            // contributes a zero factor (selected after the loads, which are
            // issued together)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const double l0 = r0[u] * rd0;
                r1[u] = ty + 16 * u > j + 1 ? (r1[u] - l0 * m) * rd1 : 0.0;
                r0[u] = ty + 16 * u > j ? l0 : 0.0;
                c1[u] = tx + 16 * u > j + 1 ? c1[u] - (c0[u] * rd0) * m : 0.0;
                c0[u] = tx + 16 * u > j ? c0[u] : 0.0;
                t1[u] -= lm * t0[u];
            }
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    A[a][b] -= r0[a] * c0[b];
                    T[a][b] -= r0[a] * t0[b];
                    A[a][b] -= r1[a] * c1[b];
                    T[a][b] -= r1[a] * t1[b];
                }
            // no second barrier: the next step writes the other buffer, and
            // this one only after the next barrier
        }
    }
    __syncthreads();
    double* D = Dinv + (size_t)kb * kT * kT;
    double pc[4], pr[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        pc[u] = sqrt(s_piv[tx + 16 * u]);
        pr[u] = sqrt(s_piv[ty + 16 * u]);
    }
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int r = ty + 16 * a, c = tx + 16 * b;
            G[(size_t)r * N + c] = c < r ? A[a][b] / pc[b] : c == r ? pc[b] : 0.0;
            D[r * kT + c] = c <= r ? T[a][b] / pr[a] : 0.0;
        }
}

// The first diagonal tile; k_dense_update factors the others.
__global__ __launch_bounds__(kDenseThreads) void k_dense_potrf_first(double* __restrict__ M, int N,
                                                                     double* __restrict__ Dinv, int* __restrict__ bad) {
    potrf_tile(M, N, 0, Dinv, bad);
}

// Blocks 0 .. t-1, the panel: L_ik = A_ik L_kk^{-T} for the row tiles
// i = kb+1+block; blocks t .. t+kb, block row kb of X = L^{-1}:
// X_kc = L_kk^{-1} X_kc for c = block - t.
__global__ __launch_bounds__(kDenseThreads) void k_dense_panel(double* __restrict__ M, double* __restrict__ X, int N,
                                                               int kb, int t, const double* __restrict__ Dinv) {
    __shared__ double Dk[kT][kTP];
    __shared__ double A[kT][kTP];
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    const int u = blockIdx.x;
    double* G = u < t ? M + (size_t)(kb + 1 + u) * kT * N + (size_t)kb * kT
                      : X + (size_t)kb * kT * N + (size_t)(u - t) * kT;
    load_tiles(Dk, Dinv + (size_t)kb * kT * kT, kT, A, G, N);
    __syncthreads();
    d4 acc[4];
    zero(acc);
    if (u < t)
        strip_product(acc, wave, lane, [&](int r, int k) { return A[r][k]; }, [&](int k, int c) { return Dk[c][k]; });
    else
        strip_product(acc, wave, lane, [&](int r, int k) { return Dk[r][k]; }, [&](int k, int c) { return A[k][c]; });
#pragma unroll
    for (int ct = 0; ct < 4; ++ct)
#pragma unroll
        for (int i = 0; i < 4; ++i) G[(size_t)res_row(wave, lane, i) * N + res_col(lane, ct)] = acc[ct][i];
}

// Decode p -> (i, j), 0 <= j <= i, p = i (i + 1) / 2 + j.
__device__ __forceinline__ void tri_index(long long p, int& i, int& j) {
    int r = (int)((sqrt(8.0 * (double)p + 1.0) - 1.0) * 0.5);
    while ((long long)(r + 1) * (r + 2) / 2 <= p) ++r;
    while ((long long)r * (r + 1) / 2 > p) --r;
    i = r;
    j = (int)(p - (long long)r * (r + 1) / 2);
}

// Blocks 0 .. T-1, T = t (t + 1) / 2, the trailing update A_ij -= L_ik L_jk^T
// for kb < j <= i (one tile per block); the others, X_mc -= L_mk X_kc for
// m = kb+1 .. kb+t and c = 0 .. kb (block T + (m - kb - 1) * (kb + 1) + c).
// Block 0 holds the next diagonal tile, which no other block touches: it
// factors it straight away, beside the rest of the update.
__global__ __launch_bounds__(kDenseThreads) void k_dense_update(double* M, double* X, int N, int kb, long long T,
                                                                double* Dinv, int* bad) {
    __shared__ double P[kT][kTP];
    __shared__ double Q[kT][kTP];
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    d4 acc[4];
    zero(acc);
    double* G;
    if (blockIdx.x < T) {
        int i, j;
        tri_index(blockIdx.x, i, j);
        const int ib = kb + 1 + i, jb = kb + 1 + j;
        load_tiles(P, M + (size_t)ib * kT * N + (size_t)kb * kT, N, Q, M + (size_t)jb * kT * N + (size_t)kb * kT, N);
        __syncthreads();
        strip_product(acc, wave, lane, [&](int r, int k) { return P[r][k]; }, [&](int k, int c) { return Q[c][k]; });
        G = M + (size_t)ib * kT * N + (size_t)jb * kT;
    } else {
        const int u = (int)(blockIdx.x - T);
        const int m = kb + 1 + u / (kb + 1), c0 = u % (kb + 1);
        load_tiles(P, M + (size_t)m * kT * N + (size_t)kb * kT, N, Q, X + (size_t)kb * kT * N + (size_t)c0 * kT, N);
        __syncthreads();
        strip_product(acc, wave, lane, [&](int r, int k) { return P[r][k]; }, [&](int k, int c) { return Q[k][c]; });
        G = X + (size_t)m * kT * N + (size_t)c0 * kT;
    }
#pragma unroll
    for (int ct = 0; ct < 4; ++ct)
#pragma unroll
        for (int q = 0; q < 4; ++q) G[(size_t)res_row(wave, lane, q) * N + res_col(lane, ct)] -= acc[ct][q];
    if (blockIdx.x == 0) {
        __threadfence_block();
        __syncthreads();                // the tile is written
        potrf_tile(M, N, kb + 1, Dinv, bad);
    }
}

// A^{-1}_ab = sum_{k >= a} X_ka^T X_kb for a >= b (one tile per block),
// written to the n x n output and mirrored; on diagonal tiles only the lower
// triangle is computed-and-mirrored so that the output is exactly symmetric.
__global__ __launch_bounds__(kDenseThreads) void k_dense_xtx(const double* __restrict__ X, int N, int nb, int n,
                                                             double* __restrict__ out) {
    __shared__ double Xa[kT][kTP];
    __shared__ double Xb[kT][kTP];
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    int a, b;
    tri_index(blockIdx.x, a, b);
    d4 acc[4];
    zero(acc);
    for (int k = a; k < nb; ++k) {
        load_tiles(Xa, X + (size_t)k * kT * N + (size_t)a * kT, N, Xb, X + (size_t)k * kT * N + (size_t)b * kT, N);
        __syncthreads();
        strip_product(acc, wave, lane, [&](int r, int kk) { return Xa[kk][r]; }, [&](int kk, int c) { return Xb[kk][c]; });
        __syncthreads();
    }
#pragma unroll
    for (int ct = 0; ct < 4; ++ct)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int r = a * kT + res_row(wave, lane, q), c = b * kT + res_col(lane, ct);
            if (r >= n || c >= n || (a == b && c > r)) continue;
            out[(size_t)r * n + c] = acc[ct][q];
            if (r != c) out[(size_t)c * n + r] = acc[ct][q];
        }
}

}  // namespace

std::unique_ptr<DenseWork> dense_work(pamg_context* ctx, int n, hipStream_t s) {
    const int N = (n + kT - 1) / kT * kT;
    const int nb = N / kT;
    const size_t NN = (size_t)N * N;
    std::unique_ptr<DenseWork> w(new DenseWork());
    w->ctx = ctx;
    w->s = s;
    auto get = [&](size_t bytes) {
        void* p = ctx_alloc(ctx, bytes, s);
        w->bufs.push_back({p, bytes});
        return p;
    };
    w->M = static_cast<double*>(get(NN * sizeof(double)));
    w->X = static_cast<double*>(get(NN * sizeof(double)));
    w->D = static_cast<double*>(get((size_t)nb * kT * kT * sizeof(double)));
    w->flag = static_cast<int*>(get(sizeof(int)));
    return w;
}

// A_L^{-1} (FP64, n x n row-major) of the coarsest level from its device CSR,
// in the workspace w (from dense_work for this n).
void coarse_inverse_device(DenseWork& w, int n, const int* rp, const int* ci, const double* v, double* ainv,
                           hipStream_t s) {
    const int N = (n + kT - 1) / kT * kT;
    const int nb = N / kT;
    const size_t NN = (size_t)N * N;
    double* dM = w.M;
    double* dX = w.X;
    double* dD = w.D;
    int* dflag = w.flag;
    HIP_CHECK(hipMemsetAsync(dM, 0, NN * sizeof(double), s));
    HIP_CHECK(hipMemsetAsync(dX, 0, NN * sizeof(double), s));
    HIP_CHECK(hipMemsetAsync(dflag, 0, sizeof(int), s));
    const int rows_grid = (N + kDenseThreads - 1) / kDenseThreads;
    hipLaunchKernelGGL(k_dense_scatter, dim3(rows_grid), dim3(kDenseThreads), 0, s, n, N, rp, ci, v, dM);
    hipLaunchKernelGGL(k_dense_eye, dim3(rows_grid), dim3(kDenseThreads), 0, s, N, dX);
    hipLaunchKernelGGL(k_dense_potrf_first, dim3(1), dim3(kDenseThreads), 0, s, dM, N, dD, dflag);
    for (int kb = 0; kb < nb; ++kb) {
        const int t = nb - kb - 1;
        hipLaunchKernelGGL(k_dense_panel, dim3(t + kb + 1), dim3(kDenseThreads), 0, s, dM, dX, N, kb, t,
                           (const double*)dD);
        const long long T = (long long)t * (t + 1) / 2;
        if (t > 0)
            hipLaunchKernelGGL(k_dense_update, dim3((unsigned)(T + (long long)t * (kb + 1))), dim3(kDenseThreads), 0,
                               s, dM, dX, N, kb, T, dD, dflag);
    }
    hipLaunchKernelGGL(k_dense_xtx, dim3((unsigned)((long long)nb * (nb + 1) / 2)), dim3(kDenseThreads), 0, s,
                       (const double*)dX, N, nb, n, ainv);
    HIP_CHECK(hipGetLastError());
    int bad = 0;
    HIP_CHECK(hipMemcpyAsync(&bad, dflag, sizeof(int), hipMemcpyDeviceToHost, s));
    HIP_CHECK(hipStreamSynchronize(s));
    if (bad) throw Error(PAMG_E_NOT_SPD, "coarsest matrix is not positive definite");
}

}  // namespace pamg
