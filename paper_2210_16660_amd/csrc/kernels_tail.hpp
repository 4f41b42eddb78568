// Building the dense operator of the cycle's last levels (device.hip, "dense
// tail"): B_l = D^-1 + E^T (D^-1 + P B_{l+1} P^T E), E = I - A D^-1, in two
// sparse times dense products of the level's CSR (a few thousand rows at most).
#pragma once

#include "kernels.hpp"

namespace pamg {

constexpr int kTailStep = 8;    // entries of a row in flight together: both products are chains of their loads

// own[m] = the aggregate of row m.
static __global__ __launch_bounds__(kBlock) void k_tail_owners(int nc, const int* __restrict__ aggptr,
                                                        int* __restrict__ own) {
    for (int I = blockIdx.x * kBlock + threadIdx.x; I < nc; I += gridDim.x * kBlock)
        for (int m = aggptr[I]; m < aggptr[I + 1]; ++m) own[m] = I;
}

// G = B_c P^T E (nc x n): kTailRowsG rows I by kTailParts workgroups, those rows
// of B_c in LDS (a row each, every one of them read the whole matrix from L2);
// G_Ij = (B_c P^T)_Ij - (sum_i (B_c P^T)_Ii a_ij) / d_j, column j of A read as
// its row j.
constexpr int kTailRowsG = 4, kTailParts = 4;
static __global__ __launch_bounds__(kBlock) void k_tail_g(int n, int nc, const int* __restrict__ rp, const int* __restrict__ ci,
                                                   const double* __restrict__ v, const double* __restrict__ dinv,
                                                   const double* __restrict__ p, const int* __restrict__ own,
                                                   const double* __restrict__ Bc, double* __restrict__ G) {
    extern __shared__ __align__(16) unsigned char s_dyn[];
    double* s_b = reinterpret_cast<double*>(s_dyn);
    const int I0 = blockIdx.x * kTailRowsG, R = min(kTailRowsG, nc - I0);
    for (int J = threadIdx.x; J < R * nc; J += kBlock) s_b[J] = Bc[(size_t)I0 * nc + J];
    __syncthreads();
    for (int j = blockIdx.y * kBlock + threadIdx.x; j < n; j += gridDim.y * kBlock) {
        double s[kTailRowsG] = {};
        for (int k = rp[j], e = rp[j + 1]; k < e; k += kTailStep) {
            int i[kTailStep], o[kTailStep];
            double a[kTailStep], q[kTailStep];
#pragma unroll
            for (int u = 0; u < kTailStep; ++u) {
                i[u] = ci[min(k + u, e - 1)];
                a[u] = v[min(k + u, e - 1)];
            }
#pragma unroll
            for (int u = 0; u < kTailStep; ++u) {
                o[u] = own[i[u]];
                q[u] = p[i[u]];
            }
#pragma unroll
            for (int u = 0; u < kTailStep; ++u)
#pragma unroll
                for (int r = 0; r < kTailRowsG; ++r) {
                    const double t = s[r] + a[u] * (q[u] * s_b[(r < R ? r : 0) * nc + o[u]]);
                    s[r] = k + u < e ? t : s[r];
                }
        }
        const double pj = p[j], dj = dinv[j];
        const int oj = own[j];
#pragma unroll
        for (int r = 0; r < kTailRowsG; ++r)
            if (r < R) G[(size_t)(I0 + r) * n + j] = pj * s_b[r * nc + oj] - s[r] * dj;
    }
}

// B_l = D^-1 + E^T Z, Z = D^-1 + P G, row i by one workgroup:
// B_ij = [i = j] / d_i + Z_ij - (sum_k a_ik Z_kj) / d_i.
static __global__ __launch_bounds__(kBlock) void k_tail_b(int n, const int* __restrict__ rp, const int* __restrict__ ci,
                                                   const double* __restrict__ v, const double* __restrict__ dinv,
                                                   const double* __restrict__ p, const int* __restrict__ own,
                                                   const double* __restrict__ G, double* __restrict__ B) {
    const int i = blockIdx.x;
    const double di = dinv[i];
    for (int j = threadIdx.x; j < n; j += kBlock) {
        const double zi = p[i] * G[(size_t)own[i] * n + j] + (i == j ? di : 0.0);
        double s = 0.0;
        for (int k = rp[i], e = rp[i + 1]; k < e; k += kTailStep) {
            int m[kTailStep];
            double a[kTailStep], g[kTailStep], q[kTailStep], d[kTailStep];
#pragma unroll
            for (int u = 0; u < kTailStep; ++u) {
                m[u] = ci[min(k + u, e - 1)];
                a[u] = v[min(k + u, e - 1)];
            }
#pragma unroll
            for (int u = 0; u < kTailStep; ++u) {
                g[u] = G[(size_t)own[m[u]] * n + j];
                q[u] = p[m[u]];
                d[u] = dinv[m[u]];
            }
#pragma unroll
            for (int u = 0; u < kTailStep; ++u) {
                const double t = s + a[u] * (q[u] * g[u] + (m[u] == j ? d[u] : 0.0));
                s = k + u < e ? t : s;
            }
        }
        B[(size_t)i * n + j] = (i == j ? di : 0.0) + (zi - di * s);
    }
}

}  // namespace pamg
