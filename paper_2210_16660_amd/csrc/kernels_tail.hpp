// Building the dense operator of the cycle's last levels (device.hip, "dense
// tail"): B_l = D^-1 + E^T (D^-1 + P B_{l+1} P^T E), E = I - A D^-1, in two
// sparse times dense products of the level's CSR (a few thousand rows at most).
#pragma once

#include "kernels.hpp"

namespace pamg {

// own[m] = the aggregate of row m.
static __global__ __launch_bounds__(kBlock) void k_tail_owners(int nc, const int* __restrict__ aggptr,
                                                        int* __restrict__ own) {
    for (int I = blockIdx.x * kBlock + threadIdx.x; I < nc; I += gridDim.x * kBlock)
        for (int m = aggptr[I]; m < aggptr[I + 1]; ++m) own[m] = I;
}

// G = B_c P^T E (nc x n): row I by one workgroup, row I of B_c in LDS;
// G_Ij = (B_c P^T)_Ij - (sum_i (B_c P^T)_Ii a_ij) / d_j, column j of A read as
// its row j.
static __global__ __launch_bounds__(kBlock) void k_tail_g(int n, int nc, const int* __restrict__ rp, const int* __restrict__ ci,
                                                   const double* __restrict__ v, const double* __restrict__ dinv,
                                                   const double* __restrict__ p, const int* __restrict__ own,
                                                   const double* __restrict__ Bc, double* __restrict__ G) {
    extern __shared__ __align__(16) unsigned char s_dyn[];
    double* s_b = reinterpret_cast<double*>(s_dyn);
    const int I = blockIdx.x;
    for (int J = threadIdx.x; J < nc; J += kBlock) s_b[J] = Bc[(size_t)I * nc + J];
    __syncthreads();
    for (int j = threadIdx.x; j < n; j += kBlock) {
        double s = 0.0;
        for (int k = rp[j]; k < rp[j + 1]; ++k) {
            const int i = ci[k];
            s += v[k] * (p[i] * s_b[own[i]]);
        }
        G[(size_t)I * n + j] = p[j] * s_b[own[j]] - s * dinv[j];
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
        for (int k = rp[i]; k < rp[i + 1]; ++k) {
            const int m = ci[k];
            s += v[k] * (p[m] * G[(size_t)own[m] * n + j] + (m == j ? dinv[m] : 0.0));
        }
        B[(size_t)i * n + j] = (i == j ? di : 0.0) + (zi - di * s);
    }
}

}  // namespace pamg
