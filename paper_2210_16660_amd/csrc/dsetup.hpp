// Device construction of the large levels of the hierarchy (dsetup.hip).
#pragma once

#include "hier.hpp"

namespace pamg {

// An input with at most kDeviceMinRows rows (the dense limit: it may stay a
// single level) is built on the host; below a larger one every level of more
// than kDeviceStopRows rows (or max_coarse, if larger) is built on the device.
// Whole setups with the stop at 65536 rows, 8192 and 1024: 64^3 trilinear 45.3,
// 28.1 and 23.4 ms, 61^3 varying coefficients 42.2, 19.2 and 14.2; with the stop
// at 1024 and 256 (after other changes) 30^3 trilinear 9.5 and 7.9, 40^3 Laplacian
// 8.5 and 7.8.  An input of 13,824 rows: on the host 11.9 ms, on the device 5.4.
constexpr int kDeviceMinRows = 8192, kDeviceStopRows = 256;

// Column dictionaries of a level's tiles (TileDict on the device).
struct DevDict {
    int* span = nullptr;        // 2 per tile: first entry, length
    int* col = nullptr;
    uint16_t* loc = nullptr;    // per matrix entry
    long long len = 0;
    int max_len = 0;
};

// Sliced rows of a level (SellRows on the device; ci is the level's).
struct DevSell {
    int *tiles = nullptr, *rowpos = nullptr, *col = nullptr;
    uint32_t* slot = nullptr;
    uint16_t* loc = nullptr;
    long long len = 0;          // dictionary entries
    int n_tiles = 0, max_len = 0;
    int32_t xcd[9] = {};
};

// One device-built level in hierarchical numbering (LayoutLevel on the
// device); its arrays belong to the hierarchy's allocation list.
struct DevLevelOut {
    int n = 0, nc = 0, pairs = 0, items = 8, n_up = 0, n_down = 0, max_agg = 0;
    long long nnz = 0;
    int *rp = nullptr, *ci = nullptr, *perm = nullptr, *iperm = nullptr, *aggptr = nullptr;
    int *up_tiles = nullptr, *down_tiles = nullptr;
    double *v = nullptr, *vd = nullptr, *dinv = nullptr, *p = nullptr;
    DevDict up_dict, down_dict;
    DevSell sell;                       // n_tiles > 0: ci, v and vd are in its order, and there are no other tiles
    long long nent = 0;                 // stored entries (with the padding of sliced rows)
    // hybrid Gauss-Seidel schedule (GsLevel on the device; device_gs_schedule)
    uint8_t *gs_df = nullptr, *gs_db = nullptr;
    int *gs_maxd = nullptr, *gs_fresh = nullptr;
    double* gs_ainv = nullptr;
    int gs_nblk = 0;
};

struct DeviceBuild {
    int m = 0;                          // (kept) levels 0..m-1 built on the device
    std::vector<DevLevelOut> dev;
    HostHierarchy host;                 // levels m..L, built on the host from level m
    std::vector<LayoutLevel> host_lay;  // their layouts
};

// The hybrid Gauss-Seidel schedule of a device-built level with blocks of nb
// rows: the host's gs_schedule, row by row and block by block, on the
// device (depths, in-block entry ranges, 1 / a_ii); arrays allocated on h.
// A non-positive diagonal gives PAMG_E_NOT_SPD, as on the host.
void device_gs_schedule(pamg_hierarchy* h, DevLevelOut& D, int nb, hipStream_t s);

// The configurations the device construction covers: pairwise aggregates
// or their composition, tentative prolongators, the l1-Jacobi or the hybrid
// Gauss-Seidel smoother, weight-eligible edges.
bool device_setup_applies(const pamg_params& prm);

// Build the hierarchy of A (validated host CSR) with its large levels on the
// device; device arrays are allocated on h.  Null: nothing to build on the
// device (a small or asymmetric-pattern input, or long rows): the host build
// applies.
std::unique_ptr<DeviceBuild> device_build(pamg_hierarchy* h, const pamg_csr& A, const pamg_params& prm, int max_coarsest,
                                          hipStream_t s);

}  // namespace pamg
