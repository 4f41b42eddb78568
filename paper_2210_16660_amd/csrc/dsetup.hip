// Device construction of the large levels of the AMG hierarchy (arXiv
// 2210.16660, Sec. 3.1), bitwise the host construction (setup.cpp):
//   * l1 diagonal, edge weights of eq. (weights) and the eligibility c > 1;
//   * the matching: concurrent proposals along every vertex's eligible
//     neighbours under the strict order (c desc, lo asc, hi asc), a better
//     proposal displacing a worse one (the Suitor algorithm, as on the host).
//     For a strict total order on the edges this is the greedy matching, which
//     eq. (approximatematch) approximates;
//   * aggregates numbered by smallest member and the tentative prolongator of
//     eq. (prolongator);
//   * the Galerkin product with every coarse entry summed in the canonical
//     order (ascending (min(i,j), max(i,j), i)), one wavefront per coarse row;
//   * with aggregate-size composition (agg_steps = s > 1), every s-th
//     pairwise level kept, its aggregates and prolongator entries composed
//     over the s pairwise steps (p multiplied finest first);
//   * the hierarchical numbering, the permuted rows (columns ascending), the
//     column-scaled values and the tiles' column dictionaries.
// A level is built here while it has more rows than a size floor (and the
// coarsening limit) and short rows (at most kRowCap entries); the first level
// that is not, that reduces too little or has no pair, and every coarser one, is
// built on the host from that level's matrix and near-null vector.
//
// Compiled with -ffp-contract=off: each written floating-point operation is
// one IEEE binary64 operation (division and square root correctly rounded),
// as on the host.
#include <algorithm>
#include <chrono>
#include <climits>
#include <cstring>
#include <numeric>

#include "dsetup.hpp"

namespace pamg {
namespace {

constexpr int kSB = 256;                 // threads of the elementwise and scan kernels
constexpr int kScanItems = 8;
constexpr int kScanTile = kSB * kScanItems;
constexpr int kRowCap = 256;             // longest row of a level built on the device
constexpr int kTermCap = 2 * kRowCap;    // Galerkin terms of one coarse row (two members)
constexpr int kRunCap = 4;               // terms of one coarse entry (2 x 2 members)
constexpr int kDictCap = kMaxItems * kBlock;   // entries of the largest tile
constexpr int kGridCap = 1 << 20;        // workgroups of the grid-stride kernels

inline int grid_for(long long n, int per) {
    long long g = (n + per - 1) / per;
    return (int)std::max<long long>(1, std::min<long long>(g, kGridCap));
}

// Device temporaries of one build (freed when it ends).
struct Temps {
    pamg_context* ctx;
    hipStream_t s;
    std::vector<DevAlloc> list, pending;
    template <typename T>
    T* get(size_t count) {
        const size_t bytes = std::max<size_t>(1, count) * sizeof(T);
        void* p = ctx_alloc(ctx, bytes, s);
        list.push_back({p, bytes});
        return static_cast<T*>(p);
    }
    // Given back at the next drain(): the kernels launched so far may still use
    // it.  (A wait of its own for each left the device idle for a launch's
    // latency, about 250 times in a setup of nine levels.)  What is pending in
    // coarsen() is below what the layout of the level takes later, and large
    // arrays there are given back at once, so the peak is the same.
    void release(void* p) {
        for (size_t i = 0; i < list.size(); ++i)
            if (list[i].p == p) {
                pending.push_back(list[i]);
                list.erase(list.begin() + i);
                return;
            }
    }
    // An array that stays: it belongs to the hierarchy from here on.
    void keep(pamg_hierarchy* h, void* p) {
        for (size_t i = 0; i < list.size(); ++i)
            if (list[i].p == p) {
                h->allocs.push_back(list[i]);
                h->info.device_bytes += list[i].bytes;
                list.erase(list.begin() + i);
                return;
            }
    }
    // The stream has been waited for since the last release.
    void drain() { ctx_free_all(ctx, pending, s); }
    void release_now(void* p, void* q) {
        release(p);
        release(q);
        HIP_CHECK(hipStreamSynchronize(s));
        drain();
    }
    ~Temps() {
        (void)hipStreamSynchronize(s);
        ctx_free_all(ctx, pending, s);
        ctx_free_all(ctx, list, s);
    }
};

template <typename T>
T read1(const T* d, hipStream_t s) {
    T x;
    HIP_CHECK(hipMemcpyAsync(&x, d, sizeof(T), hipMemcpyDeviceToHost, s));
    HIP_CHECK(hipStreamSynchronize(s));
    return x;
}

template <typename T>
void to_host(std::vector<T>& out, const T* d, size_t count, hipStream_t s) {
    out.resize(count);
    if (count) HIP_CHECK(hipMemcpyAsync(out.data(), d, count * sizeof(T), hipMemcpyDeviceToHost, s));
    HIP_CHECK(hipStreamSynchronize(s));
}

template <typename T>
void to_device(T* d, const T* src, size_t count, hipStream_t s) {
    if (count) HIP_CHECK(hipMemcpyAsync(d, src, count * sizeof(T), hipMemcpyHostToDevice, s));
    HIP_CHECK(hipStreamSynchronize(s));
}

#define GRID_STRIDE(i, n) for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < (n); \
                               i += (long long)gridDim.x * blockDim.x)

// ------------------------------------------------------------------ scans

// Exclusive prefix sums of in[0..n) into out[0..n] (out[n] = total); each
// workgroup scans kScanTile elements and leaves its total in blk.
template <typename TIn>
__global__ __launch_bounds__(kSB) void k_scan_local(long long n, const TIn* in, long long* out, long long* blk) {
    __shared__ long long s[kSB];
    const long long i0 = (long long)blockIdx.x * kScanTile + (long long)threadIdx.x * kScanItems;
    long long loc[kScanItems];
    long long sum = 0;
#pragma unroll
    for (int u = 0; u < kScanItems; ++u) {
        const long long i = i0 + u;
        loc[u] = sum;
        sum += (i < n) ? (long long)in[i] : 0;
    }
    s[threadIdx.x] = sum;
    __syncthreads();
    for (int off = 1; off < kSB; off <<= 1) {
        const long long t = threadIdx.x >= (unsigned)off ? s[threadIdx.x - off] : 0;
        __syncthreads();
        s[threadIdx.x] += t;
        __syncthreads();
    }
    const long long excl = s[threadIdx.x] - sum;
#pragma unroll
    for (int u = 0; u < kScanItems; ++u) {
        const long long i = i0 + u;
        if (i <= n) out[i] = excl + loc[u];
    }
    if (threadIdx.x == kSB - 1) blk[blockIdx.x] = s[kSB - 1];
}

__global__ void k_scan_add(long long n, long long* out, const long long* off) {
    GRID_STRIDE(i, n + 1) out[i] += off[i / kScanTile];
}

// out[0..n]: exclusive sums of in[0..n), out[n] the total (returned).
template <typename TIn>
long long scan(Temps& T, long long n, const TIn* in, long long* out, hipStream_t s) {
    const long long nb = (n + 1 + kScanTile - 1) / kScanTile;
    long long* blk = T.get<long long>(nb + 1);
    hipLaunchKernelGGL(k_scan_local<TIn>, dim3((unsigned)nb), dim3(kSB), 0, s, n, in, out, blk);
    if (nb > 1) {
        long long* off = T.get<long long>(nb + 1);
        scan<long long>(T, nb, blk, off, s);
        hipLaunchKernelGGL(k_scan_add, dim3(grid_for(n + 1, kSB)), dim3(kSB), 0, s, n, out, (const long long*)off);
        T.release(off);
    }
    T.release(blk);
    const long long total = read1(out + n, s);
    T.drain();
    return total;
}

__global__ void k_to_int(long long n, const long long* in, int* out) { GRID_STRIDE(i, n) out[i] = (int)in[i]; }

__global__ void k_fill_d(long long n, double* x, double v) { GRID_STRIDE(i, n) x[i] = v; }

// ---------------------------------------------------------- level kernels

// *m = max(*m, x).  Most callers find a value that is large enough and leave:
// one atomic per wavefront on one address held the count pass of the Galerkin
// product over 1.07 million coarse rows to 7.5 ms where the fill pass takes 1.8
// (64^3 trilinear, both passes, all levels: 3.9 ms, now 1.4).
__device__ inline void raise_max(int* m, int x) {
    if (__hip_atomic_load(m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < x) atomicMax(m, x);
}

// d_i = sum_j |a_ij| (ascending columns), a_ii, dinv = 1/d; the longest row.
__global__ void k_l1diag(int n, const int* rp, const int* ci, const double* v, double* dinv, double* diag,
                         int* maxrow) {
    int mx = 0;
    GRID_STRIDE(i, n) {
        double d = 0.0, dg = 0.0;
        for (int k = rp[i]; k < rp[i + 1]; ++k) {
            d += fabs(v[k]);
            if (ci[k] == i) dg = v[k];
        }
        dinv[i] = 1.0 / d;
        diag[i] = dg;
        mx = max(mx, rp[i + 1] - rp[i]);
    }
    raise_max(maxrow, mx);
}

// validate_csr's row checks, one thread per row, in the same order (no
// entry of a row whose bounds are out of order is read): the smallest
// failing row and its check, as (row << 8) | check.
__global__ void k_validate(int n, long long nnz, const int* rp, const int* ci, const double* v,
                           unsigned long long* first) {
    GRID_STRIDE(i, n) {
        const int b = rp[i], e = rp[i + 1];
        int err = 0;
        if (e < b || b < 0 || (long long)e > nnz) err = 1;
        bool diag = false;
        for (int k = b; k < e && !err; ++k) {
            const int c = ci[k];
            if (c < 0 || c >= n) {
                err = 2;
            } else if (k > b && c <= ci[k - 1]) {
                err = 3;
            } else if (c == (int)i) {
                diag = true;
                if (!(v[k] > 0.0)) err = 4;
            }
            if (!isfinite(v[k])) err = 6;
        }
        if (!err && !diag) err = 5;
        if (err) atomicMin(first, ((unsigned long long)i << 8) | (unsigned long long)err);
    }
}

// check_symmetry: every entry has a mirror with the same bits.
__global__ void k_check_symmetry(int n, const int* rp, const int* ci, const double* v, int* asym) {
    GRID_STRIDE(i, n) {
        for (int k = rp[i]; k < rp[i + 1]; ++k) {
            const int j = ci[k];
            int b = rp[j], e = rp[j + 1];
            while (b < e) {
                const int m = (b + e) >> 1;
                if (ci[m] < (int)i) b = m + 1; else e = m;
            }
            if (b >= rp[j + 1] || ci[b] != (int)i || __double_as_longlong(v[b]) != __double_as_longlong(v[k]))
                atomicOr(asym, 1);
        }
    }
}

__device__ inline double edge_weight(double a_lohi, double a_lolo, double a_hihi, double w_lo, double w_hi) {
    double num = ((2.0 * a_lohi) * w_lo) * w_hi;
    double den = (a_lolo * w_lo) * w_lo + (a_hihi * w_hi) * w_hi;
    return 1.0 - num / den;
}

__device__ inline int find_col(const int* ci, int b, int e, int col) {
    while (b < e) {
        const int m = (b + e) >> 1;
        if (ci[m] < col) b = m + 1; else e = m;
    }
    return b;
}

// Weight of every off-diagonal entry from the upper entry (lo, hi) of its
// edge (both directions carry the same value); 0 on the diagonal.  Flags an
// entry whose transposed entry is not stored (the device matching scans rows,
// so the pattern must be symmetric); tr: the transposed entry's position.  A
// search per entry: eight lanes share a row, so that the entries are read in
// runs and a row's searches overlap (64^3 trilinear, all levels: a lane
// per row 1.55 ms, now 0.41).
constexpr int kWeightLanes = 8;
__global__ __launch_bounds__(kSB) void k_weights(int n, const int* rp, const int* ci, const double* v,
                                                 const double* diag, const double* w, double* c, int* tr, int* asym) {
    const int lane = threadIdx.x % kWeightLanes;
    const long long stride = (long long)gridDim.x * (kSB / kWeightLanes);
    for (long long i = (long long)blockIdx.x * (kSB / kWeightLanes) + threadIdx.x / kWeightLanes; i < n; i += stride) {
        const int e = rp[i + 1];
        for (int k = rp[i] + lane; k < e; k += kWeightLanes) {
            const int j = ci[k];
            if (j == (int)i) {
                c[k] = 0.0;
                tr[k] = k;
                continue;
            }
            const int t = find_col(ci, rp[j], rp[j + 1], (int)i);
            if (t >= rp[j + 1] || ci[t] != (int)i) {
                atomicOr(asym, 1);
                c[k] = 0.0;
                tr[k] = k;
                continue;
            }
            tr[k] = t;
            const int lo = min((int)i, j), hi = max((int)i, j);
            const double a = j > (int)i ? v[k] : v[t];
            c[k] = edge_weight(a, diag[lo], diag[hi], w[lo], w[hi]);
        }
    }
}

// Bitonic sort (ascending) of P (a power of two) keys in LDS by one workgroup.
template <typename K>
__device__ inline void lds_bitonic(K* key, int P) {
    for (int size = 2; size <= P; size <<= 1)
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            for (int t = threadIdx.x; t < (P >> 1); t += blockDim.x) {
                const int a = 2 * t - (t & (stride - 1));
                const int b = a + stride;
                const K x = key[a], y = key[b];
                const bool up = (a & size) == 0;
                if ((x > y) == up) {
                    key[a] = y;
                    key[b] = x;
                }
            }
            __syncthreads();
        }
}

// A neighbour of vertex i in the matching order: heavier first; for equal
// weights the edge with the smaller (lo, hi) first, which for a fixed i is
// the smaller neighbour index.  x > y: x comes after y.
struct Nbr {
    double c;
    int j, t;               // t: the entry's place in its row
    __device__ bool operator>(const Nbr& y) const { return c < y.c || (c == y.c && j > y.j); }
};

// Every vertex's eligible neighbours (c > 1) in the matching order, at its
// row's positions in adj; their number in ecnt; pos: an eligible entry's place
// in adj, -1 for the others.  One wavefront per row.
__global__ __launch_bounds__(64) void k_sort_adj(int n, const int* rp, const int* ci, const double* c, int* adj,
                                                 int* pos, int* ecnt) {
    __shared__ Nbr key[kRowCap];
    const int lane = threadIdx.x;
    for (int i = blockIdx.x; i < n; i += gridDim.x) {
        const int b = rp[i], len = rp[i + 1] - b;
        int P = 1;
        while (P < len) P <<= 1;
        int cnt = 0;
        for (int t = lane; t < P; t += 64) {
            Nbr x{-1.0, INT_MAX, 0};
            if (t < len) {
                const int j = ci[b + t];
                const double cc = c[b + t];
                if (j != i && cc > 1.0) {
                    x = Nbr{cc, j, t};
                    ++cnt;
                } else {
                    pos[b + t] = -1;
                }
            }
            key[t] = x;
        }
        for (int off = 32; off > 0; off >>= 1) cnt += __shfl_xor(cnt, off);
        __syncthreads();
        lds_bitonic(key, P);
        for (int t = lane; t < cnt; t += 64) {
            adj[b + t] = key[t].j;
            pos[b + key[t].t] = b + t;
        }
        if (lane == 0) ecnt[i] = cnt;
        __syncthreads();
    }
}

// mirror[e]: the place of edge e of adj in its other endpoint's list (both
// directions of an edge carry the same weight, so both lists hold it).
__global__ void k_mirror(long long nnz, const int* pos, const int* tr, int* mirror) {
    GRID_STRIDE(k, nnz) {
        const int e = pos[k];
        if (e >= 0) mirror[e] = pos[tr[k]];
    }
}

// The matching by proposals: a vertex proposes along its list, heaviest edge
// first, to the first neighbour whose best proposal so far is lighter; a
// vertex whose proposal is displaced goes on from its place in its own list.
// The edges are totally ordered, so the outcome is the one matching in which
// every unmatched edge has a heavier matched neighbour, whatever the order of
// the proposals: bitwise the host's.  best[j] is the place, in j's own list, of
// the edge over which j's best proposal came (smaller is heavier), so that one
// atomic minimum is the whole proposal, and the displaced vertex and its place
// follow from the value it returns through adj and mirror, which do not change:
// nothing else is shared and no thread waits for another.  A plain look at best
// first: its values only fall, so an old one rejects nothing wrongly.  Every
// pass moves one vertex's place forward, so the proposals end.
// Bound by the longest chain of displacements (dependent trips to memory);
// rounds of mutual picks before, three launches each, took 89 rounds a level
// and 7.5 of the 17 ms of kernels of a 64^3 trilinear setup.
constexpr unsigned kNoProposal = 0xffffffffu;
__global__ __launch_bounds__(kSB) void k_propose(int n, const int* __restrict__ rp, const int* __restrict__ ecnt,
                                                 const int* __restrict__ adj, const int* __restrict__ mirror,
                                                 unsigned* best) {
    GRID_STRIDE(i, n) {
        int u = (int)i, at = rp[i];
        for (;;) {
            const int end = rp[u] + ecnt[u];
            unsigned old = kNoProposal;
            for (; at < end; ++at) {
                const int j = adj[at];
                const unsigned m = (unsigned)mirror[at];
                if (__hip_atomic_load(best + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < m) continue;
                old = atomicMin(best + j, m);
                if (m < old) break;
                old = kNoProposal;
            }
            if (old == kNoProposal) break;      // accepted by a free vertex, or the list is through
            u = adj[old];
            at = mirror[old] + 1;
        }
    }
}

// mate[i]: the vertex whose proposal i holds, if that one holds i's.
__global__ void k_mates(int n, const int* adj, const unsigned* best, int* mate) {
    GRID_STRIDE(i, n) {
        int m = -1;
        if (best[i] != kNoProposal) {
            const int u = adj[best[i]];
            if (best[u] != kNoProposal && adj[best[u]] == (int)i) m = u;
        }
        mate[i] = m;
    }
}

// Aggregate leaders (smallest member) and aggregate sizes.
__global__ void k_leaders(int n, const int* mate, int* lead, int* size) {
    GRID_STRIDE(i, n) {
        const int m = mate[i];
        const bool l = m < 0 || m > (int)i;
        lead[i] = l ? 1 : 0;
        size[i] = l ? (m < 0 ? 1 : 2) : 0;
    }
}

// agg, p, the coarse near-null vector, the members of each aggregate.
__global__ void k_aggregate(int n, const int* mate, const double* w, const long long* aid, const long long* msz,
                            int* agg, double* p, double* wc, int* mem_ptr, int* mem) {
    GRID_STRIDE(i, n) {
        const int m = mate[i];
        if (m < 0) {
            const int I = (int)aid[i];
            agg[i] = I;
            p[i] = w[i] / fabs(w[i]);
            wc[I] = fabs(w[i]);
            mem_ptr[I] = (int)msz[i];
            mem[msz[i]] = (int)i;
        } else {
            const int lo = min((int)i, m), hi = max((int)i, m);
            const double nu = sqrt(w[lo] * w[lo] + w[hi] * w[hi]);
            const int I = (int)aid[lo];
            agg[i] = I;
            p[i] = w[i] / nu;
            if ((int)i == lo) {
                wc[I] = nu;
                mem_ptr[I] = (int)msz[i];
                mem[msz[i]] = lo;
                mem[msz[i] + 1] = hi;
            }
        }
    }
}

struct GTerm {
    int k1, k2, k3;
    double t;
};

// Galerkin A_c = P^T A P, one wavefront per coarse row.  The row's terms
// (entries of its members' rows) are sorted by coarse column J; every coarse
// entry then sums its terms in ascending (min(i,j), max(i,j), i).  Count pass
// (FILL false): distinct columns per row, the longest coarse row; fill pass:
// columns and values at crp.
template <bool FILL>
__global__ __launch_bounds__(64) void k_galerkin(int nc, const int* mem_ptr, const int* mem, const int* rp,
                                                 const int* ci, const double* v, const int* agg, const double* p,
                                                 int* cnt, const long long* crp, int* cci, double* cv, int* bad) {
    __shared__ unsigned long long key[kTermCap];
    const int lane = threadIdx.x;
    int longest = 0;
    for (int I = blockIdx.x; I < nc; I += gridDim.x) {
        const int q0 = mem_ptr[I], q1 = mem_ptr[I + 1];
        const int i0 = mem[q0], i1 = q1 - q0 > 1 ? mem[q0 + 1] : -1;
        const int b0 = rp[i0], len0 = rp[i0 + 1] - b0;
        const int b1 = i1 >= 0 ? rp[i1] : 0, len1 = i1 >= 0 ? rp[i1 + 1] - b1 : 0;
        const int T = len0 + len1;
        if (T > kTermCap) {
            if (lane == 0) atomicOr(bad, 1);
            continue;
        }
        int P = 1;
        while (P < T) P <<= 1;
        for (int t = lane; t < P; t += 64) {
            unsigned long long kk = ~0ull;
            if (t < T) {
                const int k = t < len0 ? b0 + t : b1 + (t - len0);
                kk = ((unsigned long long)(unsigned)agg[ci[k]] << 32) | (unsigned)t;
            }
            key[t] = kk;
        }
        __syncthreads();
        lds_bitonic(key, P);
        const long long base = FILL ? crp[I] : 0;
        int runs = 0;
        for (int c0 = 0; c0 < T; c0 += 64) {
            const int s = c0 + lane;
            const bool start = s < T && (s == 0 || (key[s] >> 32) != (key[s - 1] >> 32));
            const unsigned long long mask = __ballot(start);
            if (FILL && start) {
                const int r = runs + __popcll(mask & ((1ull << lane) - 1));
                const unsigned J = (unsigned)(key[s] >> 32);
                GTerm g[kRunCap];
                int m = 0;
                for (int e = s; e < T && (unsigned)(key[e] >> 32) == J; ++e) {
                    if (m == kRunCap) {
                        atomicOr(bad, 2);
                        break;
                    }
                    const int t = (int)(key[e] & 0xffffffffu);
                    const int k = t < len0 ? b0 + t : b1 + (t - len0);
                    const int i = t < len0 ? i0 : i1;
                    const int j = ci[k];
                    GTerm x{min(i, j), max(i, j), i, v[k] * (p[i] * p[j])};
                    int u = m++;
                    while (u > 0 && (g[u - 1].k1 > x.k1 || (g[u - 1].k1 == x.k1 && (g[u - 1].k2 > x.k2 ||
                                     (g[u - 1].k2 == x.k2 && g[u - 1].k3 > x.k3))))) {
                        g[u] = g[u - 1];
                        --u;
                    }
                    g[u] = x;
                }
                double sum = g[0].t;
                for (int u = 1; u < m; ++u) sum = sum + g[u].t;
                cci[base + r] = (int)J;
                cv[base + r] = sum;
            }
            runs += __popcll(mask);
        }
        if (!FILL && lane == 0) cnt[I] = runs;
        longest = max(longest, runs);
        __syncthreads();
    }
    if (!FILL && lane == 0) raise_max(bad + 1, longest);
}

// ------------------------------------------------------------ layout kernels

__global__ void k_agg_sizes(int nc, const int* cip, const int* mem_ptr, int* sz) {
    GRID_STRIDE(Ip, nc) {
        const int I = cip[Ip];
        sz[Ip] = mem_ptr[I + 1] - mem_ptr[I];
    }
}

// Members of the aggregate at hierarchical coarse index Ip take the fine
// positions aggptr[Ip].., ascending.
__global__ void k_place(int nc, int n, const int* cip, const int* mem_ptr, const int* mem, const long long* ap,
                        int* aggptr, int* iperm, int* perm) {
    GRID_STRIDE(Ip, nc) {
        const int I = cip[Ip];
        const int q = (int)ap[Ip];
        aggptr[Ip] = q;
        for (int r = 0; r < mem_ptr[I + 1] - mem_ptr[I]; ++r) {
            const int i = mem[mem_ptr[I] + r];
            iperm[q + r] = i;
            perm[i] = q + r;
        }
        if (Ip == nc - 1) aggptr[nc] = n;
    }
}

__global__ void k_row_len(int n, const int* iperm, const int* rp, int* len) {
    GRID_STRIDE(ip, n) {
        const int i = iperm[ip];
        len[ip] = rp[i + 1] - rp[i];
    }
}

// Row ip of the permuted matrix: row iperm[ip] with columns renumbered by
// perm and sorted ascending (one wavefront per row); dinv and p follow.
__global__ __launch_bounds__(64) void k_reorder(int n, const int* iperm, const int* perm, const int* rp,
                                                const int* ci, const double* v, const double* dinv, const double* p,
                                                const long long* rp2, int* ci2, double* v2, double* dinv2,
                                                double* p2) {
    __shared__ unsigned long long key[kRowCap];
    const int lane = threadIdx.x;
    for (int ip = blockIdx.x; ip < n; ip += gridDim.x) {
        const int i = iperm[ip];
        const int b = rp[i], len = rp[i + 1] - b;
        int P = 1;
        while (P < len) P <<= 1;
        for (int t = lane; t < P; t += 64)
            key[t] = t < len ? (((unsigned long long)(unsigned)perm[ci[b + t]] << 32) | (unsigned)t) : ~0ull;
        __syncthreads();
        lds_bitonic(key, P);
        const long long o = rp2[ip];
        for (int t = lane; t < len; t += 64) {
            ci2[o + t] = (int)(key[t] >> 32);
            v2[o + t] = v[b + (int)(key[t] & 0xffffffffu)];
        }
        if (lane == 0) {
            dinv2[ip] = dinv[i];
            if (p2) p2[ip] = p[i];
        }
        __syncthreads();
    }
}

__global__ void k_vd(long long nnz, const int* ci, const double* v, const double* dinv, double* vd) {
    GRID_STRIDE(k, nnz) vd[k] = v[k] * dinv[ci[k]];
}

// Column dictionary of each tile: its distinct columns, ascending (count
// pass: their number and the longest; fill pass: the columns at the tile's
// offset and every entry's 16-bit position).  A tile longer than cap (one
// long row) has none.
template <bool FILL>
__global__ __launch_bounds__(kSB) void k_dict(int ntiles, const int4* tiles, const int* ci, int cap, int* dlen,
                                              const long long* doff, int* dcol, uint16_t* loc, int* maxlen) {
    __shared__ int key[kDictCap];
    __shared__ int uq[kDictCap];
    __shared__ int wsum[kSB / 64 + 1];
    for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const int4 d = tiles[t];
        const int k0 = d.x, m = d.y - d.x;
        if (m > cap) {
            if (!FILL && threadIdx.x == 0) dlen[t] = 0;
            continue;
        }
        int P = 1;
        while (P < m) P <<= 1;
        for (int u = threadIdx.x; u < P; u += kSB) key[u] = u < m ? ci[k0 + u] : INT_MAX;
        __syncthreads();
        lds_bitonic(key, P);
        // distinct columns: a scan of the run-start flags, kSB-element chunks
        int total = 0;
        for (int c0 = 0; c0 < m; c0 += kSB) {
            const int u = c0 + threadIdx.x;
            const bool st = u < m && (u == 0 || key[u] != key[u - 1]);
            const unsigned long long mask = __ballot(st);
            const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
            if (lane == 0) wsum[wv] = __popcll(mask);
            __syncthreads();
            int before = 0, all = 0;
            for (int q = 0; q < kSB / 64; ++q) {
                if (q < wv) before += wsum[q];
                all += wsum[q];
            }
            if (FILL && st) {
                const int pos = total + before + __popcll(mask & ((1ull << lane) - 1));
                uq[pos] = key[u];
                dcol[doff[t] + pos] = key[u];
            }
            total += all;
            __syncthreads();
        }
        if (!FILL) {
            if (threadIdx.x == 0) {
                dlen[t] = total;
                raise_max(maxlen, total);
            }
        } else {
            for (int u = threadIdx.x; u < m; u += kSB) {
                const int col = ci[k0 + u];
                int b = 0, e = total;
                while (b < e) {
                    const int h = (b + e) >> 1;
                    if (uq[h] < col) b = h + 1; else e = h;
                }
                loc[k0 + u] = (uint16_t)b;
            }
        }
        __syncthreads();
    }
}

__global__ void k_spans(int ntiles, const long long* doff, const int* dlen, int* span) {
    GRID_STRIDE(t, ntiles) {
        span[2 * t] = (int)doff[t];
        span[2 * t + 1] = dlen[t];
    }
}

// Column dictionary of each sliced tile (rows tiles[t].x .. .y; CSR): its
// distinct columns, ascending (count pass: their number, or kSellDict + 1 when
// there are more; fill pass: the columns at the tile's offset and the 16-bit
// position of every stored entry of its slices).  The distinct columns are
// collected in an open-addressing table in LDS, at most half full: a tile
// stops inserting once kDictStop columns are in it, and the inserts of one
// step in flight then add at most kSB more.
constexpr int kDictHash = 8192;                 // table slots
constexpr int kDictStop = kSellDict + kSB;      // a tile with this many columns is split anyway
static_assert(2 * (kDictStop + kSB) <= kDictHash, "the table must stay at most half full");

// Insert the columns of entries [k0, k0 + m) into the table (all slots -1).
__device__ inline void dict_insert(int* table, int* count, const int* ci, int k0, int m) {
    for (int u0 = 0; u0 < m; u0 += kSB) {
        const int u = u0 + threadIdx.x;
        const bool room = *(volatile int*)count < kDictStop;
        if (u < m && room) {
            const int c = ci[k0 + u];
            unsigned h = ((unsigned)c * 2654435761u) >> 19;     // 13 bits
            for (;;) {
                const int old = atomicCAS(&table[h], -1, c);
                if (old == c) break;
                if (old == -1) {
                    atomicAdd(count, 1);
                    break;
                }
                h = (h + 1) & (kDictHash - 1);
            }
        }
        __syncthreads();
    }
}

__global__ __launch_bounds__(kSB) void k_dict_count(int ntiles, const int4* tiles, const int* rp, const int* ci,
                                                    int* dlen) {
    __shared__ int table[kDictHash];
    __shared__ int count;
    for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const int k0 = rp[tiles[t].x], m = rp[tiles[t].y] - k0;
        for (int u = threadIdx.x; u < kDictHash; u += kSB) table[u] = -1;
        if (threadIdx.x == 0) count = 0;
        __syncthreads();
        dict_insert(table, &count, ci, k0, m);
        if (threadIdx.x == 0) dlen[t] = count <= kSellDict ? count : kSellDict + 1;
        __syncthreads();
    }
}

// kSlice times the longest row of each tile (rows tiles[t].x .. .y).
__global__ __launch_bounds__(kSB) void k_sell_sizes(int ntiles, const int4* tiles, const int* rp, int* size) {
    __shared__ int longest;
    for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const int4 d = tiles[t];
        if (threadIdx.x == 0) longest = 0;
        __syncthreads();
        const int i = d.x + (int)threadIdx.x;
        if (i < d.y) atomicMax(&longest, rp[i + 1] - rp[i]);
        __syncthreads();
        if (threadIdx.x == 0) size[t] = kSlice * longest;
        __syncthreads();
    }
}

// Each sliced tile from its CSR rows: the rows sorted by length (longest
// first, ties in row order), their entries step by step (padding: column 0,
// value 0), each row's first entry, the dictionary and every entry's position
// in it.
__global__ __launch_bounds__(kSB) void k_sell_fill(int ntiles, const int4* tiles, const int* rp, const int* ci,
                                                   const double* v, uint32_t* slot, int* rowpos, int* ci2, double* v2,
                                                   int* dcol, uint16_t* loc) {
    static_assert(kSlice == kSB, "one thread per row of a tile");
    __shared__ int table[kDictHash];
    __shared__ int uq[kSellDict];
    __shared__ int key[kSlice];
    __shared__ int count;
    for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const int4 d = tiles[2 * t];
        const int total = tiles[2 * t + 1].x, rows = d.y - d.x;
        const int k0 = rp[d.x], m = rp[d.y] - k0;
        const int j = threadIdx.x;
        for (int u = j; u < kDictHash; u += kSB) table[u] = -1;
        if (j == 0) count = 0;
        key[j] = j < rows ? (kSellMaxRow - (rp[d.x + j + 1] - rp[d.x + j])) << 16 | j : INT_MAX;
        __syncthreads();
        lds_bitonic(key, kSlice);
        dict_insert(table, &count, ci, k0, m);
        // compact (any order), then sort: the result does not depend on it
        if (j == 0) count = 0;
        __syncthreads();
        for (int u = j; u < kDictHash; u += kSB)
            if (table[u] >= 0) uq[atomicAdd(&count, 1)] = table[u];
        int P = 1;
        while (P < total) P <<= 1;
        for (int u = total + j; u < P; u += kSB) uq[u] = INT_MAX;
        __syncthreads();
        lds_bitonic(uq, P);
        for (int u = j; u < total; u += kSB) dcol[d.w + u] = uq[u];
        const int steps = kSellMaxRow - (key[0] >> 16);
        const bool own = j < rows;
        const int len = own ? kSellMaxRow - (key[j] >> 16) : 0, i = d.x + (own ? key[j] & 0xffff : 0);
        if (own) {
            slot[d.x + j] = (uint32_t)(i - d.x) | (uint32_t)len << 16;
            rowpos[i] = d.z + j;
        }
        const int r = rp[i];
        for (int k = 0; k < steps; ++k) {
            const size_t o = (size_t)d.z + (size_t)k * kSlice + j;
            int col = 0, b = 0;
            double a = 0.0;
            if (k < len) {
                col = ci[r + k];
                a = v[r + k];
                int e = total;
                while (b < e) {
                    const int h = (b + e) >> 1;
                    if (uq[h] < col) b = h + 1; else e = h;
                }
            }
            ci2[o] = col;
            v2[o] = a;
            loc[o] = (uint16_t)b;
        }
        __syncthreads();
    }
}

// ------------------------------------------------------ aggregate composition

// The pairwise levels composed into one kept level (at most kMaxAggSteps).
struct Chain {
    const int* agg[kMaxAggSteps];
    const double* p[kMaxAggSteps];
    int steps;
};

// Composed aggregate and prolongator entry of every row of a kept level: the
// row's aggregate followed through the chain, p multiplied finest first.
__global__ void k_compose(int n, Chain c, int* cagg, double* cp) {
    GRID_STRIDE(i, n) {
        int I = c.agg[0][i];
        double pc = c.p[0][i];
        for (int m = 1; m < c.steps; ++m) {
            pc = pc * c.p[m][I];
            I = c.agg[m][I];
        }
        cagg[i] = I;
        cp[i] = pc;
    }
}

__global__ void k_count_members(int n, const int* cagg, int* cnt) { GRID_STRIDE(i, n) atomicAdd(&cnt[cagg[i]], 1); }

__global__ void k_fill_members(int n, const int* cagg, const long long* mptr, int* fill, int* mem) {
    GRID_STRIDE(i, n) {
        const int I = cagg[i];
        mem[mptr[I] + atomicAdd(&fill[I], 1)] = (int)i;
    }
}

// Members of each composed aggregate ascending (at most 2^kMaxAggSteps).
__global__ void k_sort_members(int nc, const long long* mptr, int* mem, int* mem_ptr, int* longest) {
    int mx = 0;
    GRID_STRIDE(I, nc) {
        const int b = (int)mptr[I], e = (int)mptr[I + 1];
        for (int q = b + 1; q < e; ++q) {
            const int x = mem[q];
            int u = q;
            while (u > b && mem[u - 1] > x) {
                mem[u] = mem[u - 1];
                --u;
            }
            mem[u] = x;
        }
        mem_ptr[I] = b;
        if (I == nc - 1) mem_ptr[nc] = e;
        mx = max(mx, e - b);
    }
    raise_max(longest, mx);
}

// ------------------------------------------------------------------ driver

// A level in canonical numbering, as the device loop leaves it.
struct CanLevel {
    int n = 0, nc = 0, pairs = 0, maxrow = 0;
    long long nnz = 0;
    int *rp = nullptr, *ci = nullptr;
    double *v = nullptr, *w = nullptr, *dinv = nullptr, *p = nullptr;
    int *agg = nullptr, *mem_ptr = nullptr, *mem = nullptr;
};

int grid_rows(long long n) { return (int)std::min<long long>(std::max<long long>(n, 1), kGridCap); }

enum Coarsened { kCoarsened, kNoPairs, kAsymmetric };

// Matching, aggregates and Galerkin product of level L (canonical); fills the
// next level's matrix and near-null vector.  kNoPairs: the level is left to
// the host; kAsymmetric: the pattern is not symmetric (only the input level
// can be), the whole build is left to the host.
Coarsened coarsen(Temps& T, CanLevel& L, CanLevel& C, const pamg_params& prm, hipStream_t s) {
    const int n = L.n;
    double* diag = T.get<double>(n);
    double* c = T.get<double>(L.nnz);
    int* tr = T.get<int>(L.nnz);
    int* flag = T.get<int>(4);
    HIP_CHECK(hipMemsetAsync(flag, 0, 4 * sizeof(int), s));
    hipLaunchKernelGGL(k_l1diag, dim3(grid_for(n, kSB)), dim3(kSB), 0, s, n, (const int*)L.rp, (const int*)L.ci,
                       (const double*)L.v, L.dinv, diag, flag + 2);
    hipLaunchKernelGGL(k_weights, dim3(grid_for(n, kSB / kWeightLanes)), dim3(kSB), 0, s, n, (const int*)L.rp, (const int*)L.ci,
                       (const double*)L.v, (const double*)diag, (const double*)L.w, c, tr, flag);
    int head[3];
    HIP_CHECK(hipMemcpyAsync(head, flag, 3 * sizeof(int), hipMemcpyDeviceToHost, s));
    HIP_CHECK(hipStreamSynchronize(s));
    T.release(diag);
    T.drain();
    if (head[0]) return kAsymmetric;
    // eligible neighbours in the matching order
    int* adj = T.get<int>(L.nnz);
    int* pos = T.get<int>(L.nnz);
    int* ecnt = T.get<int>(n);
    hipLaunchKernelGGL(k_sort_adj, dim3(grid_rows(n)), dim3(64), 0, s, n, (const int*)L.rp, (const int*)L.ci,
                       (const double*)c, adj, pos, ecnt);
    T.release(c);
    int* mirror = T.get<int>(L.nnz);
    unsigned* best = T.get<unsigned>(n);
    int* mate = T.get<int>(n);
    HIP_CHECK(hipMemsetAsync(best, 0xff, sizeof(unsigned) * n, s));
    hipLaunchKernelGGL(k_mirror, dim3(grid_for(L.nnz, kSB)), dim3(kSB), 0, s, L.nnz, (const int*)pos, (const int*)tr,
                       mirror);
    hipLaunchKernelGGL(k_propose, dim3(grid_for(n, kSB)), dim3(kSB), 0, s, n, (const int*)L.rp, (const int*)ecnt,
                       (const int*)adj, (const int*)mirror, best);
    hipLaunchKernelGGL(k_mates, dim3(grid_for(n, kSB)), dim3(kSB), 0, s, n, (const int*)adj, (const unsigned*)best,
                       mate);
    T.release(adj);
    T.release(pos);
    T.release(tr);
    T.release(mirror);
    T.release(ecnt);
    T.release(best);
    // aggregates
    int* lead = T.get<int>(n);
    int* size = T.get<int>(n);
    hipLaunchKernelGGL(k_leaders, dim3(grid_for(n, kSB)), dim3(kSB), 0, s, n, (const int*)mate, lead, size);
    long long* aid = T.get<long long>((size_t)n + 1);
    long long* msz = T.get<long long>((size_t)n + 1);
    const long long nc = scan<int>(T, n, lead, aid, s);
    scan<int>(T, n, size, msz, s);
    T.release(lead);
    T.release(size);
    L.nc = (int)nc;
    L.pairs = (int)(n - nc);
    // (too little reduction on a level the dense solve can take: coarsest)
    if (L.pairs == 0 || (n <= prm.max_dense && (double)n < prm.min_ratio * (double)nc)) {
        T.release(mate);
        T.release(aid);
        T.release(msz);
        return kNoPairs;
    }
    int* agg = T.get<int>(n);
    L.agg = agg;
    L.p = T.get<double>(n);
    C.w = T.get<double>(nc);
    L.mem_ptr = T.get<int>(nc + 1);
    L.mem = T.get<int>(n);
    hipLaunchKernelGGL(k_aggregate, dim3(grid_for(n, kSB)), dim3(kSB), 0, s, n, (const int*)mate, (const double*)L.w,
                       (const long long*)aid, (const long long*)msz, agg, L.p, C.w, L.mem_ptr, L.mem);
    to_device(L.mem_ptr + nc, &n, 1, s);
    T.release(mate);
    T.release(aid);
    T.release(msz);
    // Galerkin product
    int* ccnt = T.get<int>(nc);
    long long* crp = T.get<long long>((size_t)nc + 1);
    HIP_CHECK(hipMemsetAsync(flag, 0, 4 * sizeof(int), s));
    const int gg = grid_rows(nc);
    hipLaunchKernelGGL(k_galerkin<false>, dim3(gg), dim3(64), 0, s, (int)nc, (const int*)L.mem_ptr,
                       (const int*)L.mem, (const int*)L.rp, (const int*)L.ci, (const double*)L.v, (const int*)agg,
                       (const double*)L.p, ccnt, (const long long*)nullptr, (int*)nullptr, (double*)nullptr, flag);
    const long long cnnz = scan<int>(T, nc, ccnt, crp, s);
    if (cnnz >= (1ll << 31)) throw Error(PAMG_E_OOM, "coarse matrix exceeds 2^31 entries");
    C.n = (int)nc;
    C.nnz = cnnz;
    C.rp = T.get<int>(nc + 1);
    C.ci = T.get<int>(cnnz);
    C.v = T.get<double>(cnnz);
    C.dinv = T.get<double>(nc);
    hipLaunchKernelGGL(k_galerkin<true>, dim3(gg), dim3(64), 0, s, (int)nc, (const int*)L.mem_ptr,
                       (const int*)L.mem, (const int*)L.rp, (const int*)L.ci, (const double*)L.v, (const int*)agg,
                       (const double*)L.p, ccnt, (const long long*)crp, C.ci, C.v, flag);
    hipLaunchKernelGGL(k_to_int, dim3(grid_for(nc + 1, kSB)), dim3(kSB), 0, s, nc + 1, (const long long*)crp, C.rp);
    HIP_CHECK(hipMemcpyAsync(head, flag, 2 * sizeof(int), hipMemcpyDeviceToHost, s));
    HIP_CHECK(hipStreamSynchronize(s));
    if (head[0]) throw Error(PAMG_E_DEVICE, "device Galerkin product: a coarse row exceeds its term capacity");
    C.maxrow = head[1];
    T.release(ccnt);
    T.release(crp);
    T.drain();
    return kCoarsened;
}

// Host copy of a canonical level (matrix and near-null vector).
void download_level(const CanLevel& L, HostLevel& out, hipStream_t s) {
    out.A.n = L.n;
    to_host(out.A.rp, L.rp, (size_t)L.n + 1, s);
    to_host(out.A.ci, L.ci, (size_t)L.nnz, s);
    to_host(out.A.v, L.v, (size_t)L.nnz, s);
    to_host(out.w, L.w, (size_t)L.n, s);
}

}  // namespace

bool device_setup_applies(const pamg_params& prm) {
    return prm.device_setup != 0 && prm.host_only == 0 && prm.agg_steps >= 1 && prm.smooth_prolongator == 0 &&
           (prm.smoother == PAMG_SMOOTHER_L1_JACOBI || prm.smoother == PAMG_SMOOTHER_HYBRID_GS) &&
           prm.match_all_edges == 0;
}

namespace {

// Per row of a level with blocks of nb rows: 1 / a_ii and the range of the
// row's entries whose columns lie in its block (first such entry; the counts
// before and after the row; whether a_ii is stored), as the host schedule.
__global__ void k_gs_rows(int n, int nb, RowIdx R, const int* __restrict__ ci,
                          const double* __restrict__ v, double* __restrict__ ainv, int* __restrict__ fresh,
                          int* __restrict__ bad) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const int b0 = i / nb * nb, b1 = min(n, b0 + nb);
        int first = -1, before = 0, after = 0, diag = 0;
        double a = 0.0;
        const int o = R.start(i), len = R.len(i), st = R.stride();
        for (int k = 0; k < len; ++k) {
            const int j = ci[o + k * st];
            if (j >= b0 && j < b1 && first < 0) first = k;
            if (j >= b0 && j < i) ++before;
            if (j > i && j < b1) ++after;
            if (j == i) {
                if (!(v[o + k * st] > 0.0)) *bad = 1;
                a = 1.0 / v[o + k * st];
                diag = 1;
            }
        }
        ainv[i] = a;
        fresh[2 * (size_t)i] = R.rp[i] + (first < 0 ? 0 : first);
        fresh[2 * (size_t)i + 1] = before | after << 8 | diag << 16;
    }
}

// Per block: each row's depth in the block's forward (earlier rows) and
// backward (later rows) dependency graph, and the block's largest depths.  A
// wave walks its block's rows in order, 64 at a time: their in-block columns
// (fr, from k_gs_rows) are read into LDS together, a lane per row, then a row's
// depths are looked up by a lane per entry.  (One thread walked a block and all
// its rows' entries in memory: 5.8 ms a level whatever its size, more than a level
// of a few thousand rows takes on the host; now 0.21 to 0.53 ms.)
constexpr int kDepthCols = 32;              // in-block columns of a row held in LDS; more are read again
__global__ __launch_bounds__(64) void k_gs_depths(int n, int nb, int nblk, RowIdx R, const int* __restrict__ ci,
                                                  const int2* __restrict__ fr, uint8_t* __restrict__ df,
                                                  uint8_t* __restrict__ db, int* __restrict__ maxd) {
    __shared__ int s_d[256];
    __shared__ uint8_t s_c[64][kDepthCols];
    __shared__ int s_n[64], s_o[64];
    const int lane = threadIdx.x, st = R.stride();
    for (int p = blockIdx.x; p < nblk; p += gridDim.x) {
        const int b0 = p * nb, m = min(n - b0, nb);
        for (int dir = 0; dir < 2; ++dir) {
            int most = 0;
            for (int r0 = 0; r0 < m; r0 += 64) {
                int cnt = 0, o = 0;
                if (r0 + lane < m) {
                    const int i = b0 + (dir ? m - 1 - (r0 + lane) : r0 + lane);
                    const int2 f = fr[i];
                    const int before = f.y & 0xff, after = (f.y >> 8) & 0xff, diag = (f.y >> 16) & 1;
                    cnt = dir ? after : before;
                    o = R.start(i) + (f.x - R.rp[i] + (dir ? before + diag : 0)) * st;
#pragma unroll 8
                    for (int u = 0; u < min(cnt, kDepthCols); ++u) s_c[lane][u] = (uint8_t)(ci[o + u * st] - b0);
                }
                s_n[lane] = cnt;
                s_o[lane] = o;
                __syncthreads();
                for (int w = 0; w < min(64, m - r0); ++w) {
                    const int c = s_n[w];
                    int d = 0;
                    if (lane < min(c, kDepthCols)) d = s_d[s_c[w][lane]] + 1;
                    for (int u = kDepthCols + lane; u < c; u += 64) d = max(d, s_d[ci[s_o[w] + u * st] - b0] + 1);
                    if (c > 0)
                        for (int off = 32; off > 0; off >>= 1) d = max(d, __shfl_xor(d, off));
                    if (lane == 0) s_d[dir ? m - 1 - (r0 + w) : r0 + w] = d;
                    most = max(most, d);
                    __syncthreads();
                }
            }
            uint8_t* out = dir ? db : df;
            for (int t = lane; t < m; t += 64) out[b0 + t] = (uint8_t)s_d[t];
            if (lane == 0) maxd[2 * p + dir] = most;
            __syncthreads();
        }
    }
}

}  // namespace

void device_gs_schedule(pamg_hierarchy* h, DevLevelOut& D, int nb, hipStream_t s) {
    const int n = D.n, nblk = (n + nb - 1) / nb;
    D.gs_nblk = nblk;
    D.gs_ainv = dalloc<double>(h, n, s);
    D.gs_fresh = dalloc<int>(h, 2 * (size_t)n, s);
    D.gs_df = dalloc<uint8_t>(h, n, s);
    D.gs_db = dalloc<uint8_t>(h, n, s);
    D.gs_maxd = dalloc<int>(h, 2 * (size_t)nblk, s);
    Temps T{h->ctx, s, {}, {}};
    int* bad = T.get<int>(1);
    HIP_CHECK(hipMemsetAsync(bad, 0, sizeof(int), s));
    const RowIdx R{D.rp, D.sell.rowpos};
    hipLaunchKernelGGL(k_gs_rows, dim3(grid_for(n, kSB)), dim3(kSB), 0, s, n, nb, R, (const int*)D.ci,
                       (const double*)D.v, D.gs_ainv, D.gs_fresh, bad);
    hipLaunchKernelGGL(k_gs_depths, dim3(grid_rows(nblk)), dim3(64), 0, s, n, nb, nblk, R, (const int*)D.ci,
                       reinterpret_cast<const int2*>(D.gs_fresh), D.gs_df, D.gs_db, D.gs_maxd);
    HIP_CHECK(hipGetLastError());
    if (read1(bad, s)) throw Error(PAMG_E_NOT_SPD, "non-positive diagonal on a coarse level (Gauss-Seidel smoother)");
}

std::unique_ptr<DeviceBuild> device_build(pamg_hierarchy* h, const pamg_csr& A, const pamg_params& prm, int max_coarsest,
                                          hipStream_t s) {
    std::unique_ptr<DeviceBuild> out(new DeviceBuild());
    Temps T{h->ctx, s, {}, {}};
    const int given = std::max({prm.device_min_rows, prm.max_dense, prm.max_coarse});
    const int first = prm.device_min_rows > 0 ? given : std::max(kDeviceMinRows, prm.max_coarse);
    const int rest = prm.device_min_rows > 0 ? given : std::max(kDeviceStopRows, prm.max_coarse);
    auto dev_level = [&](const CanLevel& L, int l) {
        const int limit = l == 0 ? first : rest;
        return L.n > limit && l + 1 < prm.max_levels && L.maxrow <= kRowCap;
    };
    // level 0: the input matrix (its header checked by the caller), w = 1
    std::vector<CanLevel> lev(1);
    {
        CanLevel& L0 = lev[0];
        L0.n = A.n;
        L0.nnz = A.nnz;
        int mx = 0;
        for (int i = 0; i < A.n; ++i) mx = std::max(mx, A.row_ptr[i + 1] - A.row_ptr[i]);
        L0.maxrow = mx;
        if (!dev_level(L0, 0)) return nullptr;   // the host build validates it
        L0.rp = T.get<int>((size_t)A.n + 1);
        L0.ci = T.get<int>(A.nnz);
        L0.v = T.get<double>(A.nnz);
        L0.w = T.get<double>(A.n);
        to_device(L0.rp, A.row_ptr, (size_t)A.n + 1, s);
        to_device(L0.ci, A.col_idx, (size_t)A.nnz, s);
        to_device(L0.v, A.val, (size_t)A.nnz, s);
        // validate_csr's row checks before any kernel follows the columns
        unsigned long long* first = T.get<unsigned long long>(1);
        HIP_CHECK(hipMemsetAsync(first, 0xff, sizeof(unsigned long long), s));
        hipLaunchKernelGGL(k_validate, dim3(grid_for(A.n, kSB)), dim3(kSB), 0, s, A.n, (long long)A.nnz,
                           (const int*)L0.rp, (const int*)L0.ci, (const double*)L0.v, first);
        const unsigned long long f = read1(first, s);
        if (f != ~0ull) throw Error(PAMG_E_INVALID, csr_error((int)(f & 0xff), (int64_t)(f >> 8)));
        if (prm.check_symmetry) {
            int* asym = T.get<int>(1);
            HIP_CHECK(hipMemsetAsync(asym, 0, sizeof(int), s));
            hipLaunchKernelGGL(k_check_symmetry, dim3(grid_for(A.n, kSB)), dim3(kSB), 0, s, A.n,
                               (const int*)L0.rp, (const int*)L0.ci, (const double*)L0.v, asym);
            if (read1(asym, s)) throw Error(PAMG_E_INVALID, "matrix is not bitwise symmetric");
        }
        hipLaunchKernelGGL(k_fill_d, dim3(grid_for(A.n, kSB)), dim3(kSB), 0, s, (long long)A.n, L0.w, 1.0);
    }
    // device (pairwise) levels
    const int steps = std::max(1, prm.agg_steps);
    int built = 0;
    for (;;) {
        CanLevel& L = lev[built];
        L.dinv = T.get<double>(L.n);
        CanLevel C;
        const Coarsened r = coarsen(T, L, C, prm, s);
        if (r == kAsymmetric) return nullptr;
        if (r == kNoPairs) break;          // the host takes this level
        lev.push_back(C);
        ++built;
        if (!dev_level(lev[built], built)) break;
    }
    // the host continues from a kept level (a multiple of the composition
    // step), so that every composed prolongator lies on one side
    const int m = built / steps * steps;
    if (m == 0) return nullptr;
    // host levels from level m
    {
        HostHierarchy& Hs = out->host;
        Hs.lev.emplace_back();
        download_level(lev[m], Hs.lev[0], s);
        pamg_params p2 = prm;
        p2.max_levels = prm.max_levels - m;
        extend_hierarchy(Hs, p2);
        const HostCSR& AL = Hs.lev.back().A;
        if (AL.n > prm.max_dense)
            throw Error(PAMG_E_STALLED, "coarsening stalled at " + std::to_string(AL.n) +
                                            " unknowns, above the dense-solve limit");
        if (AL.n > max_coarsest) return nullptr;
        if (steps > 1) compose_levels(Hs, steps);
        out->host_lay = build_layout(Hs);
    }
    // kept device levels: every steps-th pairwise level below m, with its
    // aggregates and prolongator composed over the steps in between
    const int K = m / steps;
    out->m = K;
    std::vector<int> kp(K), knc(K);
    std::vector<double*> kcp(K);
    std::vector<int*> kmptr(K), kmem(K);
    for (int j = 0; j < K; ++j) {
        const int a = j * steps;
        const CanLevel& L = lev[a];
        kp[j] = a;
        knc[j] = lev[a + steps].n;
        if (steps == 1) {
            kcp[j] = L.p;
            kmptr[j] = L.mem_ptr;
            kmem[j] = L.mem;
            continue;
        }
        Chain ch{};
        ch.steps = steps;
        for (int q = 0; q < steps; ++q) {
            ch.agg[q] = lev[a + q].agg;
            ch.p[q] = lev[a + q].p;
        }
        const int n = L.n, nc = knc[j];
        int* cagg = T.get<int>(n);
        kcp[j] = T.get<double>(n);
        hipLaunchKernelGGL(k_compose, dim3(grid_for(n, kSB)), dim3(kSB), 0, s, n, ch, cagg, kcp[j]);
        int* cnt = T.get<int>(nc);
        HIP_CHECK(hipMemsetAsync(cnt, 0, sizeof(int) * nc, s));
        hipLaunchKernelGGL(k_count_members, dim3(grid_for(n, kSB)), dim3(kSB), 0, s, n, (const int*)cagg, cnt);
        long long* mptr = T.get<long long>((size_t)nc + 1);
        scan<int>(T, nc, cnt, mptr, s);
        HIP_CHECK(hipMemsetAsync(cnt, 0, sizeof(int) * nc, s));
        kmem[j] = T.get<int>(n);
        kmptr[j] = T.get<int>((size_t)nc + 1);
        hipLaunchKernelGGL(k_fill_members, dim3(grid_for(n, kSB)), dim3(kSB), 0, s, n, (const int*)cagg,
                           (const long long*)mptr, cnt, kmem[j]);
        int* longest = T.get<int>(1);
        HIP_CHECK(hipMemsetAsync(longest, 0, sizeof(int), s));
        hipLaunchKernelGGL(k_sort_members, dim3(grid_for(nc, kSB)), dim3(kSB), 0, s, nc, (const long long*)mptr,
                           kmem[j], kmptr[j], longest);
        if (read1(longest, s) > (1 << kMaxAggSteps)) throw Error(PAMG_E_DEVICE, "composed aggregate too large");
        T.release(cnt);
        T.release(mptr);
        T.release(cagg);
    }
    // canonical levels a .. b-1 have been laid out (or downloaded)
    auto drop_levels = [&](int a, int b) {
        for (int l = a; l < b; ++l) {
            const CanLevel& L = lev[l];
            void* const all[] = {L.rp, L.ci, L.v, L.w, L.dinv, L.p, L.agg, L.mem_ptr, L.mem};
            for (void* p : all)
                if (p) T.release(p);
        }
    };
    drop_levels(m, (int)lev.size());
    // device layouts of the kept levels K-1 .. 0 (their arrays belong to the hierarchy)
    out->dev.resize(K);
    const int* cip = nullptr;   // hierarchical -> canonical of the coarser level
    std::vector<int> cip_host;
    int* cip_dev = nullptr;
    cip_host = out->host_lay[0].iperm;
    cip_dev = T.get<int>(cip_host.size());
    to_device(cip_dev, cip_host.data(), cip_host.size(), s);
    cip = cip_dev;
    for (int j = K - 1; j >= 0; --j) {
        const CanLevel& L = lev[kp[j]];
        DevLevelOut& D = out->dev[j];
        const int n = L.n, nc = knc[j];
        const int* mem_ptr = kmptr[j];
        const int* mem = kmem[j];
        D.n = n;
        D.nc = nc;
        D.nnz = L.nnz;
        D.pairs = L.pairs;
        int* sz = T.get<int>(nc);
        long long* ap = T.get<long long>((size_t)nc + 1);
        hipLaunchKernelGGL(k_agg_sizes, dim3(grid_for(nc, kSB)), dim3(kSB), 0, s, nc, cip, mem_ptr, sz);
        scan<int>(T, nc, sz, ap, s);
        D.aggptr = dalloc<int>(h, (size_t)nc + 1, s);
        D.iperm = dalloc<int>(h, n, s);
        D.perm = dalloc<int>(h, n, s);
        hipLaunchKernelGGL(k_place, dim3(grid_for(nc, kSB)), dim3(kSB), 0, s, nc, n, cip, mem_ptr, mem,
                           (const long long*)ap, D.aggptr, D.iperm, D.perm);
        T.release(sz);
        T.release(ap);
        int* len = T.get<int>(n);
        long long* rp2 = T.get<long long>((size_t)n + 1);
        hipLaunchKernelGGL(k_row_len, dim3(grid_for(n, kSB)), dim3(kSB), 0, s, n, (const int*)D.iperm,
                           (const int*)L.rp, len);
        scan<int>(T, n, len, rp2, s);
        T.release(len);
        // the permuted CSR: the level's own arrays, or the source of its sliced rows
        bool sell = sell_applies(n, L.nnz, L.maxrow);
        D.rp = dalloc<int>(h, (size_t)n + 1, s);
        D.dinv = dalloc<double>(h, n, s);
        D.p = dalloc<double>(h, n, s);
        int* ci2 = sell ? T.get<int>(L.nnz) : dalloc<int>(h, L.nnz, s);
        double* v2 = sell ? T.get<double>(L.nnz) : dalloc<double>(h, L.nnz, s);
        hipLaunchKernelGGL(k_reorder, dim3(grid_rows(n)), dim3(64), 0, s, n, (const int*)D.iperm,
                           (const int*)D.perm, (const int*)L.rp, (const int*)L.ci, (const double*)L.v,
                           (const double*)L.dinv, (const double*)kcp[j], (const long long*)rp2, ci2, v2, D.dinv, D.p);
        hipLaunchKernelGGL(k_to_int, dim3(grid_for(n + 1, kSB)), dim3(kSB), 0, s, (long long)n + 1,
                           (const long long*)rp2, D.rp);
        T.release(rp2);
        std::vector<int32_t> rp_h, ap_h;
        to_host(rp_h, D.rp, (size_t)n + 1, s);
        to_host(ap_h, D.aggptr, (size_t)nc + 1, s);
        T.drain();
        for (int32_t c = 0; c < nc; ++c) D.max_agg = std::max(D.max_agg, ap_h[c + 1] - ap_h[c]);
        D.nent = L.nnz;
        if (sell) {
            // tiles (host partition of the aggregates), halved until every
            // dictionary fits, while they store no more than sell_fits allows
            std::vector<int32_t> tiles = sell_tiles(ap_h, n, nc), dlen, size;
            for (;;) {
                const int nt = (int)(tiles.size() / 4);
                int4* td = T.get<int4>(nt);
                int* dl = T.get<int>(nt);
                int* sz2 = T.get<int>(nt);
                to_device(reinterpret_cast<int*>(td), tiles.data(), tiles.size(), s);
                hipLaunchKernelGGL(k_sell_sizes, dim3(grid_rows(nt)), dim3(kSB), 0, s, nt, (const int4*)td,
                                   (const int*)D.rp, sz2);
                to_host(size, sz2, (size_t)nt, s);
                sell = sell_fits(std::accumulate(size.begin(), size.end(), 0ll), L.nnz);
                if (sell) {
                    hipLaunchKernelGGL(k_dict_count, dim3(grid_rows(nt)), dim3(kSB), 0, s, nt, (const int4*)td,
                                       (const int*)D.rp, (const int*)ci2, dl);
                    to_host(dlen, dl, (size_t)nt, s);
                }
                T.release(td);
                T.release(dl);
                T.release(sz2);
                if (!sell || !split_sell_tiles(tiles, ap_h, nc, dlen)) break;
            }
            T.drain();
            if (sell) {
                DevSell& S = D.sell;
                const int nt = (int)dlen.size();
                std::vector<int32_t> full(8 * (size_t)nt, 0);
                long long at = 0;
                for (int t = 0; t < nt; ++t) {
                    const int32_t* q = &tiles[4 * (size_t)t];
                    const int32_t d[8] = {q[0], q[1], (int32_t)at, (int32_t)S.len, dlen[t], q[2], q[3], 0};
                    std::copy(d, d + 8, full.begin() + 8 * (size_t)t);
                    S.max_len = std::max(S.max_len, dlen[t]);
                    S.len += dlen[t];
                    at += size[t];
                }
                S.n_tiles = nt;
                D.nent = at;
                sell_shares(full, 8, n, S.xcd);
                S.tiles = dalloc<int>(h, full.size(), s);
                to_device(S.tiles, full.data(), full.size(), s);
                S.slot = dalloc<uint32_t>(h, n, s);
                S.rowpos = dalloc<int>(h, n, s);
                S.col = dalloc<int>(h, S.len, s);
                S.loc = dalloc<uint16_t>(h, at, s);
                D.ci = dalloc<int>(h, at, s);
                D.v = dalloc<double>(h, at, s);
                hipLaunchKernelGGL(k_sell_fill, dim3(grid_rows(nt)), dim3(kSB), 0, s, nt, (const int4*)S.tiles,
                                   (const int*)D.rp, (const int*)ci2, (const double*)v2, S.slot, S.rowpos, D.ci, D.v,
                                   S.col, S.loc);
                T.release_now(ci2, v2);
            } else {
                T.keep(h, ci2);
                T.keep(h, v2);
            }
        }
        if (!sell) {
            D.ci = ci2;
            D.v = v2;
        }
        D.vd = dalloc<double>(h, D.nent, s);
        hipLaunchKernelGGL(k_vd, dim3(grid_for(D.nent, kSB)), dim3(kSB), 0, s, D.nent, (const int*)D.ci,
                           (const double*)D.v, (const double*)D.dinv, D.vd);
        D.items = first_tile_items(L.nnz);
        if (sell) {
            cip = D.iperm;
            drop_levels(kp[j], kp[j] + steps);
            continue;
        }
        // tiles (host partition of the row pointer) and dictionaries
        int items = first_tile_items(L.nnz);
        std::vector<int32_t> up, down;
        int* dl_up = nullptr;
        int* dl_down = nullptr;
        int* flag = T.get<int>(2);
        int max_up = 0, max_down = 0;
        for (;;) {
            const int cap = items * kBlock;
            make_tiles(rp_h, ap_h, n, nc, cap, up, down);
            D.items = items;
            if (items < kDictItems) break;
            int4* tu = T.get<int4>(up.size() / 4);
            int4* td = T.get<int4>(down.size() / 4);
            to_device(reinterpret_cast<int*>(tu), up.data(), up.size(), s);
            to_device(reinterpret_cast<int*>(td), down.data(), down.size(), s);
            dl_up = T.get<int>(up.size() / 4);
            dl_down = T.get<int>(down.size() / 4);
            HIP_CHECK(hipMemsetAsync(flag, 0, 2 * sizeof(int), s));
            const int nu = (int)(up.size() / 4), nd = (int)(down.size() / 4);
            // the dictionaries hold permuted columns
            hipLaunchKernelGGL(k_dict<false>, dim3(grid_rows(nu)), dim3(kSB), 0, s, nu, (const int4*)tu,
                               (const int*)D.ci, cap, dl_up, (const long long*)nullptr, (int*)nullptr,
                               (uint16_t*)nullptr, flag);
            hipLaunchKernelGGL(k_dict<false>, dim3(grid_rows(nd)), dim3(kSB), 0, s, nd, (const int4*)td,
                               (const int*)D.ci, cap, dl_down, (const long long*)nullptr, (int*)nullptr,
                               (uint16_t*)nullptr, flag + 1);
            int mx[2];
            HIP_CHECK(hipMemcpyAsync(mx, flag, 2 * sizeof(int), hipMemcpyDeviceToHost, s));
            HIP_CHECK(hipStreamSynchronize(s));
            max_up = mx[0];
            max_down = mx[1];
            if (items == kDictItems || std::max(max_up, max_down) <= kDictMaxLarge) {
                // fill the dictionaries
                auto fill = [&](int nt, const int4* tt, int* dl, int maxl, DevDict& dd) {
                    long long* off = T.get<long long>((size_t)nt + 1);
                    const long long tot = scan<int>(T, nt, dl, off, s);
                    if (tot >= (1ll << 31)) throw Error(PAMG_E_OOM, "tile dictionaries exceed 2^31 entries");
                    dd.col = dalloc<int>(h, tot, s);
                    dd.loc = dalloc<uint16_t>(h, L.nnz, s);
                    dd.span = dalloc<int>(h, 2 * (size_t)nt, s);
                    HIP_CHECK(hipMemsetAsync(dd.loc, 0, sizeof(uint16_t) * L.nnz, s));
                    hipLaunchKernelGGL(k_dict<true>, dim3(grid_rows(nt)), dim3(kSB), 0, s, nt, tt,
                                       (const int*)D.ci, cap, dl, (const long long*)off, dd.col, dd.loc, flag);
                    hipLaunchKernelGGL(k_spans, dim3(grid_for(nt, kSB)), dim3(kSB), 0, s, nt, (const long long*)off,
                                       (const int*)dl, dd.span);
                    dd.len = tot;
                    dd.max_len = maxl;
                    T.release(off);
                };
                fill(nu, tu, dl_up, max_up, D.up_dict);
                fill(nd, td, dl_down, max_down, D.down_dict);
                HIP_CHECK(hipStreamSynchronize(s));
                break;
            }
            items /= 2;
        }
        D.up_tiles = dalloc<int>(h, up.size(), s);
        to_device(D.up_tiles, up.data(), up.size(), s);
        D.n_up = (int)(up.size() / 4);
        D.down_tiles = dalloc<int>(h, down.size(), s);
        to_device(D.down_tiles, down.data(), down.size(), s);
        D.n_down = (int)(down.size() / 4);
        cip = D.iperm;
        drop_levels(kp[j], kp[j] + steps);
    }
    HIP_CHECK(hipStreamSynchronize(s));
    return out;
}

}  // namespace pamg
