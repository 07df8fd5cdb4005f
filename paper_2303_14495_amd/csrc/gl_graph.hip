// Symmetric kNN graph with local-scaling weights from kNN lists (the
// clustering graph of Section 2.2): union of the lists, Gaussian weights with
// the bandwidth product s_i s_j, CSR out.
//
// Row i of the result is its own list and the rows that list it.  By rows: the
// reverse entries are counted, the rows' places scanned, and both kinds dealt to
// their rows; a wavefront then sorts its row (about 2k entries) by column, drops
// second occurrences and zero weights, and the kept ones move to their final
// places.  Every entry is written three times; the one sort of all (row, column)
// keys with their values moves each entry once per 8 bits of its key (5 times at
// 262 144 points) and needs 88 bytes of temporaries per list entry, and the sort's
// own, against 32.  What bounds it now is mapping those and
// the two host round trips.  Whole calls on lists of 10: 20 000 points 395 us
// sorted and 218 by rows, 100 000: 835 and 289, 262 144: 1097 and 668.
#include <hip/hip_runtime.h>
#include <hipcub/hipcub.hpp>

#include <algorithm>
#include <cmath>
#include <string>

#include "gl_internal.hpp"

namespace {

constexpr int kLongBlock = 1024;
constexpr int kRun = 4096;  // keys sorted in LDS (32 KB: two workgroups of 16 waves fill a CU)

constexpr int kCountTile = 1024;  // slots of the count's hash, and entries of a workgroup;
// four times the entries from kCountLong on, where that still fills the chip: a hub's
// additions are a quarter (262 144 lists of 10 with a hub: 1.24 -> 1.13 ms), and without
// one the count takes as long (100 us)
constexpr int64_t kCountLong = 1 << 21;
// Lists of up to kRowsK go by rows (60 000 points, sorted / by rows: lists of 4 347 /
// 272 us, 16 776 / 314, 24 863 / 313); beyond, most rows have more than a
// wavefront's 64 entries and a workgroup each costs more than the sort (lists of
// 100: 1719 and 3718 us).
constexpr int32_t kRowsK = 24;
constexpr int64_t kMaxGrid = 1 << 20;  // workgroups of the kernels with lanes per row: a launch holds < 2^32 threads

constexpr double kScaleFloor = 0x1p-256;  // s_i of a point whose scale neighbour is at distance 0

enum : int32_t { KG_BAD_INDEX = 1, KG_BAD_DIST = 2, KG_ISOLATED = 4 };

__device__ __forceinline__ double kg_scale(const float* d2, int64_t node, int32_t k, int32_t rank) {
    const double s = sqrt((double)d2[node * k + rank - 1]);
    return s > 0.0 ? s : kScaleFloor;
}

__global__ __launch_bounds__(256) void kg_init_kernel(int64_t n, int32_t k, int32_t* __restrict__ len) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) len[i] = k;
}

// len[j] += 1 for every list that holds j (len starts at k); defects flagged.
// Additions to one address are served one every 12 ns (3.2 ms for a point in
// 262 143 lists), so a workgroup first adds up its `span` entries in LDS: one slot
// per hash, the first point that takes it; others add straight to memory.
__global__ __launch_bounds__(256) void kg_count_kernel(int64_t n, int32_t k, int32_t span, const int32_t* __restrict__ idx,
                                                       const float* __restrict__ d2, int32_t* __restrict__ len,
                                                       int32_t* flags) {
    __shared__ int32_t owner[kCountTile], times[kCountTile];
    for (int u = threadIdx.x; u < kCountTile; u += 256) {
        owner[u] = -1;
        times[u] = 0;
    }
    __syncthreads();
    const int64_t t0 = (int64_t)blockIdx.x * span, t1 = min(t0 + span, n * k);
    for (int64_t t = t0 + threadIdx.x; t < t1; t += 256) {
        const int32_t j = idx[t];
        const bool ok = j >= 0 && j < n && j != t / k;
        const float dv = d2[t];
        int32_t f = ok ? 0 : (int32_t)KG_BAD_INDEX;
        if (!(dv >= 0.0f) || !(dv <= 3.4028234663852886e38f)) f |= KG_BAD_DIST;
        if (f) atomicOr(flags, f);
        if (!ok) continue;
        const int h = j & (kCountTile - 1);
        const int32_t was = atomicCAS(&owner[h], -1, j);
        if (was == -1 || was == j) atomicAdd(&times[h], 1);
        else atomicAdd(&len[j], 1);
    }
    __syncthreads();
    for (int u = threadIdx.x; u < kCountTile; u += 256)
        if (times[u]) atomicAdd(&len[owner[u]], times[u]);
}

// Longest row, and the rows of more than 64 entries: shape[0] and [1], the latter
// listed in long_rows.
__global__ __launch_bounds__(256) void kg_shape_kernel(int64_t n, const int32_t* __restrict__ len,
                                                       int32_t* __restrict__ long_rows, int32_t* shape) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int v = i < n ? len[i] : 0;
    const unsigned long long m = __ballot(v > 64);
    if (m == 0) return;
    const int lane = threadIdx.x & 63;
    int at = 0;
    if (lane == 0) at = atomicAdd(shape + 1, __popcll(m));
    at = __builtin_amdgcn_readfirstlane(at) + __popcll(m & ((1ull << lane) - 1ull));
    if (v > 64) {
        long_rows[at] = (int32_t)i;
        atomicMax(shape, v);
    }
}

// Key (column << 32 | t) of both orientations of entry t into their rows' places
// off[row] ..: the row's own entries first, the reverse ones behind them in any
// order (left[row] counts down; the sort makes the order irrelevant).
__global__ __launch_bounds__(256) void kg_deal_kernel(int64_t n, int32_t k, const int32_t* __restrict__ idx,
                                                      const int32_t* __restrict__ off, int32_t* __restrict__ left,
                                                      unsigned long long* __restrict__ keys) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= n * k) return;
    const int64_t i = t / k, j = idx[t];
    keys[off[i] + (t - i * k)] = ((unsigned long long)j << 32) | (unsigned long long)t;
    keys[off[j] + atomicSub(&left[j], 1) - 1] = ((unsigned long long)i << 32) | (unsigned long long)t;
}

__device__ __forceinline__ double kg_weight(unsigned long long key, double si, int32_t k, int32_t rank,
                                            const float* __restrict__ d2) {
    const int64_t j = (int64_t)(key >> 32);
    return exp(-(double)d2[key & 0xffffffffull] / (si * kg_scale(d2, j, k, rank)));
}

// One wavefront per row of up to 64 entries: rank of every key by counting, the
// keys moved to sorted order, first occurrences with a weight > 0 kept and
// packed at the row's place.  When an edge is in both lists the smaller t, the
// lower row's entry, comes first.
__global__ __launch_bounds__(256) void kg_row_kernel(int64_t n, int32_t k, int32_t rank_s, int64_t m2,
                                                     const int32_t* __restrict__ off,
                                                     const float* __restrict__ d2,
                                                     unsigned long long* __restrict__ keys, double* __restrict__ wts,
                                                     int32_t* __restrict__ kept, int32_t* flags) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    for (int64_t i = (int64_t)blockIdx.x * 4 + wave; i < n; i += (int64_t)gridDim.x * 4) {
        const int64_t o = off[i], e = i + 1 < n ? (int64_t)off[i + 1] : m2;
        const int len = (int)(e - o);
        if (len > 64) continue;
        const unsigned long long key = lane < len ? keys[o + lane] : ~0ull;
        int rank = 0;
        for (int u = 0; u < len; ++u) {
            const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)key, u);
            const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(key >> 32), u);
            const unsigned long long other = ((unsigned long long)hi << 32) | lo;
            rank += other < key ? 1 : 0;
        }
        const int to = lane < len ? rank : lane;  // a permutation: the keys of a row are distinct
        const unsigned lo = (unsigned)__builtin_amdgcn_ds_permute(4 * to, (int)(unsigned)key);
        const unsigned hi = (unsigned)__builtin_amdgcn_ds_permute(4 * to, (int)(unsigned)(key >> 32));
        const unsigned long long mine = ((unsigned long long)hi << 32) | lo;
        const unsigned before = (unsigned)__shfl_up((int)hi, 1, 64);
        double w = 0.0;
        if (lane < len && (lane == 0 || before != hi)) w = kg_weight(mine, kg_scale(d2, i, k, rank_s), k, rank_s, d2);
        const unsigned long long m = __ballot(w > 0.0);
        if (w > 0.0) {
            const int at = __popcll(m & ((1ull << lane) - 1ull));
            keys[o + at] = mine;
            wts[o + at] = w;
        }
        if (lane == 0) {
            kept[i] = __popcll(m);
            if (m == 0) atomicOr(flags, (int32_t)KG_ISOLATED);
        }
    }
}

// Ascending sort of len <= kRun keys in LDS by the whole workgroup: bitonic merges
// whose first step mirrors, so that every exchange is ascending and keys beyond
// len need not exist.
__device__ __forceinline__ void kg_sort(unsigned long long (&a)[kRun], int len) {
    for (int size = 2; size < 2 * len; size <<= 1) {
        for (int step = size >> 1; step > 0; step >>= 1) {
            const int flip = step == size >> 1 ? size - 1 : step;
            for (int u = threadIdx.x; u < len; u += kLongBlock) {
                const int v = u ^ flip;
                if (v > u && v < len && a[v] < a[u]) {
                    const unsigned long long x = a[u];
                    a[u] = a[v];
                    a[v] = x;
                }
            }
            __syncthreads();
        }
    }
}

// The same for the listed rows of up to kRun entries, a workgroup each.
__global__ __launch_bounds__(kLongBlock) void kg_long_kernel(int64_t n, int32_t k, int32_t rank_s, int64_t m2,
                                                             const int32_t* __restrict__ off,
                                                             const float* __restrict__ d2,
                                                             unsigned long long* __restrict__ keys,
                                                             double* __restrict__ wts, int32_t* __restrict__ kept,
                                                             const int32_t* __restrict__ long_rows, int32_t rows,
                                                             int32_t* flags) {
    __shared__ unsigned long long sh[kRun];
    __shared__ int wave_n[kLongBlock / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int r = blockIdx.x; r < rows; r += gridDim.x) {
        const int64_t i = long_rows[r];
        const int64_t o = off[i], e = i + 1 < n ? (int64_t)off[i + 1] : m2;
        const int len = (int)(e - o);
        __syncthreads();
        for (int u = threadIdx.x; u < len; u += kLongBlock) sh[u] = keys[o + u];
        __syncthreads();
        kg_sort(sh, len);
        const double si = kg_scale(d2, i, k, rank_s);
        int base = 0;
        for (int c = 0; c < len; c += kLongBlock) {
            const int u = c + (int)threadIdx.x;
            const unsigned long long key = u < len ? sh[u] : ~0ull;
            double w = 0.0;
            if (u < len && (u == 0 || (sh[u - 1] >> 32) != (key >> 32))) w = kg_weight(key, si, k, rank_s, d2);
            const unsigned long long m = __ballot(w > 0.0);
            if (lane == 0) wave_n[wave] = __popcll(m);
            __syncthreads();
            int at = base + __popcll(m & ((1ull << lane) - 1ull));
            for (int v = 0; v < kLongBlock / 64; ++v) {
                if (v < wave) at += wave_n[v];
                base += wave_n[v];
            }
            if (w > 0.0) {
                keys[o + at] = key;
                wts[o + at] = w;
            }
            __syncthreads();
        }
        if (threadIdx.x == 0) {
            kept[i] = base;
            if (base == 0) atomicOr(flags, (int32_t)KG_ISOLATED);
        }
    }
}

// The rows' kept entries to their final places (16 lanes per row); row_ptr[i] for
// i <= n, the number of entries to *total.
__global__ __launch_bounds__(256) void kg_write_kernel(int64_t n, const int32_t* __restrict__ off,
                                                       const int32_t* __restrict__ kept,
                                                       const int32_t* __restrict__ place,
                                                       const unsigned long long* __restrict__ keys,
                                                       const double* __restrict__ wts, int64_t* __restrict__ row_ptr,
                                                       int32_t* __restrict__ col, double* __restrict__ weight,
                                                       int32_t* __restrict__ total) {
    const int q = threadIdx.x % 16;
    for (int64_t i = (int64_t)blockIdx.x * 16 + threadIdx.x / 16; i < n; i += (int64_t)gridDim.x * 16) {
        const int64_t o = off[i], p = place[i];
        const int m = kept[i];
        if (q == 0) {
            row_ptr[i] = p;
            if (i == n - 1) {
                row_ptr[n] = p + m;
                *total = (int32_t)(p + m);
            }
        }
        for (int u = q; u < m; u += 16) {
            col[p + u] = (int32_t)(keys[o + u] >> 32);
            weight[p + u] = wts[o + u];
        }
    }
}

// Sorted path.  Both orientations of every list entry t = i * k + e: key (row << bits |
// col), value t (the entry whose distance gives the weight; below 2^30).  bits: of n - 1,
// so that the sort has no passes over bits that are 0 in every key (60 000 points:
// 4 passes of 8 bits instead of 6 with the row in the upper word).
__global__ void kg_emit_kernel(int64_t n, int32_t k, int32_t bits, const int32_t* __restrict__ idx,
                               const float* __restrict__ d2, unsigned long long* __restrict__ keys,
                               uint32_t* __restrict__ vals, int32_t* flags) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n * k) return;
    const int64_t i = t / k;
    const int64_t j = idx[t];
    const float dv = d2[t];
    int32_t f = 0;
    if (j < 0 || j >= n || j == i) f |= KG_BAD_INDEX;
    if (!(dv >= 0.0f) || !(dv <= 3.4028234663852886e38f)) f |= KG_BAD_DIST;
    if (f) {
        atomicOr(flags, f);
        keys[2 * t] = keys[2 * t + 1] = 0ull;  // keeps the sort defined; the call fails
    } else {
        keys[2 * t] = ((unsigned long long)i << bits) | (unsigned long long)j;
        keys[2 * t + 1] = ((unsigned long long)j << bits) | (unsigned long long)i;
    }
    vals[2 * t] = vals[2 * t + 1] = (uint32_t)t;
}

// keep[p] = 1 for the first occurrence of a key whose weight is > 0;
// wts[p] = that weight.
__global__ void kg_weight_kernel(int64_t m2, int32_t k, int32_t rank, int32_t bits,
                                 const unsigned long long* __restrict__ keys, const uint32_t* __restrict__ vals, const float* __restrict__ d2,
                                 int32_t* __restrict__ keep, double* __restrict__ wts) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= m2) return;
    const unsigned long long key = keys[p];
    int32_t kp = 0;
    double w = 0.0;
    if (p == 0 || keys[p - 1] != key) {
        const int64_t i = (int64_t)(key >> bits), j = (int64_t)(key & ((1ull << bits) - 1ull));
        w = exp(-(double)d2[vals[p]] / (kg_scale(d2, i, k, rank) * kg_scale(d2, j, k, rank)));
        kp = w > 0.0 ? 1 : 0;
    }
    keep[p] = kp;
    wts[p] = w;
}

__global__ void kg_scatter_kernel(int64_t m2, int32_t bits, const unsigned long long* __restrict__ keys,
                                  const int32_t* __restrict__ keep, const int32_t* __restrict__ pos,
                                  const double* __restrict__ wts, int32_t* __restrict__ col,
                                  double* __restrict__ weight, int32_t* __restrict__ rows) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= m2 || !keep[p]) return;
    const int64_t q = pos[p];
    col[q] = (int32_t)(keys[p] & ((1ull << bits) - 1ull));
    rows[q] = (int32_t)(keys[p] >> bits);
    weight[q] = wts[p];
}

// row_ptr[i] = first kept entry of row >= i (rows sorted); isolated rows flagged.
__global__ void kg_rowptr_kernel(int64_t n, int64_t nnz, const int32_t* __restrict__ rows,
                                 int64_t* __restrict__ row_ptr, int32_t* flags) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i > n) return;
    int64_t lo = 0, hi = nnz;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (rows[mid] < i) lo = mid + 1; else hi = mid;
    }
    row_ptr[i] = lo;
    if (i < n) {
        const bool has = lo < nnz && rows[lo] == i;
        if (!has) atomicOr(flags, (int32_t)KG_ISOLATED);
    }
}

gl_status kfail(gl_status st, const std::string& m) {
    gl::set_last_error(m);
    return st;
}

gl_status kdefect(int32_t flags) {
    if (flags & KG_BAD_INDEX) return kfail(GL_E_INVALID_ARG, "a neighbour index is out of [0, n) or the point itself");
    if (flags & KG_BAD_DIST) return kfail(GL_E_INVALID_ARG, "a squared distance is negative or not finite");
    return kfail(GL_E_BAD_GRAPH, "a point has no edge of positive weight (isolated)");
}

gl_status kdone(hipError_t e) {
    return e == hipSuccess ? GL_OK : kfail(GL_E_HIP, std::string("kNN graph: ") + hipGetErrorString(e));
}

size_t al(size_t b) { return (b + 255) & ~(size_t)255; }

// Defects of the lists, the rows' lengths (len) and the rows of more than 64 entries
// (long_rows), found before anything is allocated: the two arrays and the four words
// behind them lie in the caller's weight array, which has room for 16 n k bytes.
// The graph is made row by row unless one is longer than kRun (a hub of 262 143
// entries sorted by one workgroup: 11 ms, the sort of all keys 1.1), or more than
// one in 16 has over 64 entries.
struct RowShape {
    int32_t *len, *long_rows;
    int32_t longest, n_long;
    bool rows_fit(int64_t n) const { return longest <= kRun && (int64_t)n_long * 16 <= n; }
};

gl_status row_shape(int64_t n, int32_t k, const int32_t* idx, const float* d2, double* weight, RowShape& r,
                    hipStream_t s) {
    const int64_t m = n * k;
    r.len = (int32_t*)weight;
    r.long_rows = r.len + n;
    int32_t* words = r.long_rows + n;  // defects, longest row, long rows
    const unsigned g_n = (unsigned)((n + 255) / 256);
    int32_t host[3] = {0, 0, 0};
    hipError_t e = hipMemsetAsync(words, 0, sizeof(host), s);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(kg_init_kernel, dim3(g_n), dim3(256), 0, s, n, k, r.len);
        const int32_t span = m < kCountLong ? kCountTile : 4 * kCountTile;
        hipLaunchKernelGGL(kg_count_kernel, dim3((unsigned)((m + span - 1) / span)), dim3(256), 0, s, n, k, span, idx, d2,
                           r.len, words);
        hipLaunchKernelGGL(kg_shape_kernel, dim3(g_n), dim3(256), 0, s, n, (const int32_t*)r.len, r.long_rows,
                           words + 1);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipMemcpyAsync(host, words, sizeof(host), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return kdone(e);
    r.longest = host[1];
    r.n_long = host[2];
    return host[0] ? kdefect(host[0]) : GL_OK;
}

// The graph row by row.
gl_status by_rows(int64_t n, int32_t k, const int32_t* idx, const float* d2, int32_t scale_rank, const RowShape& shape,
                  int64_t* row_ptr, int32_t* col, double* weight, int64_t& count, hipStream_t s) {
    const int64_t m = n * k, m2 = 2 * m;
    size_t scan_bytes = 0;
    hipError_t e = hipcub::DeviceScan::ExclusiveSum(nullptr, scan_bytes, (const int32_t*)nullptr, (int32_t*)nullptr,
                                                    (int)n, s);
    if (e != hipSuccess) return kfail(GL_E_HIP, std::string("temporary size query: ") + hipGetErrorString(e));
    const size_t b_keys = al((size_t)m2 * 8), b_w = al((size_t)m2 * 8), b_n = al((size_t)n * 4);
    const size_t total = b_keys + b_w + 3 * b_n + 256 + al(scan_bytes);
    char* base = nullptr;
    if (hipMallocAsync((void**)&base, total, s) != hipSuccess) {
        (void)hipGetLastError();
        return kfail(GL_E_NOMEM, "temporary device memory for the kNN graph");
    }
    char* q = base;
    auto take = [&](size_t b) { char* r = q; q += b; return r; };
    unsigned long long* keys = (unsigned long long*)take(b_keys);
    double* wts = (double*)take(b_w);
    int32_t* off = (int32_t*)take(b_n);
    int32_t* kept = (int32_t*)take(b_n);
    int32_t* place = (int32_t*)take(b_n);
    int32_t* flags = (int32_t*)take(256);  // defects, entries
    void* scan_tmp = take(al(scan_bytes));

    const unsigned g_m = (unsigned)((m + 255) / 256);
    int32_t host[2] = {0, 0};
    gl_status st = GL_OK;
    e = hipMemsetAsync(flags, 0, sizeof(host), s);
    if (e == hipSuccess) e = hipcub::DeviceScan::ExclusiveSum(scan_tmp, scan_bytes, shape.len, off, (int)n, s);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(kg_deal_kernel, dim3(g_m), dim3(256), 0, s, n, k, idx, (const int32_t*)off, shape.len, keys);
        hipLaunchKernelGGL(kg_row_kernel, dim3((unsigned)std::min<int64_t>((n + 3) / 4, kMaxGrid)), dim3(256), 0, s, n,
                           k, scale_rank, m2, (const int32_t*)off, d2, keys, wts, kept, flags);
        if (shape.n_long > 0)
            hipLaunchKernelGGL(kg_long_kernel, dim3((unsigned)std::min(shape.n_long, 512)), dim3(kLongBlock), 0, s, n,
                               k, scale_rank, m2, (const int32_t*)off, d2, keys, wts, kept,
                               (const int32_t*)shape.long_rows, shape.n_long, flags);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipcub::DeviceScan::ExclusiveSum(scan_tmp, scan_bytes, kept, place, (int)n, s);
    if (e == hipSuccess) {  // overwrites shape's arrays
        hipLaunchKernelGGL(kg_write_kernel, dim3((unsigned)std::min<int64_t>((n + 15) / 16, kMaxGrid)), dim3(256), 0, s,
                           n, (const int32_t*)off, (const int32_t*)kept, (const int32_t*)place,
                           (const unsigned long long*)keys, (const double*)wts, row_ptr, col, weight, flags + 1);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipMemcpyAsync(host, flags, sizeof(host), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e == hipSuccess && host[0]) st = kdefect(host[0]);
    count = host[1];
    const hipError_t ef = hipFreeAsync(base, s);
    const hipError_t es = hipStreamSynchronize(s);
    if (st != GL_OK) return st;
    return kdone(e != hipSuccess ? e : (ef != hipSuccess ? ef : es));
}

// The graph from one sort of all (row, column) keys; checked: the lists have no defects.
gl_status by_sort(int64_t n, int32_t k, const int32_t* idx, const float* d2, int32_t scale_rank, bool checked,
                  int64_t* row_ptr, int32_t* col, double* weight, int64_t& count, hipStream_t s) {
    const int64_t m = n * k, m2 = 2 * m;
    // temporaries: keys (2 buffers), values (2), keep, positions, weights, rows, flags, sort storage
    int bits = 1;
    while ((n - 1) >> bits) ++bits;
    const int nbits = 2 * bits;
    size_t sort_bytes = 0;
    hipcub::DoubleBuffer<unsigned long long> kb(nullptr, nullptr);
    hipcub::DoubleBuffer<uint32_t> vb(nullptr, nullptr);
    if (hipcub::DeviceRadixSort::SortPairs(nullptr, sort_bytes, kb, vb, (int)0, 0, nbits, s) != hipSuccess)
        return kfail(GL_E_HIP, "radix sort size query failed");
    hipError_t e = hipcub::DeviceRadixSort::SortPairs(nullptr, sort_bytes, kb, vb, (int)m2, 0, nbits, s);
    size_t scan_bytes = 0;
    if (e == hipSuccess)
        e = hipcub::DeviceScan::ExclusiveSum(nullptr, scan_bytes, (const int32_t*)nullptr, (int32_t*)nullptr,
                                             (int)m2, s);
    if (e != hipSuccess) return kfail(GL_E_HIP, std::string("temporary size query: ") + hipGetErrorString(e));
    const size_t b_keys = al((size_t)m2 * 8), b_vals = al((size_t)m2 * 4), b_i32 = al((size_t)m2 * 4),
                 b_w = al((size_t)m2 * 8);
    const size_t total = 2 * b_keys + 2 * b_vals + 3 * b_i32 + b_w + 256 + al(sort_bytes) + al(scan_bytes);
    char* base = nullptr;
    if (hipMallocAsync((void**)&base, total, s) != hipSuccess) {
        (void)hipGetLastError();
        return kfail(GL_E_NOMEM, "temporary device memory for the kNN graph");
    }
    char* q = base;
    auto take = [&](size_t b) { char* r = q; q += b; return r; };
    unsigned long long* k0 = (unsigned long long*)take(b_keys);
    unsigned long long* k1 = (unsigned long long*)take(b_keys);
    uint32_t* v0 = (uint32_t*)take(b_vals);
    uint32_t* v1 = (uint32_t*)take(b_vals);
    int32_t* keep = (int32_t*)take(b_i32);
    int32_t* pos = (int32_t*)take(b_i32);
    int32_t* rows = (int32_t*)take(b_i32);
    double* wts = (double*)take(b_w);
    int32_t* flags = (int32_t*)take(256);
    void* sort_tmp = take(al(sort_bytes));
    void* scan_tmp = take(al(scan_bytes));

    const unsigned g_m = (unsigned)((m + 255) / 256), g_m2 = (unsigned)((m2 + 255) / 256);
    int32_t hflags = 0, hlast[2] = {0, 0};
    e = hipMemsetAsync(flags, 0, 4, s);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(kg_emit_kernel, dim3(g_m), dim3(256), 0, s, n, k, bits, idx, d2, k0, v0, flags);
        e = hipGetLastError();
    }
    if (e == hipSuccess && !checked) {
        e = hipMemcpyAsync(&hflags, flags, 4, hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
    }
    gl_status st = GL_OK;
    if (e == hipSuccess && hflags) st = kdefect(hflags);
    if (e == hipSuccess && st == GL_OK) {
        hipcub::DoubleBuffer<unsigned long long> keys(k0, k1);
        hipcub::DoubleBuffer<uint32_t> vals(v0, v1);
        e = hipcub::DeviceRadixSort::SortPairs(sort_tmp, sort_bytes, keys, vals, (int)m2, 0, nbits, s);
        const unsigned long long* ks = keys.Current();
        const uint32_t* vs = vals.Current();
        if (e == hipSuccess) {
            hipLaunchKernelGGL(kg_weight_kernel, dim3(g_m2), dim3(256), 0, s, m2, k, scale_rank, bits, ks, vs, d2, keep,
                               wts);
            e = hipGetLastError();
        }
        if (e == hipSuccess) e = hipcub::DeviceScan::ExclusiveSum(scan_tmp, scan_bytes, keep, pos, (int)m2, s);
        if (e == hipSuccess) e = hipMemcpyAsync(&hlast[0], pos + (m2 - 1), 4, hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipMemcpyAsync(&hlast[1], keep + (m2 - 1), 4, hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        count = (int64_t)hlast[0] + hlast[1];
        if (e == hipSuccess) {
            hipLaunchKernelGGL(kg_scatter_kernel, dim3(g_m2), dim3(256), 0, s, m2, bits, ks, keep, pos, wts, col, weight,
                               rows);
            e = hipGetLastError();
        }
        if (e == hipSuccess) {
            hipLaunchKernelGGL(kg_rowptr_kernel, dim3((unsigned)((n + 1 + 255) / 256)), dim3(256), 0, s, n, count,
                               rows, row_ptr, flags);
            e = hipGetLastError();
        }
        if (e == hipSuccess) e = hipMemcpyAsync(&hflags, flags, 4, hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e == hipSuccess && (hflags & KG_ISOLATED))
            st = kdefect(hflags);
    }
    const hipError_t ef = hipFreeAsync(base, s);
    const hipError_t es = hipStreamSynchronize(s);
    if (st != GL_OK) return st;
    return kdone(e != hipSuccess ? e : (ef != hipSuccess ? ef : es));
}

}  // namespace

extern "C" gl_status gl_knn_graph(int64_t n, int32_t k, const int32_t* idx, const float* d2, int32_t scale_rank,
                                  int64_t* row_ptr, int32_t* col, double* weight, int64_t capacity, int64_t* nnz,
                                  void* stream) {
    if (!idx || !d2 || !row_ptr || !col || !weight || !nnz)
        return kfail(GL_E_INVALID_ARG, "arrays and nnz must not be NULL");
    if (n < 2 || n >= ((int64_t)1 << 31)) return kfail(GL_E_INVALID_ARG, "n must lie in [2, 2^31)");
    if (k < 1 || (int64_t)k >= n || k > 1024) return kfail(GL_E_INVALID_ARG, "k must lie in [1, min(n - 1, 1024)]");
    if (scale_rank < 1 || scale_rank > k) return kfail(GL_E_INVALID_ARG, "scale_rank must lie in [1, k]");
    const int64_t m = n * k, m2 = 2 * m;
    if (capacity < m2) return kfail(GL_E_INVALID_ARG, "capacity must be >= 2 n k");
    hipStream_t s = (hipStream_t)stream;
    if (m2 > (int64_t)INT32_MAX) return kfail(GL_E_INVALID_ARG, "2 n k must be < 2^31");
    int64_t count = 0;
    gl_status st = GL_OK;
    RowShape shape = {};
    const bool checked = k <= kRowsK;
    if (checked) st = row_shape(n, k, idx, d2, weight, shape, s);
    if (st == GL_OK) {
        if (checked && shape.rows_fit(n))
            st = by_rows(n, k, idx, d2, scale_rank, shape, row_ptr, col, weight, count, s);
        else
            st = by_sort(n, k, idx, d2, scale_rank, checked, row_ptr, col, weight, count, s);
    }
    if (st == GL_OK) *nnz = count;
    return st;
}
