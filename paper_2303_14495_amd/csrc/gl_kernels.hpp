// Kernels of the gfx950 preconditioned-DCA library and their launch helpers.
#pragma once

#include "gl_device.hpp"
#include "gl_fold.hpp"

namespace gl {

constexpr int kBlock = 256;  // 4 wavefronts of 64 lanes

// Per-launch geometry shared by the row kernels: block b (after the XCD remap)
// owns rows [b * rows_per_block, (b + 1) * rows_per_block), processed as `tiles`
// passes of 256 / G rows.
struct RowGeom {
    int64_t n;
    int64_t rows_per_block;
    int32_t G;
    int32_t log2G;
    int32_t tiles;
    int32_t remap;
};

template <typename A> struct SweepCoef {
    A eps, c, eta;          // model parameters
    A inv_eps;              // 1 / eps
    A half_eps, quarter_inv_eps, half_eta;  // energy prefactors
    A ginv0, ginv1;         // 1 / g for unlabelled (Lambda = 0) and labelled rows (L_s)
    A alpha, kappa;         // r = alpha (u^t - v) + kappa (b - T v)
    A ga, gd, gl;           // unnormalized L: g_i = ga + gd d_i + gl Lambda_i
};

template <typename TW, typename TU, typename OffT> struct SweepArgs {
    typedef typename acc_of<TU>::type A;
    const OffT* rp;
    const int32_t* col;
    const TW* w;
    const TU* ut;      // u^t, read on the own row for b
    const TU* vin;     // v^s, gathered
    TU* vout;          // v^{s+1}; nullptr for the energy-only pass
    const int32_t* labels;
    const int32_t* order;  // node of each row position, or nullptr (identity)
    const A* dd;       // diagonal d_i of L = D - W, or nullptr for L_s (diagonal 1)
    A* partials;       // [2K][grid] block partial sums, or nullptr
    RowGeom g;
    int32_t energy;    // also accumulate the energy terms (vin == ut)
    SweepCoef<A> k;
    const int32_t* heavy;  // direct layout: rows longer than 16 G, summed by workgroups of their own
    int32_t nheavy;        // number of heavy rows
    int32_t hblocks;       // their workgroups (nheavy rounded up to a multiple of 8), first in the launch
};

// Fixed-order double reduction of one statistic per block: block s sums
// partials[s * nb .. s * nb + nb).
template <typename P>
__device__ __forceinline__ double block_sum(const P* __restrict__ src, int64_t nb) {
    __shared__ double sh[kBlock / 64];
    double acc = 0.0;
    for (int64_t i = threadIdx.x; i < nb; i += kBlock) acc += (double)src[i];
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = acc;
    __syncthreads();
    return ((sh[0] + sh[1]) + sh[2]) + sh[3];
}

// Solve statistics of up to kStatGroup sweeps, reduced by one launch: set j
// (block column j) holds the 2K statistics of one sweep at partials + j *
// stride; block s < K sums energy column s into energy_dst[j][s] (nullptr:
// none), block K + k the |r|^2 of column k into res_dst[j][k], each in the
// fixed order of block_sum.  A non-finite sum sets *flag to 1.
constexpr int kStatGroup = 16;
struct StatGroup {
    double* energy_dst[kStatGroup];
    double* res_dst[kStatGroup];
};

template <typename P>
__global__ __launch_bounds__(kBlock) void finalize_group_kernel(const P* partials, int64_t nb, int64_t stride,
                                                                int32_t K, StatGroup g, double* flag) {
    const int s = blockIdx.x, j = blockIdx.y;
    double* dst = s < K ? g.energy_dst[j] : g.res_dst[j];
    if (dst == nullptr) return;  // uniform per block
    const double v = block_sum(partials + (int64_t)j * stride + (int64_t)s * nb, nb);
    if (threadIdx.x == 0) {
        dst[s < K ? s : s - K] = v;
        if (!(fabs(v) <= 1.7976931348623157e308)) *flag = 1.0;
    }
}

// Power method: scale_out = 1 / sqrt(sum partial[scale_stat]); sums_out gets both
// sums in double, and sums_out[2] 0 with `first`, 1 once the one of scale_stat is
// below 2^-90 or no number.
static __global__ __launch_bounds__(kBlock) void power_finalize_kernel(const float* partials, int64_t nb,
                                                                int32_t scale_stat, int32_t first, float* scale_out,
                                                                double* sums_out) {
    const double s0 = block_sum(partials, nb);
    __syncthreads();
    const double s1 = block_sum(partials + nb, nb);
    if (threadIdx.x == 0) {
        const double norm2 = scale_stat ? s1 : s0;
        *scale_out = (float)(1.0 / sqrt(norm2));
        sums_out[0] = s0;
        sums_out[1] = s1;
        if (first) sums_out[2] = 0.0;
        else if (!(norm2 >= 0x1p-90)) sums_out[2] = 1.0;
    }
}

static __global__ void fill_double_kernel(double* p, int64_t n, double v) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

static __global__ void copy_bytes_kernel(const u32x4* __restrict__ src, u32x4* __restrict__ dst, int64_t n16,
                                  const uint8_t* __restrict__ src_tail, uint8_t* __restrict__ dst_tail,
                                  int32_t tail) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n16) dst[i] = src[i];
    if (i < tail) dst_tail[i] = src_tail[i];
}

// Move whole rows between node order and position order:
//   gather  (scatter = 0): dst[p] = src[order[p]]
//   scatter (scatter = 1): dst[order[p]] = src[p]
// Rows are `words` units of W (a row of K field values).
template <typename W>
__global__ void permute_rows_kernel(int64_t n, int32_t words, const int32_t* __restrict__ order,
                                    const W* __restrict__ src, W* __restrict__ dst, int32_t scatter) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n * words) return;
    const int64_t p = i / words, j = i - p * words;
    const int64_t o = (int64_t)order[p] * words + j;
    if (scatter)
        dst[o] = src[i];
    else
        dst[i] = src[o];
}

// Bandwidth ceilings (measurement helpers).  Each thread moves four 16-byte
// vectors per step (non-temporal, grid-stride); the read-only kernel folds
// what it reads into a value it stores only if it matches `never`, so the
// loads cannot be dropped and nothing is written in practice.
static __global__ __launch_bounds__(256) void stream_read_kernel(const u32x4* __restrict__ src, int64_t n16,
                                                                 uint32_t never, u32x4* __restrict__ sink) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    u32x4 acc = {0u, 0u, 0u, 0u};
    for (; i + 3 * stride < n16; i += 4 * stride) {
        const u32x4 a = __builtin_nontemporal_load(src + i);
        const u32x4 b = __builtin_nontemporal_load(src + i + stride);
        const u32x4 c = __builtin_nontemporal_load(src + i + 2 * stride);
        const u32x4 d = __builtin_nontemporal_load(src + i + 3 * stride);
        acc ^= (a ^ b) ^ (c ^ d);
    }
    for (; i < n16; i += stride) acc ^= __builtin_nontemporal_load(src + i);
    if ((acc.x ^ acc.y ^ acc.z ^ acc.w) == never) sink[0] = acc;
}

static __global__ __launch_bounds__(256) void stream_copy_kernel(const u32x4* __restrict__ src,
                                                                 u32x4* __restrict__ dst, int64_t n16) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (; i + 3 * stride < n16; i += 4 * stride) {
        const u32x4 a = __builtin_nontemporal_load(src + i);
        const u32x4 b = __builtin_nontemporal_load(src + i + stride);
        const u32x4 c = __builtin_nontemporal_load(src + i + 2 * stride);
        const u32x4 d = __builtin_nontemporal_load(src + i + 3 * stride);
        __builtin_nontemporal_store(a, dst + i);
        __builtin_nontemporal_store(b, dst + i + stride);
        __builtin_nontemporal_store(c, dst + i + 2 * stride);
        __builtin_nontemporal_store(d, dst + i + 3 * stride);
    }
    for (; i < n16; i += stride) __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
}

template <typename TU>
__global__ void labels_kernel(int64_t n, int32_t K, const TU* __restrict__ U, int32_t* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    typedef typename acc_of<TU>::type A;
    if (K == 1) {
        out[i] = cvt<A>(U[i]) >= (A)0 ? 1 : 0;
        return;
    }
    A best = cvt<A>(U[i * K]);
    int32_t arg = 0;
    for (int k = 1; k < K; ++k) {
        const A v = cvt<A>(U[i * K + k]);
        if (v > best) {
            best = v;
            arg = k;
        }
    }
    out[i] = arg;
}

// ---------------------------------------------------------------------------
// operator construction (once per graph)
// ---------------------------------------------------------------------------
enum : int32_t {
    BAD_ROWPTR = 1,
    BAD_COL_RANGE = 2,
    BAD_COL_ORDER = 4,
    BAD_SELF_LOOP = 8,
    BAD_WEIGHT = 16,
    BAD_ASYMMETRIC = 32,
    BAD_DEGREE = 64
};

constexpr int kRowLanes = 16;  // lanes per row of the construction kernels

template <typename T, typename OP> __device__ __forceinline__ T row_reduce(T v, OP op) {
#pragma unroll
    for (int off = kRowLanes / 2; off > 0; off >>= 1) v = op(v, __shfl_xor(v, off, kRowLanes));
    return v;
}

// What the construction finds out about a graph (zeroed, the firsts all ones).
struct GraphCheck {
    int32_t flags;         // defects of the structure or the weights
    int32_t degree_flags;  // BAD_DEGREE (meaningful when flags == 0)
    unsigned long long first, first_degree;  // first rows with them
    int32_t heavy;         // rows longer than heavy_min
    int32_t pad;
};

// The defects of row i among its entries before `stop` (the row ends at the
// first column out of range, which is a defect itself), for one of the row's
// kRowLanes lanes; *range: that lane's first column out of range.
template <typename TIN>
__device__ __forceinline__ int32_t check_entries(int64_t i, int64_t n, int64_t nnz, const int64_t* __restrict__ rp,
                                                 const int32_t* __restrict__ col, const TIN* __restrict__ w,
                                                 int64_t beg, int64_t stop, int q, int64_t& range, double& sum) {
    int32_t f = 0;
    for (int64_t p = beg + q; p < stop; p += kRowLanes) {
        const int64_t j = col[p];
        if (j < 0 || j >= n) {
            f |= BAD_COL_RANGE;
            range = p;
            break;
        }
        if (p > beg && j <= (int64_t)col[p - 1]) f |= BAD_COL_ORDER;
        if (j == i) f |= BAD_SELF_LOOP;
        const TIN wp = w[p];
        const double wv = (double)wp;
        if (!(wv > 0.0) || !(wv <= 1.7976931348623157e308)) f |= BAD_WEIGHT;
        sum += wv;
        // symmetry: find i in row j by binary search and compare the weight bits
        const int64_t jb = rp[j], je = rp[j + 1];
        if (jb < 0 || je < jb || je > nnz) {
            f |= BAD_ROWPTR;
            continue;
        }
        int64_t lo = jb, hi = je;
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if (col[mid] < i) lo = mid + 1; else hi = mid;
        }
        if (lo >= je || col[lo] != i || !(w[lo] == wp)) f |= BAD_ASYMMETRIC;
    }
    return f;
}

// Checks of the CSR graph and its degrees d_i = sum of row i's weights (double,
// every kRowLanes-th entry in turn, then a butterfly).  kRowLanes lanes per row:
// a lane per row walked its 20-odd entries alone, a dependent chain of about
// five loads each, and the degrees were a second pass (535 + 59 us for the 5.4 M
// entries of a 453 x 601 image's graph, 129 us so; 327 + 24 us and 195 us for the
// 4 M of 262 144 points' kNN graph).
template <typename TIN>
__global__ __launch_bounds__(256) void validate_kernel(int64_t n, int64_t nnz, const int64_t* __restrict__ rp,
                                                       const int32_t* __restrict__ col, const TIN* __restrict__ w,
                                                       int64_t heavy_min, double* __restrict__ d,
                                                       GraphCheck* __restrict__ check) {
    const int64_t i = (folded(blockIdx.x, blockIdx.y, gridDim.x) * 256 + threadIdx.x) / kRowLanes;
    const int q = threadIdx.x % kRowLanes;
    if (i >= n) return;  // whole groups
    const int64_t beg = rp[i], end = rp[i + 1];
    int32_t f = 0;
    double s = 0.0;
    if (beg < 0 || end < beg || end > nnz) {
        f = BAD_ROWPTR;
    } else {
        int64_t range = INT64_MAX;
        f = check_entries(i, n, nnz, rp, col, w, beg, end, q, range, s);
        const int64_t stop = row_reduce(range, [](int64_t a, int64_t b) { return a < b ? a : b; });
        if (stop != INT64_MAX) {
            s = 0.0;
            f = check_entries(i, n, nnz, rp, col, w, beg, stop, q, range, s) | BAD_COL_RANGE;
        }
        f = row_reduce(f, [](int32_t a, int32_t b) { return a | b; });
        s = row_reduce(s, [](double a, double b) { return a + b; });
        if (q == 0 && end - beg > heavy_min) atomicAdd(&check->heavy, 1);
    }
    if (q != 0) return;
    d[i] = s;
    if (f) {
        atomicOr(&check->flags, f);
        atomicMin(&check->first, (unsigned long long)i);
    } else if (!(s > 0.0) || !(s <= 1.7976931348623157e308)) {
        atomicOr(&check->degree_flags, (int32_t)BAD_DEGREE);
        atomicMin(&check->first_degree, (unsigned long long)i);
    }
}

// what_ij = w_ij / (sqrt(d_i) sqrt(d_j)) in double, rounded once to TOUT; the index
// arrays are copied (row offsets narrowed to OffT) in the same pass.
// raw != 0 (unnormalized L = D - W): w_ij itself, rounded once to TOUT.
// kRowLanes lanes per row, so that the arrays are read and written in runs (4 M
// entries to bf16: 190 us with a lane per row, 35 us so).
template <typename TIN, typename TOUT, typename OffT>
__global__ __launch_bounds__(256) void normalize_kernel(int64_t n, const int64_t* __restrict__ rp,
                                                        const int32_t* __restrict__ col, const TIN* __restrict__ w,
                                                        const double* __restrict__ d, OffT* __restrict__ rp_out,
                                                        int32_t* __restrict__ col_out, TOUT* __restrict__ w_out,
                                                        int32_t raw) {
    const int64_t i = (folded(blockIdx.x, blockIdx.y, gridDim.x) * 256 + threadIdx.x) / kRowLanes;
    const int q = threadIdx.x % kRowLanes;
    if (i > n) return;
    const int64_t beg = rp[i];
    if (q == 0) rp_out[i] = (OffT)beg;
    if (i == n) return;
    const int64_t end = rp[i + 1];
    const double ri = raw ? 1.0 : sqrt(d[i]);
    for (int64_t p = beg + q; p < end; p += kRowLanes) {
        const int32_t j = col[p];
        col_out[p] = j;
        w_out[p] = store_as<TOUT>::from(raw ? (double)w[p] : (double)w[p] / (ri * sqrt(d[j])));
    }
}

// Workgroups of 256 threads for `rows` rows of kRowLanes lanes (from 2^28 rows on, more
// threads than one dimension of a launch holds).
inline dim3 row_grid(int64_t rows) {
    const Fold f = fold_blocks((rows * kRowLanes + 255) / 256);
    return dim3(f.x, f.y);
}

// Diagonal of the unnormalized operator as stored: dd_p = sum of the row's
// stored (rounded) weights, summed in double in storage order, rounded to A.
// Keeps L 1 = 0 for the weights the sweeps actually use.
template <typename TW, typename OffT, typename A>
__global__ void rowsum_kernel(int64_t n, const OffT* __restrict__ rp, const TW* __restrict__ w,
                              A* __restrict__ dd) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double s = 0.0;
    for (int64_t p = rp[i]; p < rp[i + 1]; ++p) s += cvt<double>(w[p]);
    dd[i] = (A)s;
}

// Largest entry of a diagonal as the bits of a non-negative double (monotone
// as unsigned) in out[0], and out[1] != 0 where an entry is not positive and finite.
template <typename A>
__global__ __launch_bounds__(256) void diagonal_kernel(int64_t n, const A* __restrict__ dd, unsigned long long* out) {
    double m = 0.0;
    bool bad = false;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const double v = (double)dd[i];
        if (!(v > 0.0) || !(v <= 1.7976931348623157e308)) bad = true;
        else m = v > m ? v : m;
    }
    for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off, 64));
    const bool any = __ballot(bad) != 0;
    if ((threadIdx.x & 63) == 0) {
        atomicMax(out, (unsigned long long)__double_as_longlong(m));
        if (any) atomicMax(out + 1, 1ull);
    }
}

}  // namespace gl
