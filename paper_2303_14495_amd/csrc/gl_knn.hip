// Exact k-nearest-neighbour search in R^d, the step that builds a clustering
// graph before the method runs (Section 2.2 uses the k nearest neighbours in
// Euclidean distance of the feature vectors; Section 6 names a parallel kNN as
// the missing piece for clustering).
//
// The result is fixed: distances are sum_c (q_c - p_c)^2 accumulated in f32
// with FMA in coordinate order, ties go to the lower index.  For d <= 64 it is
// found in two ways.
//
// Few points (or a stream under capture): every query over all points, no temporary
// memory, by knn_scan_kernel, a wavefront per query or per four, or, when the queries
// are enough to fill the chip so, by knn_block_kernel, a thread per query.
//
// Otherwise the n^2 distances are first formed approximately on the matrix
// cores, but to nearly f32 accuracy: the centred points are scaled by a power
// of two and split into two f16 parts, x = hi + lo, and <q, p> = hi hi + hi lo
// + lo hi, and |p|^2 / 2 with it, is one chain of v_mfma_f32_32x32x16_f16 over
// 3 d + 2 products (knn_tile_kernel).  Per 1024 pairs that is one or two matrix
// instructions (d <= 4, d <= 10) instead of 2 d + 2 vector instructions per
// pair and lane, and the vector work left is one minimum and one compare per
// 16 pairs.  Each lane keeps the T > k smallest approximate values of its
// query; knn_refine_kernel forms the exact distances of those candidates,
// takes the k best and proves from the error bound that no other point can
// enter or tie; queries without that proof (ties at the k-th place, mostly: whole
// numbers, copies) are scanned by the same two kernels, starting from the k-th
// distance that their candidates gave.
// Nothing of size n x n is ever formed, and no step waits for the host.
//
// Measured (k = 15, one vector-ALU kernel with a thread per query before): n =
// 120 011, d = 10: 21.2 -> 2.0 ms; n = 60 000, d = 64, k = 10: 27.7 -> 2.2 ms; n =
// 300, d = 10, k = 10: 239 -> 25 us.  The tile kernel takes 9 of 10 parts of it, about
// 300 cycles per SIMD and 1024 pairs where its matrix instructions take 64: bound
// by the vector work on what passes the thresholds.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <string>

#include "gl_internal.hpp"
#include "gl_device.hpp"
#include "gl_fold.hpp"

namespace gl {
namespace {

typedef _Float16 kn_h8 __attribute__((ext_vector_type(8)));
typedef float kn_f16v __attribute__((ext_vector_type(16)));
typedef float kn_f4 __attribute__((ext_vector_type(4)));

constexpr int kKnnMaxD = 64;
// n (d + 10) up to which every query is scanned: below it the tile path's six
// launches and list fills cost more than the scan's n^2 d operations (d = 10:
// n = 2000 63 us scanned and about 150 in tiles, 4000 173 and 184, 8000 431 and
// 236; d = 27: n = 4000 284 and 206).
constexpr int64_t kKnnScanMax = 4096 * 20;
// The points are cut into segments, with lists of their own, while that leaves
// at most this many wavefronts (two per SIMD): every further segment starts its
// lists empty again, and those first values are most of what a list ever takes
// (60 000 points, d = 10, k = 15: 0.86 ms with at most 2048, 0.90 with 4096).
constexpr int64_t kKnnWaves = 2048;
constexpr int kStatBlocks = 256;

// What the approximate path derives from the points (one block on the device).
struct KnnFrame {
    float mu[kKnnMaxD];  // column means
    float scale;         // power of two: largest centred coordinate in [2^11, 2^12)
    float inv2;          // 2 / scale^2
    float sub;           // |error| of a vector from coordinates below the normal f16 range
    int32_t bad;         // the split cannot be used: every query is scanned
};

// Column sums (double), minima and maxima over block b's rows: lane t reads
// column t % d of consecutive rows, so that loads are contiguous.
__global__ __launch_bounds__(256) void knn_stats_kernel(const float* __restrict__ x, int64_t n, int32_t d,
                                                        double* __restrict__ psum, float* __restrict__ pmin,
                                                        float* __restrict__ pmax) {
    __shared__ double ss[256];
    __shared__ float sn[256], sx[256];
    const int64_t b = blockIdx.x;
    const int64_t e0 = n * b / kStatBlocks * d, e1 = n * (b + 1) / kStatBlocks * d;
    const int step = 256 / d * d, t = threadIdx.x;
    double s = 0.0;
    float mn = INFINITY, mx = -INFINITY;
    if (t < step)
#pragma unroll 4
        for (int64_t e = e0 + t; e < e1; e += step) {
            const float v = x[e];
            s += (double)v;
            mn = fminf(mn, v);
            mx = fmaxf(mx, v);
        }
    ss[t] = s;
    sn[t] = mn;
    sx[t] = mx;
    __syncthreads();
    if (t < d) {
        for (int u = t + d; u < step; u += d) {
            s += ss[u];
            mn = fminf(mn, sn[u]);
            mx = fmaxf(mx, sx[u]);
        }
        psum[b * kKnnMaxD + t] = s;
        pmin[b * kKnnMaxD + t] = mn;
        pmax[b * kKnnMaxD + t] = mx;
    }
}

// The frame from the partials, and the failure counter's zero.  A NaN or an
// infinity anywhere makes a column sum non-finite.
__global__ __launch_bounds__(256) void knn_frame_kernel(const double* __restrict__ psum,
                                                        const float* __restrict__ pmin,
                                                        const float* __restrict__ pmax, int64_t n, int32_t d,
                                                        KnnFrame* __restrict__ f, unsigned int* fail_count) {
    __shared__ double ss[256];
    __shared__ float sn[256], sx[256];
    const int t = threadIdx.x, c = t & 63, part = t >> 6;
    double s = 0.0;
    float mn = INFINITY, mx = -INFINITY;
    if (c < d)
#pragma unroll 8
        for (int b = part * (kStatBlocks / 4); b < (part + 1) * (kStatBlocks / 4); ++b) {
            s += psum[b * kKnnMaxD + c];
            mn = fminf(mn, pmin[b * kKnnMaxD + c]);
            mx = fmaxf(mx, pmax[b * kKnnMaxD + c]);
        }
    ss[t] = s;
    sn[t] = mn;
    sx[t] = mx;
    __syncthreads();
    if (t >= 64) return;
    s = ((ss[c] + ss[c + 64]) + ss[c + 128]) + ss[c + 192];
    mn = fminf(fminf(sn[c], sn[c + 64]), fminf(sn[c + 128], sn[c + 192]));
    mx = fmaxf(fmaxf(sx[c], sx[c + 64]), fmaxf(sx[c + 128], sx[c + 192]));
    const float mu = c < d ? (float)(s / (double)n) : 0.0f;
    const bool finite = c >= d || fabs(s) <= 1.7976931348623157e308;
    float am = c < d ? fmaxf(mx - mu, mu - mn) : 0.0f;
    for (int off = 32; off > 0; off >>= 1) am = fmaxf(am, __shfl_xor(am, off, 64));
    const bool bad = __ballot(!finite) != 0 || !(am >= 0x1p-40f && am <= 0x1p40f);
    f->mu[c] = mu;
    if (c == 0) {
        const int ex = bad ? 0 : 11 - ilogbf(am);
        f->scale = ldexpf(1.0f, ex);
        f->inv2 = ldexpf(1.0f, 1 - 2 * ex);
        f->sub = ldexpf(sqrtf((float)d), -13 - ex);
        f->bad = bad ? 1 : 0;
        *fail_count = 0u;
    }
}

// hi and lo of a centred, scaled coordinate.
__device__ __forceinline__ void knn_split(float v, _Float16& hi, _Float16& lo) {
    hi = (_Float16)v;
    lo = (_Float16)(v - (float)hi);
}

// Points as MFMA A fragments: tile t of 32 points, k-step ks, lane l holds row
// l % 32, factors 16 ks + 8 (l / 32) .. + 7 of the 3 d + 2 products: hi, lo, hi
// of every coordinate in turn, then |p|^2 / 2 as 2^15 (hi + 2^-11 lo), zeros
// behind; a wavefront's fragment is one contiguous KiB.  The rows that fill the
// last tile get the largest |p|^2 / 2 there is.  half_norm: |p|^2 / 2 in scaled
// units.
template <int KS>
__global__ __launch_bounds__(256) void knn_pack_kernel(const float* __restrict__ x, int64_t n, int64_t np, int32_t d,
                                                       const KnnFrame* __restrict__ f, kn_h8* __restrict__ frag,
                                                       float* __restrict__ half_norm) {
    const int64_t e = folded(blockIdx.x, blockIdx.y, gridDim.x) * 256 + threadIdx.x;
    if (e >= np * 2 * KS) return;
    const int64_t tile = e / (64 * KS);
    const int rest = (int)(e - tile * (64 * KS));
    const int ks = rest >> 6, lane = rest & 63;
    const int64_t p = tile * 32 + (lane & 31);
    const float scale = f->scale;
    float hn = 0.0f;
    if (p < n)
        for (int c = 0; c < d; ++c) {
            const float w = (x[p * d + c] - f->mu[c]) * scale;
            hn = fmaf(w, w, hn);
        }
    hn *= 0.5f;
    kn_h8 v;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int k = 16 * ks + 8 * (lane >> 5) + i;
        _Float16 r = (_Float16)0.0f;
        if (k < 3 * d) {
            if (p < n) {
                const int sec = k / d, c = k - sec * d;
                _Float16 hi, lo;
                knn_split((x[p * d + c] - f->mu[c]) * scale, hi, lo);
                r = sec == 1 ? lo : hi;
            }
        } else if (k < 3 * d + 2) {
            const float s = hn * 0x1p-15f;
            const _Float16 hi = s < 0x1p-14f ? (_Float16)0.0f : (_Float16)s;
            r = k == 3 * d ? hi : (_Float16)((s - (float)hi) * 0x1p11f);
            if (p >= n) r = k == 3 * d ? (_Float16)65504.0f : (_Float16)0.0f;
        }
        v[i] = r;
    }
    frag[e] = v;
    if (ks == 0 && lane < 32) half_norm[p] = hn;
}

constexpr int kBuf = 20;        // buffered values per lane and query (a tile adds at most 16)
constexpr int kTileWaves = 4;   // wavefronts per workgroup

// Wavefront w of workgroup (qb, seg) works for a tile of 32 queries against the
// point tiles of segment seg: lane l sees, of every point tile, the 16 points
// 8 (r / 4) + 4 (l / 32) + r % 4 (the rows of its MFMA results) for query l % 32
// of its tile; |p|^2 / 2 - <q, p> arrive in 16 registers, no LDS in between.
// A value below the query's threshold goes to the lane's buffer in LDS; when
// some lane's buffer could overflow, every lane sorts its buffer into its list
// of the T smallest values, and the threshold becomes the T-th smallest of the
// two lists of the query (lanes l and l + 32).  Appending costs a few
// instructions for the lanes concerned; sorting runs with all lanes busy.
// Rejected values are >= the threshold of their time, hence >= the final one.
template <int KS, int T>
__global__ __launch_bounds__(64 * kTileWaves) void knn_tile_kernel(
    const float* __restrict__ x, int64_t n, int32_t d, const KnnFrame* __restrict__ f,
    const kn_h8* __restrict__ frag, int32_t tiles, int32_t segs, float* __restrict__ bound,
    int32_t* __restrict__ cand) {
    __shared__ float2 buf[kTileWaves][kBuf][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int half = lane >> 5, col = lane & 31;
    const int64_t block = folded(blockIdx.x, blockIdx.y, gridDim.x);
    const int qb = (int)(block / segs), seg = (int)(block - (int64_t)qb * segs);
    const int64_t qt64 = (int64_t)qb * kTileWaves + wave;
    if (qt64 >= tiles || f->bad) return;
    const int qt = (int)qt64;
    const int64_t q = (int64_t)qt * 32 + col;
    const int t0 = (int)((int64_t)tiles * seg / segs), t1 = (int)((int64_t)tiles * (seg + 1) / segs);

    // the query's B fragments: -hi, -hi, -lo against the points' hi, lo, hi,
    // and the factors of |p|^2 / 2
    kn_h8 b[KS];
    {
        const float* xq = x + (q < n ? q : n - 1) * d;
        const float scale = f->scale;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int k = 16 * ks + 8 * half + i;
                _Float16 r = (_Float16)0.0f;
                if (k < 3 * d) {
                    const int sec = k / d, c = k - sec * d;
                    _Float16 hi, lo;
                    knn_split((xq[c] - f->mu[c]) * scale, hi, lo);
                    r = sec == 2 ? -lo : -hi;
                } else if (k < 3 * d + 2) {
                    r = k == 3 * d ? (_Float16)32768.0f : (_Float16)16.0f;
                }
                b[ks][i] = r;
            }
    }

    float bv[T], thr = INFINITY;
    int32_t bj[T];
    int cnt = 0;
#pragma unroll
    for (int i = 0; i < T; ++i) {
        bv[i] = INFINITY;
        bj[i] = -1;
    }
    float2(*mine)[64] = buf[wave];
    auto sort_in = [&]() {
        const int rounds = wave_max_nonneg(cnt);
        for (int s = 0; s < rounds; ++s) {
            const float2 e = mine[s][lane];
            float v = s < cnt ? e.x : INFINITY;
            int32_t j = __float_as_int(e.y);
#pragma unroll
            for (int i = 0; i < T; ++i) {
                const bool lt = v < bv[i];
                const float ov = bv[i];
                const int32_t oj = bj[i];
                bv[i] = lt ? v : ov;
                bj[i] = lt ? j : oj;
                v = lt ? ov : v;
                j = lt ? oj : j;
            }
        }
        cnt = 0;
        // the T smallest of two ascending lists a, b are min(a[i], b[T - 1 - i])
        float m = -INFINITY;
#pragma unroll
        for (int i = 0; i < T; ++i) m = fmaxf(m, fminf(bv[i], __shfl_xor(bv[T - 1 - i], 32, 64)));
        thr = m;
    };

    kn_h8 a[KS];
    auto fetch = [&](int t) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) a[ks] = frag[((int64_t)t * KS + ks) * 64 + lane];
    };
    if (t0 < t1) fetch(t0);
    for (int t = t0; t < t1; ++t) {
        kn_f16v acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[ks], b[ks], acc, 0, 0, 0);
        fetch(t + 1 < t1 ? t + 1 : t);
        if (t == qt) {  // the query itself
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (8 * (r >> 2) + 4 * half + (r & 3) == col) acc[r] = INFINITY;
        }
        float m[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) m[g] = fminf(fminf(fminf(acc[4 * g], acc[4 * g + 1]), acc[4 * g + 2]), acc[4 * g + 3]);
        if (__ballot(fminf(fminf(m[0], m[1]), fminf(m[2], m[3])) < thr)) {
            const int32_t row0 = t * 32 + 4 * half;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                if (__ballot(m[g] < thr)) {
#pragma unroll
                    for (int r = 4 * g; r < 4 * g + 4; ++r)
                        if (acc[r] < thr) {
                            mine[cnt][lane] = make_float2(acc[r], __int_as_float(row0 + 8 * g + (r & 3)));
                            ++cnt;
                        }
                }
            }
            if (__ballot(cnt > kBuf - 16)) sort_in();
        }
    }
    sort_in();
    if (q < n) {
        int32_t* out = cand + (q * (2 * segs) + 2 * seg + half) * T;
#pragma unroll
        for (int i = 0; i < T; ++i) out[i] = bj[i];
        if (half == 0) bound[q * segs + seg] = thr;
    }
}

// Exact f32 distance: one FMA per coordinate, in order.
__device__ __forceinline__ float knn_exact(const float* __restrict__ a, const float* __restrict__ b, int32_t d) {
    float acc = 0.0f;
#pragma unroll 8
    for (int c = 0; c < d; ++c) {
        const float t = a[c] - b[c];
        acc = fmaf(t, t, acc);
    }
    return acc;
}

// One wavefront per query: exact distances of its candidates, their ranks by
// (distance, index), the k best written out, and the proof that no other
// point is nearer.  Every point outside the candidates has an approximate
// distance >= nu = |q|^2 + 2 min over the segments of their thresholds.  A point
// with |p| > P = |q| + 1.01 sqrt(d_k) is further than d_k anyway; for the
// others the approximation is off by at most
//   E = 2 [(3 2^-22 + g) |q| P + sub (|q| + P) + sub^2 + (g + 2^-22) P^2 / 2]
//       + tiny + b (|q|^2 + P^2) + h (|q| + P)^2,
// the split (2^-22 of each factor and the dropped lo lo product), g = (3 d + 4)
// 2^-23 of the accumulation over 3 d + 2 products, sub and tiny (2^-10 in scaled
// units) the range that the matrix cores may flush, b = (d + 4) 2^-23 of the f32
// norms and the final sum, h = 2^-22 of the centring.  The exact f32 distance is within rel of the
// real one.
__global__ __launch_bounds__(256) void knn_refine_kernel(const float* __restrict__ x, int64_t n, int32_t d, int32_t k,
                                                        const KnnFrame* __restrict__ f,
                                                        const float* __restrict__ half_norm, int32_t segs, int32_t T,
                                                        const float* __restrict__ bound,
                                                        const int32_t* __restrict__ cand,
                                                        int32_t* __restrict__ idx_out, float* __restrict__ d2_out,
                                                        int32_t* __restrict__ fails, float* __restrict__ fail_dk,
                                                        unsigned int* fail_count) {
    extern __shared__ float2 rsm[];  // [4][2 segs T] (distance, index)
    __shared__ float kth[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t q = folded(blockIdx.x, blockIdx.y, gridDim.x) * 4 + wave;
    const int C = 2 * segs * T;
    float2* sm = rsm + wave * C;
    const bool live = q < n, usable = live && !f->bad;
    float nu = INFINITY;
    if (usable) {
        for (int c = lane; c < C; c += 64) {
            const int32_t j = cand[q * C + c];
            float v = INFINITY;
            if (j >= 0 && j < n) v = knn_exact(x + q * d, x + (int64_t)j * d, d);
            sm[c] = make_float2(v, __int_as_float(j >= 0 && j < n ? j : INT32_MAX));
        }
        for (int s = 0; s < segs; ++s) nu = fminf(nu, bound[q * segs + s]);
    }
    if (lane == 0) kth[wave] = INFINITY;
    __syncthreads();
    if (usable) {
        for (int c = lane; c < C; c += 64) {
            const float v = sm[c].x;
            const int32_t j = __float_as_int(sm[c].y);
            if (!(v < INFINITY)) continue;
            int rank = 0;
            for (int o = 0; o < C; ++o) {
                const float2 u = sm[o];
                rank += (u.x < v || (u.x == v && __float_as_int(u.y) < j)) ? 1 : 0;
            }
            if (rank < k) {
                idx_out[q * k + rank] = j;
                if (d2_out) d2_out[q * k + rank] = v;
            }
            if (rank == k - 1) kth[wave] = v;
        }
    }
    __syncthreads();
    if (live && lane == 0) {
        bool ok = false;
        if (usable) {
            const float dk = kth[wave];
            const float nq = half_norm[q] * f->inv2, aq = sqrtf(nq) * 1.000001f;
            const float P = aq + 1.01f * sqrtf(dk), sub = f->sub;
            const float g = (float)(3 * d + 4) * 0x1p-23f, b = (float)(d + 4) * 0x1p-23f, h = 0x1p-22f;
            const float E = 1.01f * (2.0f * ((3.0f * 0x1p-22f + g) * aq * P + sub * (aq + P) + sub * sub +
                                             0.5f * (g + 0x1p-22f) * P * P) +
                                     f->inv2 * 0x1p-10f + b * (aq * aq + P * P) + h * (aq + P) * (aq + P));
            const float rel = (float)(d + 4) * 0x1.1p-24f;
            ok = (nq + f->inv2 * nu - E) * (1.0f - rel) > dk;
        }
        if (!ok) {
            const unsigned int slot = atomicAdd(fail_count, 1u);
            fails[slot] = (int32_t)q;
            fail_dk[slot] = kth[wave];
        }
    }
}

// The queries that are scanned: every point, or a list of *count of them, each with
// the k-th distance that its candidates gave (infinity when there were too few, or
// none).  Points beyond that distance cannot be among its k best, points at it can.
struct KnnRows {
    const int32_t* rows;        // NULL: every point
    const float* dk;
    const unsigned int* count;
    const KnnFrame* frame;
    int64_t limit, limit_free;  // queries from which on knn_block_kernel takes them: with the distances, without

    __device__ int64_t total(int64_t n) const { return rows ? (int64_t)*count : n; }
    __device__ bool many(int64_t m) const { return m >= (rows && !frame->bad ? limit : limit_free); }
    __device__ int64_t query(int64_t at) const { return rows ? (int64_t)rows[at] : at; }
    // distances below this are taken: the least float above dk
    __device__ float start(int64_t at) const {
        if (!rows) return INFINITY;
        const uint32_t b = __float_as_uint(dk[at]);  // not negative
        return __uint_as_float(b < 0x7f800000u ? b + 1u : 0x7f800000u);
    }
};

constexpr int kScanPts = 4;                      // points per lane and step
constexpr int kScanQ = 4;                        // queries per wavefront when there are many
constexpr int kScanCap = 64 * kScanPts + 64;     // buffered distances per query

// One wavefront per query, or per kScanQ queries when there are enough of them
// (each point is then read once for all): the distances of every point, 64 in
// the first step, which sets the first threshold, up to 256 in the later ones.
// Those below the running k-th best are appended to the query's buffer in LDS;
// when it holds more than 64 the k best are kept (by rank among the buffered)
// and the k-th becomes the threshold.  Points come in increasing order, so a
// later point tied with the k-th never enters, and a distance that is NaN or
// infinite is never below the threshold.
__global__ __launch_bounds__(256) void knn_scan_kernel(const float* __restrict__ x, int64_t n, int32_t d, int32_t k,
                                                       KnnRows r, int32_t* __restrict__ idx_out,
                                                       float* __restrict__ d2_out) {
    __shared__ float2 sb[4][kScanQ][kScanCap];
    __shared__ float sq[4][kScanQ][kKnnMaxD];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int64_t total = r.total(n);
    if (r.many(total)) return;
    const int per = total > 8192 ? kScanQ : 1;
    const int64_t groups = (total + per - 1) / per;
    auto settle = [] { __builtin_amdgcn_wave_barrier(); };  // LDS is in order within a wavefront
    for (int64_t g = (int64_t)blockIdx.x * 4 + wave; g < groups; g += (int64_t)gridDim.x * 4) {
        int64_t q[kScanQ];
        float thr[kScanQ];
        int cnt[kScanQ], live = 0;
        settle();
#pragma unroll
        for (int u = 0; u < kScanQ; ++u) {
            const int64_t at = g * per + u;
            const bool on = u < per && at < total;
            q[u] = on ? r.query(at) : 0;
            live += on ? 1 : 0;
            thr[u] = on ? r.start(at) : INFINITY;
            cnt[u] = 0;
            if (lane < d) sq[wave][u][lane] = x[q[u] * d + lane];
        }
        settle();
        for (int64_t base = 0, step = 64; base < n; base += step, step = step < 64 * kScanPts ? 2 * step : step) {
            const int64_t stop = base + step < n ? base + step : n;
            for (int64_t first = base; first < stop; first += 64) {
                const int64_t j = first + lane;
                const bool ok = j < stop;
                const float* p = x + (ok ? j : n - 1) * d;
                float acc[kScanQ];
#pragma unroll
                for (int u = 0; u < kScanQ; ++u) acc[u] = 0.0f;
                int c = 0;
                for (; c + 4 <= d; c += 4) {
                    float v[4];
                    __builtin_memcpy(v, p + c, 16);
#pragma unroll
                    for (int u = 0; u < kScanQ; ++u)
                        if (u < live)
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                const float t = sq[wave][u][c + e] - v[e];
                                acc[u] = fmaf(t, t, acc[u]);
                            }
                }
                for (; c < d; ++c) {
                    const float v = p[c];
#pragma unroll
                    for (int u = 0; u < kScanQ; ++u) {
                        const float t = sq[wave][u][c] - v;
                        acc[u] = fmaf(t, t, acc[u]);
                    }
                }
#pragma unroll
                for (int u = 0; u < kScanQ; ++u) {
                    const bool in = u < live && ok && acc[u] < thr[u] && j != q[u];
                    const unsigned long long m = __ballot(in);
                    if (m) {
                        const int at = cnt[u] + (int)__builtin_amdgcn_mbcnt_hi(
                                                    (unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
                        if (in) sb[wave][u][at] = make_float2(acc[u], __int_as_float((int32_t)j));
                        cnt[u] += __popcll(m);
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < kScanQ; ++u) {
                if (u < live && (cnt[u] > 64 || step <= 128 || stop == n)) {
                    float2* b = sb[wave][u];
                    const int have = cnt[u];
                    float2 mine[kScanCap / 64];
                    int rank[kScanCap / 64];
                    settle();
#pragma unroll
                    for (int e = 0; e < kScanCap / 64; ++e) {
                        rank[e] = k;
                        if (64 * e < have) {
                            const int at = 64 * e + lane;
                            mine[e] = b[at < have ? at : 0];
                            const int32_t j = __float_as_int(mine[e].y);
                            int r = at < have ? 0 : k;
                            for (int o = 0; o < have; ++o) {
                                const float2 w = b[o];
                                r += (w.x < mine[e].x || (w.x == mine[e].x && __float_as_int(w.y) < j)) ? 1 : 0;
                            }
                            rank[e] = r;
                        }
                    }
                    settle();
#pragma unroll
                    for (int e = 0; e < kScanCap / 64; ++e)
                        if (rank[e] < k) b[rank[e]] = mine[e];
                    settle();
                    cnt[u] = have < k ? have : k;
                    if (have >= k) thr[u] = b[k - 1].x;
                }
            }
        }
#pragma unroll
        for (int u = 0; u < kScanQ; ++u) {
            if (u < live && lane < k) {
                const float2 e = sb[wave][u][lane];
                idx_out[q[u] * k + lane] = lane < cnt[u] ? __float_as_int(e.y) : -1;
                if (d2_out) d2_out[q[u] * k + lane] = lane < cnt[u] ? e.x : INFINITY;
            }
        }
    }
}

constexpr int kBlockQ = 256;  // queries and threads of a workgroup (64 and 128: more staging per query, up to 1.5 times as long)

template <int D, int KM> struct KnnBlock {
    static constexpr int points = D <= 20 ? 256 : 128;  // staged at a time: at most 32 KB
    static constexpr int ahead = D <= 16 && D + KM <= 40 ? 4 : 2;  // points whose distances are formed together
    // wavefronts per SIMD that the query, its list and one point leave registers for
    static constexpr int regs = 2 * D + 2 * KM + (D > 40 ? 44 : 24);
    static constexpr int waves = regs > 168 ? 2 : regs > 128 ? 3 : 4;
};

// One query per thread, its coordinates and its k best in registers; the points go
// through LDS and are read as broadcasts, so a pair costs little more than its 2 D
// vector instructions, which bound it.  Made for many queries: up to one workgroup
// per CU the time does not depend on their number.  Points come in increasing order,
// so a later point tied with the k-th never enters.
template <int D, int KM>
__global__ __launch_bounds__(kBlockQ, (KnnBlock<D, KM>::waves)) void knn_block_kernel(
    const float* __restrict__ x, int64_t n, int32_t d, int32_t k, KnnRows r, int32_t* __restrict__ idx_out,
    float* __restrict__ d2_out) {
    constexpr int TP = KnnBlock<D, KM>::points, P = KnnBlock<D, KM>::ahead;
    __shared__ float tile[TP * D];
    const int64_t total = r.total(n), at = (int64_t)blockIdx.x * kBlockQ + threadIdx.x;
    if (!r.many(total) || (int64_t)blockIdx.x * kBlockQ >= total) return;
    const bool active = at < total;
    const int64_t q = active ? r.query(at) : 0;
    float qc[D];
#pragma unroll
    for (int c = 0; c < D; ++c) qc[c] = c < d ? x[q * d + c] : 0.0f;
    float best[KM];
    int32_t bi[KM];
#pragma unroll
    for (int i = 0; i < KM; ++i) {
        best[i] = INFINITY;
        bi[i] = -1;
    }
    float thr = active ? r.start(at) : 0.0f;
    for (int64_t base = 0; base < n; base += TP) {
        const int cnt = (int)(n - base < TP ? n - base : TP);
        __syncthreads();
        for (int e = threadIdx.x; e < TP * D; e += kBlockQ) {
            const int p = e / D, c = e - p * D;
            tile[e] = (p < cnt && c < d) ? x[(base + p) * d + c] : 0.0f;
        }
        __syncthreads();
        for (int p = 0; p < cnt; p += P) {
            float acc[P];
#pragma unroll
            for (int u = 0; u < P; ++u) {
                acc[u] = 0.0f;
#pragma unroll
                for (int c = 0; c < D; ++c) {
                    const float t = qc[c] - tile[(p + u) * D + c];
                    acc[u] = fmaf(t, t, acc[u]);
                }
            }
            float nearest = acc[0];
#pragma unroll
            for (int u = 1; u < P; ++u) nearest = fminf(nearest, acc[u]);
            // one branch for all of them in most steps (100 000 points, d = 2: 6.3 -> 4.1 ms; not
            // where it has the compiler hold the points' reads back: d = 64, k = 15 50 -> 57)
            if ((D <= 40 || KM > 16) && !(nearest < thr)) continue;
#pragma unroll
            for (int u = 0; u < P; ++u) {
                const int64_t j = base + p + u;
                if (acc[u] < thr && j != q && p + u < cnt) {
                    // insert after every entry <= acc and shift the rest down one place
                    // (descending i reads each old entry before it is overwritten)
#pragma unroll
                    for (int i = KM - 1; i >= 1; --i) {
                        const bool shift = acc[u] < best[i - 1], here = acc[u] < best[i];
                        best[i] = shift ? best[i - 1] : (here ? acc[u] : best[i]);
                        bi[i] = shift ? bi[i - 1] : (here ? (int32_t)j : bi[i]);
                    }
                    if (acc[u] < best[0]) {
                        best[0] = acc[u];
                        bi[0] = (int32_t)j;
                    }
                    float t = best[0];
#pragma unroll
                    for (int i = 1; i < KM; ++i) t = (i == k - 1) ? best[i] : t;
                    thr = fminf(thr, t);
                }
            }
        }
    }
    if (!active) return;
#pragma unroll
    for (int i = 0; i < KM; ++i) {
        if (i < k) {
            idx_out[q * k + i] = bi[i];
            if (d2_out) d2_out[q * k + i] = best[i];
        }
    }
}

template <int D, int KM>
void knn_block_launch_t(const float* x, int64_t n, int32_t d, int32_t k, const KnnRows& r, int32_t* idx, float* d2,
                        hipStream_t s) {
    hipLaunchKernelGGL((knn_block_kernel<D, KM>), dim3((unsigned)((n + kBlockQ - 1) / kBlockQ)), dim3(kBlockQ), 0, s, x, n,
                       d, k, r, idx, d2);
}

template <int D>
void knn_block_launch_d(const float* x, int64_t n, int32_t d, int32_t k, const KnnRows& r, int32_t* idx, float* d2,
                        hipStream_t s) {
    if (k <= 8) knn_block_launch_t<D, 8>(x, n, d, k, r, idx, d2, s);
    else if (k <= 16) knn_block_launch_t<D, 16>(x, n, d, k, r, idx, d2, s);
    else if (k <= 24) knn_block_launch_t<D, 24>(x, n, d, k, r, idx, d2, s);
    else knn_block_launch_t<D, 32>(x, n, d, k, r, idx, d2, s);
}

void knn_block_launch(const float* x, int64_t n, int32_t d, int32_t k, const KnnRows& r, int32_t* idx, float* d2,
                      hipStream_t s) {
    switch (d) {
#define GL_KNN_D(DD) \
    case DD:         \
        return knn_block_launch_d<DD>(x, n, d, k, r, idx, d2, s);
        GL_KNN_D(1) GL_KNN_D(2) GL_KNN_D(3) GL_KNN_D(4) GL_KNN_D(5) GL_KNN_D(6) GL_KNN_D(7) GL_KNN_D(8)
        GL_KNN_D(9) GL_KNN_D(10) GL_KNN_D(11) GL_KNN_D(12) GL_KNN_D(13) GL_KNN_D(14) GL_KNN_D(15)
        GL_KNN_D(16)
#undef GL_KNN_D
        default:
            break;
    }
    // wider features: padded to the next width with zero coordinates
    if (d <= 20) return knn_block_launch_d<20>(x, n, d, k, r, idx, d2, s);
    if (d <= 24) return knn_block_launch_d<24>(x, n, d, k, r, idx, d2, s);
    if (d <= 28) return knn_block_launch_d<28>(x, n, d, k, r, idx, d2, s);
    if (d <= 32) return knn_block_launch_d<32>(x, n, d, k, r, idx, d2, s);
    if (d <= 40) return knn_block_launch_d<40>(x, n, d, k, r, idx, d2, s);
    if (d <= 48) return knn_block_launch_d<48>(x, n, d, k, r, idx, d2, s);
    if (d <= 56) return knn_block_launch_d<56>(x, n, d, k, r, idx, d2, s);
    return knn_block_launch_d<64>(x, n, d, k, r, idx, d2, s);
}

// Queries from which on knn_block_kernel is the faster of the two, whose time does
// not depend on their number up to some 65 000.  With a k-th distance to start from
// (100 000 points, k = 15, scan / block in ms without the 1.6 to 7.1 of the products):
// d = 2: 30 000 queries 3.6 / 4.0, 60 000 7.5 / 4.0; d = 10: 7.5 / 8.7 and 15.4 / 8.7;
// d = 27: 16 000 11.1 / 21.1, 30 000 23.9 / 21.1; d = 64: 19.8 / 42.3 and 43.1 / 42.3.
int64_t knn_block_min_listed(int32_t d) { return d <= 16 ? 36000 : 28000; }

// Without one (every point, k = 15): d = 3: 48 000 points 2.9 / 2.7, 65 000 5.2 / 3.6, k = 32:
// 100 000 13.4 / 14.1; d = 10: 48 000 4.4 / 4.6, 65 000 8.0 / 6.2; d = 27: 32 000 6.5 / 7.3,
// 48 000 14.2 / 10.5; d = 64: 13.7 / 15.2 and 28.9 / 21.9.
int64_t knn_block_min(int32_t d, int32_t k) { return d > 16 ? 36000 : d <= 3 && k > 16 ? 110000 : 50000; }

// The queries of r by whichever of the two kernels they are enough for: known here
// for every point, on the device for a list.
hipError_t knn_scan(const float* x, int64_t n, int32_t d, int32_t k, KnnRows r, int32_t* idx, float* d2, hipStream_t s) {
    r.limit = knn_block_min_listed(d);
    r.limit_free = knn_block_min(d, k);
    const bool block = n >= (r.rows ? std::min(r.limit, r.limit_free) : r.limit_free);
    if (r.rows || !block) {
        const int64_t blocks = r.rows ? 1024 : n > 8192 ? (n + 4 * kScanQ - 1) / (4 * kScanQ) : (n + 3) / 4;
        hipLaunchKernelGGL(knn_scan_kernel, dim3((unsigned)std::min<int64_t>(blocks, 1 << 20)), dim3(256), 0, s, x, n, d,
                           k, r, idx, d2);
    }
    if (block) knn_block_launch(x, n, d, k, r, idx, d2, s);
    return hipGetLastError();
}

template <int KS>
hipError_t knn_tile_launch(const float* x, int64_t n, int32_t d, int32_t T, int32_t tiles, int32_t segs,
                           const KnnFrame* f, kn_h8* frag, float* half_norm, float* bound, int32_t* cand,
                           hipStream_t s) {
    const int64_t np = (int64_t)tiles * 32;
    // from 67 M points (the refinement) and 165 M (the operands of 64 coordinates) on, more
    // threads than one dimension of a launch holds
    const Fold fp = fold_blocks((np * 2 * KS + 255) / 256);
    hipLaunchKernelGGL(knn_pack_kernel<KS>, dim3(fp.x, fp.y), dim3(256), 0, s, x, n, np, d, f, frag, half_norm);
    const Fold ft = fold_blocks(((int64_t)tiles + kTileWaves - 1) / kTileWaves * segs);
    const dim3 grid(ft.x, ft.y), block(64 * kTileWaves);
#define GL_KNN_T(TT)                                                                                        \
    case TT:                                                                                                \
        hipLaunchKernelGGL((knn_tile_kernel<KS, TT>), grid, block, 0, s, x, n, d, f, (const kn_h8*)frag,    \
                           tiles, segs, bound, cand);                                                       \
        break;
    switch (T) {
        GL_KNN_T(8) GL_KNN_T(12) GL_KNN_T(16) GL_KNN_T(20) GL_KNN_T(24) GL_KNN_T(32) GL_KNN_T(36)
        default: return hipErrorInvalidValue;
    }
#undef GL_KNN_T
    return hipGetLastError();
}

// One coordinate is scanned: near neighbours on a line are closer than the
// approximate distances can tell apart, and most queries would be scanned anyway.
// limit: an allocation of more bytes counts as failed.  rescanned (or NULL, and then
// nothing waits): the queries scanned over all points.
hipError_t knn_launch(const float* x, int64_t n, int32_t d, int32_t k, int32_t* idx, float* d2, size_t limit,
                      int64_t* rescanned, hipStream_t s) {
    if (rescanned) *rescanned = n;
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    hipError_t e = hipStreamIsCapturing(s, &cap);
    if (e != hipSuccess) return e;
    if (n * (d + 10) <= kKnnScanMax || d == 1 || cap != hipStreamCaptureStatusNone)
        return knn_scan(x, n, d, k, KnnRows{}, idx, d2, s);
    const int32_t tiles = (int32_t)((n + 31) / 32);
    const int64_t np = (int64_t)tiles * 32;
    const int32_t T = k <= 4 ? 8 : k <= 8 ? 12 : k <= 12 ? 16 : k <= 16 ? 20 : k <= 20 ? 24 : k <= 28 ? 32 : 36;
    const int32_t KS = d <= 4 ? 1 : d <= 10 ? 2 : d <= 15 ? 3 : d <= 20 ? 4 : d <= 31 ? 6 : d <= 42 ? 8 : 13;
    int32_t segs = 1;
    while (segs < 8 && (int64_t)tiles * segs * 2 <= kKnnWaves) segs *= 2;
    auto al = [](size_t b) { return (b + 255) & ~(size_t)255; };
    const size_t b_frag = al((size_t)np * KS * 32), b_norm = al((size_t)np * 4),
                 b_cand = al((size_t)n * 2 * segs * T * 4), b_bound = al((size_t)n * segs * 4), b_fail = al((size_t)n * 4),
                 b_sum = al((size_t)kStatBlocks * kKnnMaxD * 8), b_mm = al((size_t)kStatBlocks * kKnnMaxD * 4),
                 b_frame = al(sizeof(KnnFrame)) + 256;
    const size_t total = b_frag + b_norm + b_cand + b_bound + 2 * b_fail + b_sum + 2 * b_mm + b_frame;
    char* base = nullptr;
    if (total > limit || hipMallocAsync((void**)&base, total, s) != hipSuccess) {
        (void)hipGetLastError();
        return knn_scan(x, n, d, k, KnnRows{}, idx, d2, s);
    }
    char* p = base;
    auto take = [&](size_t b) { char* r = p; p += b; return r; };
    kn_h8* frag = (kn_h8*)take(b_frag);
    float* half_norm = (float*)take(b_norm);
    int32_t* cand = (int32_t*)take(b_cand);
    float* bound = (float*)take(b_bound);
    int32_t* fails = (int32_t*)take(b_fail);
    float* fail_dk = (float*)take(b_fail);
    double* psum = (double*)take(b_sum);
    float* pmin = (float*)take(b_mm);
    float* pmax = (float*)take(b_mm);
    KnnFrame* f = (KnnFrame*)take(b_frame - 256);
    unsigned int* fail_count = (unsigned int*)p;
    hipLaunchKernelGGL(knn_stats_kernel, dim3(kStatBlocks), dim3(256), 0, s, x, n, d, psum, pmin, pmax);
    hipLaunchKernelGGL(knn_frame_kernel, dim3(1), dim3(256), 0, s, (const double*)psum, (const float*)pmin,
                       (const float*)pmax, n, d, f, fail_count);
    e = hipGetLastError();
    if (e == hipSuccess) {
        switch (KS) {
#define GL_KNN_KS(KK)                                                                                     \
    case KK:                                                                                              \
        e = knn_tile_launch<KK>(x, n, d, T, tiles, segs, f, frag, half_norm, bound, cand, s);         \
        break;
            GL_KNN_KS(1) GL_KNN_KS(2) GL_KNN_KS(3) GL_KNN_KS(4) GL_KNN_KS(6) GL_KNN_KS(8) GL_KNN_KS(13)
#undef GL_KNN_KS
            default: e = hipErrorInvalidValue;
        }
    }
    if (e == hipSuccess) {
        const Fold fr = fold_blocks((n + 3) / 4);
        hipLaunchKernelGGL(knn_refine_kernel, dim3(fr.x, fr.y), dim3(256), (size_t)4 * 2 * segs * T * 8, s, x, n, d, k,
                           (const KnnFrame*)f, (const float*)half_norm, segs, T, (const float*)bound,
                           (const int32_t*)cand, idx, d2, fails, fail_dk, fail_count);
        e = hipGetLastError();
    }
    if (e == hipSuccess) {
        KnnRows r{};
        r.rows = fails;
        r.dk = fail_dk;
        r.count = fail_count;
        r.frame = f;
        e = knn_scan(x, n, d, k, r, idx, d2, s);
    }
    if (e == hipSuccess && rescanned) {
        unsigned int listed = 0;
        e = hipMemcpyAsync(&listed, fail_count, sizeof(listed), hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        *rescanned = listed;
    }
    const hipError_t ef = hipFreeAsync(base, s);
    return e != hipSuccess ? e : ef;
}

}  // namespace
}  // namespace gl

namespace {
thread_local int64_t g_knn_fallback = 0;
}

extern "C" int64_t gl_knn_fallback_rows(void) { return g_knn_fallback; }

static gl_status knn_call(const float* x, int64_t n, int32_t d, int32_t k, int32_t* idx_out, float* d2_out, size_t limit,
                          int64_t* rescanned, void* stream) {
    if (!x || !idx_out) {
        gl::set_last_error("x and idx_out must not be NULL");
        return GL_E_INVALID_ARG;
    }
    if (d < 1 || d > 4096) {
        gl::set_last_error("d must lie in [1, 4096]");
        return GL_E_INVALID_ARG;
    }
    if (k < 1 || k > 32) {
        gl::set_last_error("k must lie in [1, 32]");
        return GL_E_INVALID_ARG;
    }
    if (n <= k || n > INT32_MAX) {
        gl::set_last_error("need k < n < 2^31");
        return GL_E_INVALID_ARG;
    }
    if (d > 64) {
        int64_t fb = 0;
        const gl_status st = gl::knn_wide(x, n, d, k, idx_out, d2_out, limit, (hipStream_t)stream, &fb);
        g_knn_fallback = st == GL_OK ? fb : -1;
        if (rescanned) *rescanned = fb;
        return st;
    }
    g_knn_fallback = 0;
    const hipError_t e = gl::knn_launch(x, n, d, k, idx_out, d2_out, limit, rescanned, (hipStream_t)stream);
    if (e != hipSuccess) {
        gl::set_last_error(std::string("knn launch: ") + hipGetErrorString(e));
        return GL_E_HIP;
    }
    return GL_OK;
}

extern "C" gl_status gl_knn(const float* x, int64_t n, int32_t d, int32_t k, int32_t* idx_out, float* d2_out,
                            void* stream) {
    return knn_call(x, n, d, k, idx_out, d2_out, SIZE_MAX, nullptr, stream);
}

extern "C" gl_status gl_knn_bounded(const float* x, int64_t n, int32_t d, int32_t k, int32_t* idx_out, float* d2_out,
                                    size_t temp_bytes, int64_t* rescanned, void* stream) {
    if (!rescanned) {
        gl::set_last_error("rescanned must not be NULL");
        return GL_E_INVALID_ARG;
    }
    const gl_status st = knn_call(x, n, d, k, idx_out, d2_out, temp_bytes, rescanned, stream);
    if (st == GL_OK && hipStreamSynchronize((hipStream_t)stream) != hipSuccess) {
        gl::set_last_error("knn");
        return GL_E_HIP;
    }
    return st;
}
