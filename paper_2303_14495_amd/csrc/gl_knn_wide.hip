// k nearest neighbours for wide features (64 < d <= 4096), with the same
// result as the exact kernel: the k smallest f32 distances
// sum_c (q_c - p_c)^2 (FMA, coordinate order), ties to the lower index.
//
// The n^2 d work is a Gram matrix, so it runs on the matrix cores: the points
// are centred, scaled by a power of two, rounded to f16 and laid out as matrix
// operands, and one kernel multiplies a block of 256 queries by blocks of 256
// points with v_mfma_f32_32x32x16_f16 (f32 accumulation) and keeps, for every
// query, the points of the largest <q, p> - |p|^2 / 2, which are the nearest; no
// product leaves the chip.  A query's points are dealt to 4 lists per segment of
// the point blocks, each keeping its T best, and a list's last entry bounds what
// it left out: nu, the smallest such distance, is a lower bound, approximately, on
// every point that is no candidate.  A second kernel takes the candidates that can
// be among the k best given the approximation error E_q, recomputes their exact
// f32 distances and checks a certificate: E_q is a bound from the f16 rounding,
// the f32 accumulation and the norms, so if nu - E_q exceeds the exact k-th
// distance no other point can enter or tie.  Rows without the certificate are
// recomputed by an exact scan.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>

#include "gl_internal.hpp"

namespace {


gl_status wfail(gl_status st, const std::string& m) {
    gl::set_last_error(m);
    return st;
}

// Column means, so the approximate distances are formed from centred points,
// whose smaller norms shrink the error bound: double partial sums over the
// rows r = slice, slice + kMeanSlices, ... (one block row per slice), then the
// slices added in order.
constexpr int kMeanSlices = 256;

__global__ void kw_mean_partial_kernel(const float* __restrict__ x, int64_t n, int32_t d,
                                       double* __restrict__ part) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= d) return;
    double s = 0.0;
    for (int64_t i = blockIdx.y; i < n; i += kMeanSlices) s += (double)x[i * d + c];
    part[(int64_t)blockIdx.y * d + c] = s;
}

__global__ void kw_mean_final_kernel(const double* __restrict__ part, int64_t n, int32_t d,
                                     float* __restrict__ mu) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= d) return;
    double s = 0.0;
    for (int r = 0; r < kMeanSlices; ++r) s += part[(int64_t)r * d + c];
    mu[c] = (float)(s / (double)n);
}

// |x_i - mu|^2 (f32, fixed-order wave reduction), a wavefront per row, and the
// maxima of |x_ic - mu_c| and of the norms over all points as the bits of
// non-negative floats (monotone as unsigned; a NaN is larger than any number).
// One addition to the maxima per workgroup of many rows: one per row took 0.8 ms
// at 70 000 x 784, all of it waiting for one address.
__global__ __launch_bounds__(256) void kw_norms_kernel(const float* __restrict__ x, const float* __restrict__ mu,
                                                      int64_t n, int32_t d, float* __restrict__ norm2,
                                                      unsigned int* maxima) {
    __shared__ unsigned int sh[2][4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    float m = 0.f;
    unsigned int mn = 0u;
    for (int64_t i = (int64_t)blockIdx.x * 4 + wave; i < n; i += (int64_t)gridDim.x * 4) {
        float s = 0.f;
        for (int c = lane; c < d; c += 64) {
            const float v = x[i * d + c] - mu[c];
            s = fmaf(v, v, s);
            m = fmaxf(m, fabsf(v));
        }
        for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
        if (lane == 0) norm2[i] = s;
        mn = max(mn, __float_as_uint(s) & 0x7fffffffu);
    }
    for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
    if (lane == 0) {
        sh[0][wave] = __float_as_uint(m);
        sh[1][wave] = mn;
    }
    __syncthreads();
    if (threadIdx.x < 2)
        atomicMax(maxima + threadIdx.x, max(max(sh[threadIdx.x][0], sh[threadIdx.x][1]),
                                            max(sh[threadIdx.x][2], sh[threadIdx.x][3])));
}

typedef _Float16 kw_h8 __attribute__((ext_vector_type(8)));
typedef float kw_f16v __attribute__((ext_vector_type(16)));
typedef uint32_t kw_u4 __attribute__((ext_vector_type(4)));

// f16(scale * (x[i][c] - mu[c])) as matrix operands: xp[i / 32][c / 16][lane][8],
// lane l holding coordinates 16 (c / 16) + 8 (l / 32) .. + 7 of row i % 32 = l % 32,
// rows from n to 32 tiles and coordinates from d on zero.  A wavefront writes
// four neighbouring 1 KB operands, whose rows share lines of x.
__global__ __launch_bounds__(256) void kw_pack_kernel(const float* __restrict__ x, const float* __restrict__ mu,
                                                     int64_t n, int32_t d, int64_t tiles, int32_t nks, float scale,
                                                     kw_h8* __restrict__ xp) {
    const int lane = threadIdx.x & 63;
    const int32_t groups = (nks + 3) / 4;
    const int64_t item = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (item >= tiles * groups) return;
    const int64_t tile = item / groups;
    const int ks0 = (int)(item - tile * groups) * 4;
    const int64_t i = tile * 32 + (lane & 31);
    for (int ks = ks0; ks < min(ks0 + 4, nks); ++ks) {
        const int c0 = ks * 16 + 8 * (lane >> 5);
        kw_h8 h;
#pragma unroll
        for (int e = 0; e < 8; ++e)
            h[e] = i < n && c0 + e < d ? (_Float16)(scale * (x[i * d + c0 + e] - mu[c0 + e])) : (_Float16)0.0f;
        xp[(tile * nks + ks) * 64 + lane] = h;
    }
}

// cn[i] = -|x_i|^2 scale^2 / 2, the products' starting value; -inf for rows that pad.
__global__ __launch_bounds__(256) void kw_start_kernel(const float* __restrict__ norm2, int64_t n, int64_t np,
                                                      double factor, float* __restrict__ cn) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < np) cn[i] = i < n ? (float)(factor * (double)norm2[i]) : -INFINITY;
}

// Insert (v, j) into an ascending list of T entries (ties by index); returns
// the entry pushed out at the end.
template <int T>
__device__ __forceinline__ void kw_insert(float (&bv)[T], int32_t (&bj)[T], float v, int32_t j, float& out_v) {
    out_v = bv[T - 1];
#pragma unroll
    for (int t = T - 1; t > 0; --t) {
        const bool mv = v < bv[t - 1] || (v == bv[t - 1] && j < bj[t - 1]);
        const bool here = !mv && (v < bv[t] || (v == bv[t] && j < bj[t]));
        if (mv) {
            bv[t] = bv[t - 1];
            bj[t] = bj[t - 1];
        } else if (here) {
            bv[t] = v;
            bj[t] = j;
        }
    }
    if (v < bv[0] || (v == bv[0] && j < bj[0])) {
        bv[0] = v;
        bj[0] = j;
    }
}

// Pop the wave-wide smallest (v, j) head among the lanes' ascending lists;
// every lane receives it, and the owning lane advances its list.
template <int T>
__device__ __forceinline__ void kw_pop_min(float (&bv)[T], int32_t (&bj)[T], float& v, int32_t& j) {
    float hv = bv[0];
    int32_t hj = bj[0];
    for (int off = 32; off > 0; off >>= 1) {
        const float ov = __shfl_xor(hv, off, 64);
        const int32_t oj = __shfl_xor(hj, off, 64);
        if (ov < hv || (ov == hv && oj < hj)) {
            hv = ov;
            hj = oj;
        }
    }
    v = hv;
    j = hj;
    if (bj[0] == hj && bv[0] == hv && hj >= 0) {
#pragma unroll
        for (int t = 0; t < T - 1; ++t) {
            bv[t] = bv[t + 1];
            bj[t] = bj[t + 1];
        }
        bv[T - 1] = INFINITY;
        bj[T - 1] = INT32_MAX;
    }
}

constexpr int kWB = 256;             // queries and points per block
constexpr int kWThreads = 512;       // 8 wavefronts: 2 point halves x 4 query quarters
constexpr int kWStep = 32;           // coordinates per staging step (two MFMA k-steps)
constexpr int kWStage = 2048;        // 16-byte vectors of a staged step: 2 x 8 operand tiles x 2 x 64 lanes
constexpr int kWHits = 12;           // entries of a lane's queue
constexpr int kWSegs = 4;            // segments per query block of a full round
constexpr int kWRound = 64;          // query blocks of a full round: 64 x 4 workgroups, one per CU
constexpr int kWMaxSegs = 16;
constexpr int kWMaxCand = 768;       // candidates of a query: 4 kWMaxSegs lists of 12
constexpr size_t kWLds = (size_t)3 * kWStage * 16 + (size_t)kWHits * kWThreads * 8 + (size_t)2 * kWB * 4;

// How the (query block, point segment) pairs of one pass are dealt to workgroups.
// Full rounds of 64 query blocks x 4 segments: the 32 workgroups of an XCD
// (blockIdx % 8) hold 8 query blocks, each read by 4 of them, and 4 segments, each
// read by 8, so that its L2 serves most of the operands' reads.  The query blocks
// left over are cut into seg_r segments to fill the chip once more (16 at most: a
// segment has 4 lists of candidates per query).  One pass takes all query blocks
// unless their lists cannot be allocated.
struct KwPlan {
    int32_t nblk;   // blocks of kWB points
    int32_t first;  // first query block of the pass
    int32_t nq;     // its query blocks
    int32_t full;   // those of them in full rounds
    int32_t seg_r;  // segments of the others
    __host__ __device__ int32_t per() const { return ((nq - full) * seg_r + 7) / 8; }
    __host__ __device__ uint32_t blocks() const { return (uint32_t)full * kWSegs + 8u * (uint32_t)per(); }
    // lists of query q of the pass (q = 0: its first)
    __host__ __device__ int32_t lists(int64_t q) const { return 4 * (q < (int64_t)full * kWB ? kWSegs : seg_r); }
    __host__ __device__ int64_t first_list(int64_t q) const {
        const int64_t nf = (int64_t)full * kWB;
        return q < nf ? q * 4 * kWSegs : nf * 4 * kWSegs + (q - nf) * 4 * seg_r;
    }
};

KwPlan kw_plan(int32_t nblk, int32_t first, int32_t nq) {
    KwPlan p{nblk, first, nq, nq / kWRound * kWRound, 1};
    const int32_t rest = nq - p.full;
    if (rest) p.seg_r = std::max(kWSegs, std::min(std::min(kWMaxSegs, nblk), 256 / rest));
    return p;
}

// Most lists of the passes of `step` query blocks each.
int64_t kw_lists(int32_t nblk, int32_t step) {
    const KwPlan p = kw_plan(nblk, 0, step), last = kw_plan(nblk, 0, nblk % step);
    return std::max(p.first_list((int64_t)step * kWB), last.first_list((int64_t)last.nq * kWB));
}

// One 256 x 256 block of products per step of the tile loop.  Wavefront w computes
// points 128 (w / 4) .. by queries 64 (w % 4) .. with 4 x 2 MFMA tiles of 32 x 32
// (lane l: A row / B column l % 32, coordinates 8 (l / 32) .. + 7; result r: row
// (point) 8 (r / 4) + 4 (l / 32) + r % 4, column (query) l % 32), so a lane has 64
// points of each of its two queries, a list of T for each, and no exchange of
// distances between lanes.
//
// What bounds it: LDS (12 KB of operands read per wavefront for 16 MFMAs, 94 of the
// 128 bytes per clock at full matrix rate, and the staging writes) and the
// selection.  128 x 64 per wavefront halves the operand reads of 32 x 64 tiles.
// Three staging buffers: while step i is multiplied, step i + 1 is complete, so
// its first operands are read early, step i + 2 is being written and step i + 3 is
// on its way from memory; one barrier per step.
//
// Selection: a point better than the list's last entry goes to the lane's queue in
// LDS; queues are emptied into the lists (T med3 steps each) when one may
// overflow, after eight points, and at the end of the lane's 64.
// 70 000 x 784, k = 10: 8.4 ms (910 TFLOP/s) against 17.7 with 32 x 64 products per
// wavefront and distances exchanged through LDS; 25, 12, 6 and 3 staging steps (784, 384,
// 192 and 96 coordinates) take 8.65, 5.01, 3.58 and 2.95, which is 0.28 per step and
// 1.6 for selection and the blocks' starts at the long end.  The whole call 21.5 ->
// 10.4 ms, with k = 32 78 -> 10.9.
template <int T>
__global__ __launch_bounds__(kWThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void kw_tile_kernel(
    const kw_h8* __restrict__ xp, const float* __restrict__ cn, int64_t n, int32_t ns, KwPlan plan,
    uint2* __restrict__ cand) {
    extern __shared__ __attribute__((aligned(16))) unsigned char kw_smem[];
    kw_h8* stage = reinterpret_cast<kw_h8*>(kw_smem);
    uint32_t* queue = reinterpret_cast<uint32_t*>(kw_smem + (size_t)3 * kWStage * 16);
    float* start = reinterpret_cast<float*>(kw_smem + (size_t)3 * kWStage * 16 + (size_t)kWHits * kWThreads * 8);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wp = wave >> 2, wq = wave & 3;
    int qb, seg, nseg;
    if ((int)blockIdx.x < plan.full * kWSegs) {
        const int i = blockIdx.x & 255;
        qb = (int)(blockIdx.x >> 8) * kWRound + (i & 7) * 8 + (i >> 5);
        seg = (i >> 3) & 3;
        nseg = kWSegs;
    } else {
        const int i = (int)blockIdx.x - plan.full * kWSegs, item = (i & 7) * plan.per() + (i >> 3);
        if (i >= 8 * plan.per() || item >= (plan.nq - plan.full) * plan.seg_r) return;
        qb = __builtin_amdgcn_readfirstlane(plan.full + item / plan.seg_r);
        seg = __builtin_amdgcn_readfirstlane(item % plan.seg_r);
        nseg = plan.seg_r;
    }
    // fewer blocks than segments: each takes every fourth point of all of them
    const bool dealt = plan.nblk < kWSegs;
    const int b0 = dealt ? 0 : (int)((int64_t)plan.nblk * seg / nseg);
    const int b1 = dealt ? plan.nblk : (int)((int64_t)plan.nblk * (seg + 1) / nseg);
    auto start_of = [&](int b) {  // this lane's point of block b
        const float v = cn[(int64_t)min(b, b1 - 1) * kWB + tid];
        return dealt && (tid & 3) != seg ? -INFINITY : v;
    };

    // staging: wavefront w copies operand tile w of the points and of the queries, 1 KB per instruction
    const int64_t tile_v = (int64_t)ns * 128;  // vectors of an operand tile
    const kw_h8* qsrc = xp + ((int64_t)(plan.first + qb) * 8 + wave) * tile_v;
    const kw_h8* psrc = xp + ((int64_t)b0 * 8 + wave) * tile_v;
    int fb = b0, fs = 0;  // block and step of the next request; past the end the last block is read again
    kw_h8 r0, r1, r2, r3;
    auto fetch = [&]() {
        const kw_h8 *ps = psrc + fs * 128, *qs = qsrc + fs * 128;
        r0 = ps[lane];
        r1 = ps[64 + lane];
        r2 = qs[lane];
        r3 = qs[64 + lane];
        const bool wrap = ++fs == ns, more = wrap && fb + 1 < b1;
        fs = wrap ? 0 : fs;
        fb += more ? 1 : 0;
        psrc += more ? 8 * tile_v : 0;
    };
    auto put = [&](int at) {
        kw_h8* dst = stage + at + wave * 128 + lane;
        dst[0] = r0;
        dst[64] = r1;
        dst[1024] = r2;
        dst[1024 + 64] = r3;
    };
    kw_h8 fa[2][4], fq[2][2];
    auto frags = [&](int at, int ks) {
#pragma unroll
        for (int m = 0; m < 4; ++m) fa[ks][m] = stage[at + (wp * 4 + m) * 128 + ks * 64 + lane];
#pragma unroll
        for (int c = 0; c < 2; ++c) fq[ks][c] = stage[at + 1024 + (wq * 2 + c) * 128 + ks * 64 + lane];
    };

    float bv[2][T];
    uint32_t bj[2][T];
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int t = 0; t < T; ++t) {
            bv[c][t] = -INFINITY;
            bj[c][t] = 0x7fffffffu;
        }
    const int64_t q0 = (int64_t)(plan.first + qb) * kWB + wq * 64 + (lane & 31);

    fetch();
    put(0);
    fetch();
    put(kWStage);
    fetch();
    float next_start = 0.f;
    if (tid < kWB) {
        start[tid] = start_of(b0);
        next_start = start_of(b0 + 1);
    }
    __syncthreads();
    frags(0, 0);
    int cur = 0, nxt = kWStage, nx2 = 2 * kWStage;

    for (int b = b0; b < b1; ++b) {
        kw_f16v acc[4][2];
        const float* st = start + ((b - b0) & 1) * kWB + wp * 128 + 4 * (lane >> 5);
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const float4 v = *reinterpret_cast<const float4*>(st + m * 32 + g * 8);
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    acc[m][c][4 * g] = v.x;
                    acc[m][c][4 * g + 1] = v.y;
                    acc[m][c][4 * g + 2] = v.z;
                    acc[m][c][4 * g + 3] = v.w;
                }
            }
        if (tid < kWB) {  // that half was read before the last block's barriers
            start[((b + 1 - b0) & 1) * kWB + tid] = next_start;
            next_start = start_of(b + 2);
        }
        for (int s = 0; s < ns; ++s) {
            frags(cur, 1);
#pragma unroll
            for (int m = 0; m < 4; ++m)
#pragma unroll
                for (int c = 0; c < 2; ++c)
                    acc[m][c] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[0][m], fq[0][c], acc[m][c], 0, 0, 0);
            put(nx2);
            fetch();
            frags(nxt, 0);
#pragma unroll
            for (int m = 0; m < 4; ++m)
#pragma unroll
                for (int c = 0; c < 2; ++c)
                    acc[m][c] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[1][m], fq[1][c], acc[m][c], 0, 0, 0);
            __syncthreads();
            const int free = cur;
            cur = nxt;
            nxt = nx2;
            nx2 = free;
        }
        const uint32_t j0 = (uint32_t)b * kWB + wp * 128 + 4 * (lane >> 5);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const uint32_t self = (uint32_t)(q0 + 32 * c) - j0;
            uint32_t top = tid;
            auto empty = [&]() {
                for (uint32_t at = tid; __any(at < top); at += 2 * kWThreads) {
                    const bool in = at < top;
                    const uint32_t o = queue[at + kWThreads];
                    const float v = in && o != self ? __uint_as_float(queue[at]) : -INFINITY;
                    const uint32_t j = j0 + o;
                    bool up[T];
#pragma unroll
                    for (int t = 0; t < T; ++t) up[t] = v > bv[c][t];
#pragma unroll
                    for (int t = T - 1; t > 0; --t) {
                        bv[c][t] = __builtin_amdgcn_fmed3f(v, bv[c][t - 1], bv[c][t]);
                        bj[c][t] = up[t - 1] ? bj[c][t - 1] : (up[t] ? j : bj[c][t]);
                    }
                    bv[c][0] = up[0] ? v : bv[c][0];
                    bj[c][0] = up[0] ? j : bj[c][0];
                }
                top = tid;
            };
#pragma unroll
            for (int m = 0; m < 4; ++m)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
#pragma unroll
                    for (int r = 8 * h; r < 8 * h + 8; ++r) {
                        if (acc[m][c][r] > bv[c][T - 1]) {
                            queue[top] = __float_as_uint(acc[m][c][r]);
                            queue[top + kWThreads] = m * 32 + 8 * (r >> 2) + (r & 3);
                            top += 2 * kWThreads;
                        }
                    }
                    if ((m == 3 && h == 1) || __any(top >= (kWHits - 7) * 2 * kWThreads)) empty();
                }
        }
    }
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int64_t q = q0 + 32 * c;
        if (q >= n) continue;
        uint2* out = cand + (plan.first_list(q - (int64_t)plan.first * kWB) + seg * 4 + wp * 2 + (lane >> 5)) * T;
#pragma unroll
        for (int t = 0; t < T; ++t) out[t] = make_uint2(__float_as_uint(bv[c][t]), bj[c][t]);
    }
}

// Exact f32 distance as the exact kernel forms it (one FMA per coordinate,
// in order); rows whose length is a multiple of 4 are read 16 bytes at a time.
__device__ __forceinline__ float kw_exact(const float* __restrict__ a, const float* __restrict__ b, int32_t d) {
    float acc = 0.f;
    int c = 0;
    if ((d & 3) == 0) {
        const float4* a4 = reinterpret_cast<const float4*>(a);
        const float4* b4 = reinterpret_cast<const float4*>(b);
#pragma unroll 4
        for (int c4 = 0; c4 < d / 4; ++c4) {
            const float4 u = a4[c4], v = b4[c4];
            float t = u.x - v.x;
            acc = fmaf(t, t, acc);
            t = u.y - v.y;
            acc = fmaf(t, t, acc);
            t = u.z - v.z;
            acc = fmaf(t, t, acc);
            t = u.w - v.w;
            acc = fmaf(t, t, acc);
        }
        c = d;
    }
    for (; c < d; ++c) {
        const float t = a[c] - b[c];
        acc = fmaf(t, t, acc);
    }
    return acc;
}

// Bitonic sort of one (v, j) pair per lane across the wavefront, ascending.
__device__ __forceinline__ void kw_wave_sort(float& v, int32_t& j) {
    const int lane = threadIdx.x & 63;
    for (int size = 2; size <= 64; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            const float ov = __shfl_xor(v, stride, 64);
            const int32_t oj = __shfl_xor(j, stride, 64);
            const bool up = (lane & size) == 0;
            const bool lower = (lane & stride) == 0;
            const bool other_less = ov < v || (ov == v && oj < j);
            const bool take = (lower == up) ? other_less : !other_less;
            if (take && !(ov == v && oj == j)) {
                v = ov;
                j = oj;
            }
        }
    }
}

// Unsigned integers in the order of the floats.
__device__ __forceinline__ uint32_t kw_order(float v) {
    const uint32_t b = __float_as_uint(v);
    return b ^ ((b >> 31) ? 0xffffffffu : 0x80000000u);
}

__device__ __forceinline__ float kw_unorder(uint32_t u) {
    return __uint_as_float(u ^ ((u >> 31) ? 0x80000000u : 0xffffffffu));
}

constexpr int kWOwn = kWMaxCand / 64;  // candidates per lane, at most

// The rank-th smallest of the wavefront's keys (rank >= 1, at most their number), bit by bit.
__device__ __forceinline__ uint32_t kw_select(const uint32_t (&key)[kWOwn], int own, int rank) {
    uint32_t res = 0u;
    for (int bit = 31; bit >= 0; --bit) {
        const uint32_t below = res | ((1u << bit) - 1u);  // the bit clear, all lower ones set
        int c = 0;
#pragma unroll
        for (int u = 0; u < kWOwn; ++u)
            if (u < own) c += __popcll(__ballot(key[u] <= below));
        if (c < rank) res |= 1u << bit;
    }
    return res;
}

// One wavefront per query.  Of its lists' candidates only those within twice the
// error bound of the k-th smallest approximate distance can be among the k best;
// their exact distances are formed (at most 64 of them, a lane each), the k best
// written out, and the certificate nu - E_q > d_k checked, nu being the smallest
// approximate distance of anything left out; failures listed.  Exact distances
// read a row of x each: forming all 64 of a query took 2.1 ms at 70 000 x 784,
// this 1.0.
__global__ __launch_bounds__(256) void kw_refine_kernel(const float* __restrict__ x, int64_t n, int32_t d,
                                                       int32_t k, const uint2* __restrict__ cand, KwPlan plan,
                                                       int32_t T, const float* __restrict__ norm2, float m2inv,
                                                       float err_a, float err_b, float err_c, float rel_exact,
                                                       int32_t* __restrict__ idx_out, float* __restrict__ d2_out,
                                                       int32_t* fail_list, unsigned int* fail_count) {
    __shared__ int32_t chosen[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t local = (int64_t)blockIdx.x * 4 + wave, q = (int64_t)plan.first * kWB + local;
    if (q >= n || local >= (int64_t)plan.nq * kWB) return;
    const int total = plan.lists(local) * T, own = (total + 63) / 64;
    const uint2* cq = cand + plan.first_list(local) * T;
    const float nq = norm2[q];
    const float eq = err_a * sqrtf(nq) + err_b * nq + err_c;
    uint32_t key[kWOwn];
    int32_t cj[kWOwn];
    float nu = INFINITY;
#pragma unroll
    for (int u = 0; u < kWOwn; ++u) {
        key[u] = 0xffffffffu;
        cj[u] = INT32_MAX;
        const int c = u * 64 + lane;
        if (u < own && c < total) {
            const uint2 e = cq[c];
            float v = fmaf(m2inv, __uint_as_float(e.x), nq);
            if (!(v <= 3.4028234663852886e38f)) v = INFINITY;  // an empty place, or not a number
            key[u] = kw_order(v);
            cj[u] = (int32_t)e.y;
            if (c % T == T - 1) nu = fminf(nu, v);  // the list may have left out anything from here on
        }
    }
    for (int off = 32; off > 0; off >>= 1) nu = fminf(nu, __shfl_xor(nu, off, 64));
    const float vk = kw_unorder(kw_select(key, own, k));
    float limit = vk + 2.02f * eq + 8.0f * rel_exact * (fabsf(vk) + eq);
    uint32_t klim = kw_order(limit);
    if (!(limit <= 3.4028234663852886e38f)) klim = kw_order(3.4028234663852886e38f);
    int count = 0;
#pragma unroll
    for (int u = 0; u < kWOwn; ++u)
        if (u < own) count += __popcll(__ballot(key[u] <= klim));
    if (count > 64) {  // the 63 smallest, or fewer when some tie there
        klim = kw_select(key, own, 64) - 1u;
        limit = kw_unorder(klim + 1u);
    }
    nu = fminf(nu, limit);
    int32_t* list = chosen[wave];
    int at = 0;
#pragma unroll
    for (int u = 0; u < kWOwn; ++u)
        if (u < own) {
            const bool in = key[u] <= klim;
            const unsigned long long m = __ballot(in);
            if (in) list[at + __popcll(m & ((1ull << lane) - 1ull))] = cj[u];
            at += __popcll(m);
        }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    int32_t j = lane < at ? list[lane] : INT32_MAX;
    float v = INFINITY;
    if (j >= 0 && j < n) v = kw_exact(x + q * d, x + (int64_t)j * d, d);
    else j = INT32_MAX;
    kw_wave_sort(v, j);
    if (lane < k) {
        idx_out[q * k + lane] = j;
        if (d2_out) d2_out[q * k + lane] = v;
    }
    const float dk = __shfl(v, k - 1, 64);
    if (lane == 0) {
        // every other point's approximate distance is >= nu, its real distance
        // >= nu - E_q, its exact f32 distance >= (nu - E_q)(1 - rel_exact)
        if (!((nu - eq) * (1.0f - rel_exact) > dk)) {
            const unsigned int slot = atomicAdd(fail_count, 1u);
            fail_list[slot] = (int32_t)q;
        }
    }
}

// Exact scan for the rows without a certificate.  Block (slice, row) takes
// the points j = slice * per, ... (per = points per slice, at most 8 per lane)
// and writes the k best of them, ascending with ties by index; a second
// kernel merges a row's slices.
constexpr int kScanLane = 8;  // points per lane and slice

__global__ __launch_bounds__(256) void kw_scan_slice_kernel(const float* __restrict__ x, int64_t n, int32_t d,
                                                           int32_t k, int64_t per, int32_t slices,
                                                           const int32_t* __restrict__ rows,
                                                           float* __restrict__ pv, int32_t* __restrict__ pj) {
    __shared__ float sv[4][32];
    __shared__ int32_t sj[4][32];
    const int64_t q = rows[blockIdx.y];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    float bv[kScanLane];
    int32_t bj[kScanLane];
#pragma unroll
    for (int t = 0; t < kScanLane; ++t) {
        bv[t] = INFINITY;
        bj[t] = INT32_MAX;
    }
    const int64_t j0 = (int64_t)blockIdx.x * per, j1 = j0 + per < n ? j0 + per : n;
    for (int64_t j = j0 + threadIdx.x; j < j1; j += 256) {
        if (j == q) continue;
        float out;
        kw_insert<kScanLane>(bv, bj, kw_exact(x + q * d, x + j * d, d), (int32_t)j, out);
    }
    for (int t = 0; t < k; ++t) {
        float v;
        int32_t j;
        kw_pop_min<kScanLane>(bv, bj, v, j);
        if (lane == 0) {
            sv[wave][t] = v;
            sj[wave][t] = j;
        }
    }
    __syncthreads();
    if (wave == 0) {
        // merge the four sorted wavefront lists: lane w < 4 walks list w
        int pos = 0;
        const int64_t o = ((int64_t)blockIdx.y * slices + blockIdx.x) * k;
        for (int t = 0; t < k; ++t) {
            const float hv = (lane < 4 && pos < k) ? sv[lane][pos] : INFINITY;
            const int32_t hj = (lane < 4 && pos < k) ? sj[lane][pos] : INT32_MAX;
            float mv = hv;
            int32_t mj = hj;
            for (int off = 32; off > 0; off >>= 1) {
                const float ov = __shfl_xor(mv, off, 64);
                const int32_t oj = __shfl_xor(mj, off, 64);
                if (ov < mv || (ov == mv && oj < mj)) {
                    mv = ov;
                    mj = oj;
                }
            }
            if (lane < 4 && hj == mj && hv == mv) ++pos;
            if (lane == 0) {
                pv[o + t] = mv;
                pj[o + t] = mj;
            }
        }
    }
}

// One wavefront per rescanned row: lane l keeps the k best of the slices
// l, l + 64, ...; the wavefront then pops the row's k best.
__global__ __launch_bounds__(64) void kw_scan_merge_kernel(int32_t k, int32_t slices,
                                                          const int32_t* __restrict__ rows,
                                                          const float* __restrict__ pv,
                                                          const int32_t* __restrict__ pj,
                                                          int32_t* __restrict__ idx_out,
                                                          float* __restrict__ d2_out) {
    constexpr int KM = 32;
    const int64_t q = rows[blockIdx.x];
    const int lane = threadIdx.x;
    float bv[KM];
    int32_t bj[KM];
#pragma unroll
    for (int t = 0; t < KM; ++t) {
        bv[t] = INFINITY;
        bj[t] = INT32_MAX;
    }
    for (int sl = lane; sl < slices; sl += 64) {
        const int64_t o = ((int64_t)blockIdx.x * slices + sl) * k;
        for (int t = 0; t < k; ++t) {
            float out;
            kw_insert<KM>(bv, bj, pv[o + t], pj[o + t], out);
        }
    }
    for (int t = 0; t < k; ++t) {
        float v;
        int32_t j;
        kw_pop_min<KM>(bv, bj, v, j);
        if (lane == 0) {
            idx_out[q * k + t] = j;
            if (d2_out) d2_out[q * k + t] = v;
        }
    }
}

}  // namespace

namespace gl {

// Wide-feature path of gl_knn; arguments already checked (64 < d <= 4096).
gl_status knn_wide(const float* x, int64_t n, int32_t d, int32_t k, int32_t* idx_out, float* d2_out, size_t limit,
                   hipStream_t s, int64_t* fallback_rows) {
    const int32_t dp = (d + kWStep - 1) / kWStep * kWStep, ns = dp / kWStep;
    const int32_t nblk = (int32_t)((n + kWB - 1) / kWB);
    // A list must not be expected to hold more than T of the nearest points: 16
    // lists of 8 bound what they leave out by about the 50th nearest point, 16 of 12
    // by the 100th.
    const int32_t T = k <= 12 ? 8 : 12;
    const int64_t np = (int64_t)nblk * kWB;
    auto al = [](size_t b) { return (b + 255) & ~(size_t)255; };
    const size_t b_xh = al((size_t)np * dp * 2), b_n = al((size_t)n * 4), b_cn = al((size_t)np * 4),
                 b_f = al((size_t)n * 4);
    const size_t b_mu = al((size_t)d * 4) + al((size_t)kMeanSlices * d * 8);
    // The lists take 1024 or 1536 bytes per query, several times that below 16 384
    // points: where they cannot be had, the query blocks are taken in passes, each
    // half as many as the last try, down to one block.
    char* base = nullptr;
    int32_t step = nblk;
    size_t b_c = 0;
    for (;; step = (step + 1) / 2) {
        b_c = al((size_t)kw_lists(nblk, step) * T * 8);
        const size_t total = b_xh + b_n + b_cn + b_c + b_f + b_mu + 256;
        if (total <= limit && hipMallocAsync((void**)&base, total, s) == hipSuccess) break;
        (void)hipGetLastError();
        base = nullptr;
        if (step == 1) return wfail(GL_E_NOMEM, "temporary device memory for the wide kNN");
    }
    char* p = base;
    kw_h8* xp = (kw_h8*)p;
    p += b_xh;
    float* norm2 = (float*)p;
    p += b_n;
    float* cn = (float*)p;
    p += b_cn;
    uint2* cand = (uint2*)p;
    p += b_c;
    int32_t* fails = (int32_t*)p;
    p += b_f;
    float* mu = (float*)p;
    double* mu_part = (double*)(p + al((size_t)d * 4));
    p += b_mu;
    unsigned int* counters = (unsigned int*)p;  // [0] max |x| bits, [1] max norm bits, [2] failures

    gl_status st = GL_OK;
    hipError_t e = hipMemsetAsync(counters, 0, 12, s);
    unsigned int hc[3] = {0, 0, 0};
    if (e == hipSuccess) {
        hipLaunchKernelGGL(kw_mean_partial_kernel, dim3((unsigned)((d + 255) / 256), kMeanSlices), dim3(256), 0, s,
                           x, n, d, mu_part);
        e = hipGetLastError();
        if (e == hipSuccess) {
            hipLaunchKernelGGL(kw_mean_final_kernel, dim3((unsigned)((d + 255) / 256)), dim3(256), 0, s,
                               (const double*)mu_part, n, d, mu);
            e = hipGetLastError();
        }
    }
    if (e == hipSuccess) {
        hipLaunchKernelGGL(kw_norms_kernel, dim3((unsigned)std::min<int64_t>((n + 3) / 4, 1024)), dim3(256), 0, s, x, (const float*)mu, n,
                           d, norm2, counters);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipMemcpyAsync(hc, counters, 8, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    float amax = 0.f, nmax = 0.f;
    if (e == hipSuccess) {
        std::memcpy(&amax, &hc[0], 4);
        std::memcpy(&nmax, &hc[1], 4);
        if (!std::isfinite(amax) || !std::isfinite(nmax)) st = wfail(GL_E_INVALID_ARG, "x holds a non-finite coordinate");
    }
    // scale by a power of two so that the largest coordinate is in [2^13, 2^14)
    const int ex = amax > 0.f ? 13 - (int)std::floor(std::log2((double)amax)) : 0;
    const double scale = std::ldexp(1.0, ex);
    if (e == hipSuccess && st == GL_OK) {
        const int64_t items = (int64_t)nblk * 8 * ((2 * ns + 3) / 4);
        hipLaunchKernelGGL(kw_pack_kernel, dim3((unsigned)((items + 3) / 4)), dim3(256), 0, s, x, (const float*)mu, n, d,
                           (int64_t)nblk * 8, 2 * ns, (float)scale, xp);
        hipLaunchKernelGGL(kw_start_kernel, dim3((unsigned)nblk), dim3(256), 0, s, (const float*)norm2, n, np,
                           -0.5 * scale * scale, cn);
        e = hipGetLastError();
    }
    // Error of an approximate distance |q|^2 + |p|^2 - 2 <q~, p~> (tilde: f16):
    //   f16 rounding of both factors, |<q~,p~> - <q,p>| <= (2u + u^2) |q| |p|
    //   (u = 2^-11) plus the range below the smallest normal f16 (2^-14, which
    //   the matrix cores may flush to zero), sub = 2^-14 sqrt(d) / scale, times
    //   (|q| + |p|); f32 accumulation over dp terms, which starts from -|p|^2 / 2 (one
    //   ulp, 2^-23, of |q| |p| + |p|^2 / 2 per term at most), the f32 norms and the
    //   final combination: g |q| |p| and g (|q|^2 + |p|^2) with a generous
    //   g = 4 (dp + 8) 2^-24; the f32 rounding of the centring changes a
    //   distance by at most h (|q| + |p|)^2, h = 2^-22.  Norms are those of the
    //   centred points; with |p| <= P:
    //   E_q = A |q| + B |q|^2 + C,  A = 2 (2u + u^2 + g) P + 2 sub + 2 h P,
    //   B = g + h,  C = 2 sub P + (g + h) P^2, each raised by 1 %.
    const double maxn2 = (double)nmax;
    const double P = std::sqrt(maxn2) * (1.0 + 1e-6);
    const double u = std::ldexp(1.0, -11), g = 4.0 * (dp + 8) * std::ldexp(1.0, -24);
    const double sub = std::ldexp(1.0, -14) * std::sqrt((double)d) / scale;
    const double hcen = std::ldexp(1.0, -22);
    const float err_a = (float)(1.01 * (2.0 * (2.0 * u + u * u + g) * P + 2.0 * sub + 2.0 * hcen * P));
    const float err_b = (float)(1.01 * (g + hcen));
    const float err_c = (float)(1.01 * (2.0 * sub * P + (g + hcen) * maxn2));
    // the exact f32 distance (d fused multiply-adds) is within d 2^-24 of the real one, relatively
    const float rel_exact = (float)(1.01 * (d + 2) * std::ldexp(1.0, -24));
    const float m2inv = (float)(-2.0 / (scale * scale));
    for (int32_t first = 0; first < nblk && st == GL_OK && e == hipSuccess; first += step) {
        const KwPlan plan = kw_plan(nblk, first, std::min(step, nblk - first));
        const auto kernel = T == 8 ? kw_tile_kernel<8> : kw_tile_kernel<12>;
        hipLaunchKernelGGL(kernel, dim3(plan.blocks()), dim3(kWThreads), kWLds, s, (const kw_h8*)xp, (const float*)cn, n,
                           ns, plan, cand);
        const int64_t queries = std::min((int64_t)plan.nq * kWB, n - (int64_t)first * kWB);
        hipLaunchKernelGGL(kw_refine_kernel, dim3((unsigned)((queries + 3) / 4)), dim3(256), 0, s, x, n, d, k,
                           (const uint2*)cand, plan, T, (const float*)norm2, m2inv, err_a, err_b, err_c, rel_exact,
                           idx_out, d2_out, fails, counters + 2);
        e = hipGetLastError();
    }
    if (st == GL_OK && e == hipSuccess) e = hipMemcpyAsync(&hc[2], counters + 2, 4, hipMemcpyDeviceToHost, s);
    if (st == GL_OK && e == hipSuccess) e = hipStreamSynchronize(s);
    if (st == GL_OK && e == hipSuccess && hc[2] > 0) {
        const int64_t per = 256 * kScanLane;
        const int32_t slices = (int32_t)((n + per - 1) / per);
        float* pv = nullptr;
        const size_t pb = (size_t)hc[2] * slices * k;
        e = hipMallocAsync((void**)&pv, pb * 8, s);
        if (e == hipSuccess) {
            int32_t* pj = (int32_t*)(pv + pb);
            hipLaunchKernelGGL(kw_scan_slice_kernel, dim3((unsigned)slices, hc[2]), dim3(256), 0, s, x, n, d, k, per,
                               slices, fails, pv, pj);
            e = hipGetLastError();
            if (e == hipSuccess) {
                hipLaunchKernelGGL(kw_scan_merge_kernel, dim3(hc[2]), dim3(64), 0, s, k, slices, fails,
                                   (const float*)pv, (const int32_t*)pj, idx_out, d2_out);
                e = hipGetLastError();
            }
            const hipError_t e2 = hipFreeAsync(pv, s);
            if (e == hipSuccess) e = e2;
        } else {
            st = wfail(GL_E_NOMEM, "temporary device memory for the exact rescan");
        }
    }
    if (fallback_rows) *fallback_rows = hc[2];
    const hipError_t ef = hipFreeAsync(base, s);
    const hipError_t es = hipStreamSynchronize(s);
    if (st != GL_OK) return st;
    if (e != hipSuccess || ef != hipSuccess || es != hipSuccess)
        return wfail(GL_E_HIP, std::string("wide kNN: ") +
                                   hipGetErrorString(e != hipSuccess ? e : (ef != hipSuccess ? ef : es)));
    return GL_OK;
}

}  // namespace gl
