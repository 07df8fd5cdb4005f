// Construction of the window operator (the image graph of Section 2.2) and the
// host side of its power-method pass.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <string>
#include <vector>

#include "gl_fold.hpp"
#include "gl_internal.hpp"
#include "gl_window.hpp"

namespace gl {
namespace {

struct WinAlpha {
    double g[kWinMaxRp + 1];  // normalised patch weights by distance from the centre: alpha_(a,b) = g(|a|) g(|b|)
};

// Colours with a border of rp pixels replicated from the nearest edge pixel,
// channels padded to four: J[(y + rp) * (width + 2 rp) + x + rp] = C(clamp(y), clamp(x)).
__global__ void window_pad_kernel(const float* __restrict__ img, int32_t h, int32_t w, int32_t C, int32_t rp,
                                  float4* __restrict__ J) {
    const int64_t Jw = (int64_t)w + 2 * rp, Jh = (int64_t)h + 2 * rp;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= Jw * Jh) return;
    const int64_t yy = i / Jw, xx = i - yy * Jw;
    const int64_t y = yy - rp < 0 ? 0 : (yy - rp >= h ? h - 1 : yy - rp);
    const int64_t x = xx - rp < 0 ? 0 : (xx - rp >= w ? w - 1 : xx - rp);
    const float* c = img + (y * w + x) * C;
    float4 v;
    v.x = c[0];
    v.y = C > 1 ? c[1] : 0.f;
    v.z = C > 2 ? c[2] : 0.f;
    v.w = C > 3 ? c[3] : 0.f;
    J[i] = v;
}

__device__ __forceinline__ double lane_shift(double x, bool up) {
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    int lo = (int)(uint32_t)u, hi = (int)(uint32_t)(u >> 32);
    if (up) {
        lo = __builtin_amdgcn_update_dpp(0, lo, 0x138, 0xf, 0xf, false);  // wave_shr:1
        hi = __builtin_amdgcn_update_dpp(0, hi, 0x138, 0xf, 0xf, false);
    } else {
        lo = __builtin_amdgcn_update_dpp(0, lo, 0x130, 0xf, 0xf, false);  // wave_shl:1
        hi = __builtin_amdgcn_update_dpp(0, hi, 0x130, 0xf, 0xf, false);
    }
    return __builtin_bit_cast(double, ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

// A wavefront's patch distances: lane l holds column X0 + l of the padded image
// J and rows Y0 .. Y0 + ROWS + 2 RP - 1, so that lanes RP .. 63 - RP form the
// weights of the pixels x = X0 + l - RP, y = Y0 .. Y0 + ROWS - 1 to their
// neighbours at one window offset.  The patch sum is separable: the squared
// colour differences of the lane's column are combined down the rows, then
// across the lanes with wave shifts, so a pair costs about (1 + 2 RP / ROWS)
// colour differences instead of (2 RP + 1)^2.  Everything is double; the sums'
// order is symmetric in the pair, so both of its ends form the same bits.
template <int RP, int ROWS> struct WinPatch {
    static constexpr int JR = ROWS + 2 * RP, OUT = 64 - 2 * RP;  // padded rows; pixels per row
    float4 p[JR];

    __device__ __forceinline__ void load(const float4* __restrict__ J, int64_t Jw, int64_t Jh, int X0, int Y0, int lane) {
        const int64_t jc = min((int64_t)X0 + lane, Jw - 1);
#pragma unroll
        for (int a = 0; a < JR; ++a) p[a] = J[min((int64_t)Y0 + a, Jh - 1) * Jw + jc];
    }

    // sum over the patch for the offset (dy, dx) of every row
    __device__ __forceinline__ void distance(const float4* __restrict__ J, int64_t Jw, int64_t Jh, int X0, int Y0,
                                             int lane, int dy, int dx, bool c4, const WinAlpha& al,
                                             double (&out)[ROWS]) const {
        const int64_t jc = min(max((int64_t)X0 + lane + dx, (int64_t)0), Jw - 1);
        double d[JR];
#pragma unroll
        for (int a = 0; a < JR; ++a) {
            const int64_t jr = min(max((int64_t)Y0 + a + dy, (int64_t)0), Jh - 1);
            const float4 q = J[jr * Jw + jc];
            const double d0 = (double)p[a].x - (double)q.x, d1 = (double)p[a].y - (double)q.y;
            const double d2 = (double)p[a].z - (double)q.z;
            d[a] = (d0 * d0 + d1 * d1) + d2 * d2;
            if (c4) {
                const double d3 = (double)p[a].w - (double)q.w;
                d[a] += d3 * d3;
            }
        }
#pragma unroll
        for (int y = 0; y < ROWS; ++y) {
            double v = al.g[0] * d[y + RP];
#pragma unroll
            for (int k = 1; k <= RP; ++k) v += al.g[k] * (d[y + RP - k] + d[y + RP + k]);
            double s = al.g[0] * v, lo = v, hi = v;
#pragma unroll
            for (int k = 1; k <= RP; ++k) {
                lo = lane_shift(lo, true);
                hi = lane_shift(hi, false);
                s += al.g[k] * (lo + hi);
            }
            out[y] = s;
        }
    }
};

constexpr int kDegRows = 8;   // image rows of a degree workgroup
constexpr int kDegWaves = 8;  // its wavefronts, each taking every eighth window row

// d_p = sum over the window of w_pq in double, and its root: wavefront v of a
// workgroup sums the window rows v, v + 8, .. of its pixels, offsets in order,
// and the eight sums are added in order.  The weights are formed here and again
// by window_fill_kernel rather than kept: their F64 copy was 8 bytes per pixel
// and offset (5.2 GB for a 1024 x 1024 image with the 25 x 25 window), written
// once and read twice, and allocating it cost more than forming them.
template <int RP>
__global__ __launch_bounds__(64 * kDegWaves) void window_degree_kernel(const float4* __restrict__ J, int32_t h, int32_t w,
                                                                       int32_t r, bool c4, WinAlpha al, double inv_s2,
                                                                       double* __restrict__ d, double* __restrict__ root,
                                                                       int32_t* flags, unsigned long long* first_bad) {
    typedef WinPatch<RP, kDegRows> P;
    __shared__ double part[kDegWaves][kDegRows][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int strips = (w + P::OUT - 1) / P::OUT;
    const int64_t block = folded(blockIdx.x, blockIdx.y, gridDim.x);
    if (block >= (int64_t)strips * ((h + kDegRows - 1) / kDegRows)) return;
    const int by = (int)(block / strips), X0 = (int)(block - (int64_t)by * strips) * P::OUT, Y0 = by * kDegRows;
    const int64_t Jw = (int64_t)w + 2 * RP, Jh = (int64_t)h + 2 * RP;
    const int x = X0 + lane - RP;
    const bool col = lane >= RP && lane < 64 - RP && x < w;
    P pt;
    pt.load(J, Jw, Jh, X0, Y0, lane);
    double acc[kDegRows];
#pragma unroll
    for (int y = 0; y < kDegRows; ++y) acc[y] = 0.0;
    for (int dy = wave - r; dy <= r; dy += kDegWaves) {
        if (Y0 + kDegRows - 1 + dy < 0 || Y0 + dy >= h) continue;  // no row of the workgroup has such a neighbour
        for (int dx = -r; dx <= r; ++dx) {
            if (dy == 0 && dx == 0) continue;
            double s[kDegRows];
            pt.distance(J, Jw, Jh, X0, Y0, lane, dy, dx, c4, al, s);
            const bool in = col && x + dx >= 0 && x + dx < w;
#pragma unroll
            for (int y = 0; y < kDegRows; ++y) {
                const int qy = Y0 + y + dy;
                const double wgt = exp(-s[y] * inv_s2);
                if (in && qy >= 0 && qy < h) acc[y] += wgt;
            }
        }
    }
#pragma unroll
    for (int y = 0; y < kDegRows; ++y) part[wave][y][lane] = acc[y];
    __syncthreads();
    // wavefront v finishes row v
    const int y = Y0 + wave;
    if (!col || y >= h) return;
    double s = 0.0;
#pragma unroll
    for (int v = 0; v < kDegWaves; ++v) s += part[v][wave][lane];
    const int64_t p = (int64_t)y * w + x;
    d[p] = s;
    root[p] = sqrt(s);
    if (!(s > 0.0) || !(s <= 1.7976931348623157e308)) {
        atomicOr(flags, (int32_t)BAD_DEGREE);
        atomicMin(first_bad, (unsigned long long)p);
    }
}

// Stored weights: what_pq = w_pq / (sqrt(d_p) sqrt(d_q)) (raw = 0) or w_pq (raw !=
// 0), rounded once to TW, for the first half of each pixel's window: a
// wavefront per 4 image rows x OUT columns and vector of GS offsets.  Ragged
// tiles' lanes outside the image, offsets outside it and padding store 0.
template <int RP, typename TW>
__global__ __launch_bounds__(256) void window_fill_kernel(const float4* __restrict__ J, const double* __restrict__ root,
                                                          int32_t h, int32_t w, int32_t r, int32_t tiles_x, int32_t M,
                                                          bool c4, WinAlpha al, double inv_s2, int32_t raw_mode,
                                                          u32x4* __restrict__ out) {
    typedef WinPatch<RP, kWinTY> P;
    constexpr int GS = 16 / (int)sizeof(TW);
    const int ng = window_groups(M, GS), side = 2 * r + 1;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int g = (int)blockIdx.y * 4 + wave;
    if (g >= ng) return;
    const int strips = (tiles_x * kWinTX + P::OUT - 1) / P::OUT;
    const int64_t block = folded(blockIdx.x, blockIdx.z, gridDim.x);
    if (block >= (int64_t)strips * ((h + kWinTY - 1) / kWinTY)) return;
    const int ty = (int)(block / strips), X0 = (int)(block - (int64_t)ty * strips) * P::OUT, Y0 = ty * kWinTY;
    const int64_t Jw = (int64_t)w + 2 * RP, Jh = (int64_t)h + 2 * RP;
    const int x = X0 + lane - RP;
    const bool col = x < w;
    P pt;
    pt.load(J, Jw, Jh, X0, Y0, lane);
    double rp_[kWinTY];
#pragma unroll
    for (int y = 0; y < kWinTY; ++y)
        rp_[y] = col && x >= 0 && Y0 + y < h ? root[(int64_t)(Y0 + y) * w + x] : 1.0;
    // the vector of a pixel is shifted in from the top, one weight at a time
    u32x4 v[kWinTY];
#pragma unroll
    for (int y = 0; y < kWinTY; ++y) v[y] = u32x4{0u, 0u, 0u, 0u};
    for (int e = 0; e < GS; ++e) {
        const int m = g * GS + e;
        const int dy = m / side - r, dx = m - (m / side) * side - r;  // the cell index of the scan equals m
        double s[kWinTY];
        const bool live = m < M / 2;
        if (live) pt.distance(J, Jw, Jh, X0, Y0, lane, dy, dx, c4, al, s);
        const bool in = live && col && x >= 0 && x + dx >= 0 && x + dx < w;
#pragma unroll
        for (int y = 0; y < kWinTY; ++y) {
            const int qy = Y0 + y + dy;
            double o = 0.0;
            if (in && Y0 + y < h && qy >= 0) {
                o = exp(-s[y] * inv_s2);
                if (!raw_mode && o != 0.0) o = o / (rp_[y] * root[(int64_t)qy * w + x + dx]);
            }
            const TW q = store_as<TW>::from(o);
            if constexpr (sizeof(TW) == 8) {
                uint64_t b;
                __builtin_memcpy(&b, &q, 8);
                v[y] = u32x4{v[y].z, v[y].w, (uint32_t)b, (uint32_t)(b >> 32)};
            } else if constexpr (sizeof(TW) == 4) {
                uint32_t b;
                __builtin_memcpy(&b, &q, 4);
                v[y] = u32x4{v[y].y, v[y].z, v[y].w, b};
            } else {
                uint16_t b;
                __builtin_memcpy(&b, &q, 2);
                v[y] = u32x4{(v[y].x >> 16) | (v[y].y << 16), (v[y].y >> 16) | (v[y].z << 16),
                             (v[y].z >> 16) | (v[y].w << 16), (v[y].w >> 16) | ((uint32_t)b << 16)};
            }
        }
    }
    if (lane < RP || lane >= 64 - RP || x >= tiles_x * kWinTX) return;
    const int64_t tile = (int64_t)ty * tiles_x + x / kWinTX;
#pragma unroll
    for (int y = 0; y < kWinTY; ++y) out[(tile * ng + g) * 256 + y * kWinTX + x % kWinTX] = v[y];
}

// Unnormalized L: diagonal dd_p = sum of the stored weights of p's whole window
// (double, offset order: the first half from p's vectors, the second half
// from the neighbours', which keep the weight of the mirrored offset),
// rounded to the accumulator type A.
template <typename TW, typename A>
__global__ __launch_bounds__(256) void window_rowsum_kernel(const TW* __restrict__ wst, int32_t h, int32_t w,
                                                            int32_t r, int32_t tiles_x, int32_t M,
                                                            A* __restrict__ dd) {
    constexpr int GS = 16 / (int)sizeof(TW);
    const int64_t b = blockIdx.x;
    const int ty = (int)(b / tiles_x), tx = (int)(b - (int64_t)ty * tiles_x);
    const int x = tx * kWinTX + (threadIdx.x & 63), y = ty * kWinTY + (threadIdx.x >> 6);
    if (x >= w || y >= h) return;
    const int ng = window_groups(M, GS), side = 2 * r + 1;
    auto stored = [&](int qy, int qx, int m) {
        const int64_t qb = (int64_t)(qy / kWinTY) * tiles_x + qx / kWinTX;
        const int ql = (qy % kWinTY) * kWinTX + qx % kWinTX;
        return cvt<double>(wst[((qb * ng + m / GS) * 256 + ql) * GS + m % GS]);
    };
    double s = 0.0;
    for (int m = 0; m < M; ++m) {
        if (m < M / 2) {
            s += stored(y, x, m);
        } else {
            const int cell = m + 1;
            const int qy = y + cell / side - r, qx = x + cell % side - r;
            if (qy < h && qx >= 0 && qx < w) s += stored(qy, qx, M - 1 - m);
        }
    }
    dd[(int64_t)y * w + x] = (A)s;
}

// Patch radius and colours, and what the two passes over the weights need.
struct WinBuild {
    const float4* J;
    const double* root;
    int32_t rp;
    bool c4;
    WinAlpha al;
    double inv_s2;
};

template <int RP>
hipError_t launch_degree_t(const WinBuild& b, const gl_operator* op, double* root, int32_t* flags,
                           unsigned long long* first_bad, hipStream_t s) {
    constexpr int out = WinPatch<RP, kDegRows>::OUT;
    const Fold f = fold_blocks((int64_t)((op->wwidth + out - 1) / out) * ((op->wheight + kDegRows - 1) / kDegRows));
    hipLaunchKernelGGL(window_degree_kernel<RP>, dim3(f.x, f.y), dim3(64 * kDegWaves), 0, s, b.J, op->wheight, op->wwidth, op->wr,
                       b.c4, b.al, b.inv_s2, op->degree, root, flags, first_bad);
    return hipGetLastError();
}

template <int RP, typename TW>
hipError_t launch_fill_t(const WinBuild& b, const gl_operator* op, int raw_mode, hipStream_t s) {
    constexpr int GS = 16 / (int)sizeof(TW), out = WinPatch<RP, kWinTY>::OUT;
    const int tiles_y = (op->wheight + kWinTY - 1) / kWinTY;
    const int strips = (op->wtiles_x * kWinTX + out - 1) / out;
    // a narrow image of 2^25 rows has two strips of 2^23 workgroups: 2^32 threads
    const Fold f = fold_blocks((int64_t)strips * tiles_y);
    const dim3 grid(f.x, (unsigned)((window_groups(op->wM, GS) + 3) / 4), f.y);
    hipLaunchKernelGGL((window_fill_kernel<RP, TW>), grid, dim3(256), 0, s, b.J, b.root, op->wheight, op->wwidth, op->wr,
                       op->wtiles_x, op->wM, b.c4, b.al, b.inv_s2, raw_mode, (u32x4*)op->w);
    return hipGetLastError();
}

template <int RP>
hipError_t launch_fill(const WinBuild& b, const gl_operator* op, int raw_mode, hipStream_t s) {
    switch (op->store_w) {
        case GL_F64: return launch_fill_t<RP, double>(b, op, raw_mode, s);
        case GL_F32: return launch_fill_t<RP, float>(b, op, raw_mode, s);
        case GL_BF16: return launch_fill_t<RP, bf16>(b, op, raw_mode, s);
        default: return launch_fill_t<RP, f16>(b, op, raw_mode, s);
    }
}

template <typename TW, typename A>
hipError_t launch_rowsum_t(const gl_operator* op, hipStream_t s) {
    hipLaunchKernelGGL((window_rowsum_kernel<TW, A>), dim3((unsigned)op->nblocks), dim3(256), 0, s,
                       (const TW*)op->w, op->wheight, op->wwidth, op->wr, op->wtiles_x, op->wM, (A*)op->dd);
    return hipGetLastError();
}

size_t wdtype_size(gl_dtype d) {
    switch (d) {
        case GL_F64: return 8;
        case GL_F32: return 4;
        case GL_BF16:
        case GL_F16: return 2;
    }
    return 0;
}

gl_status wfail(gl_status st, const std::string& msg) {
    set_last_error(msg);
    return st;
}

}  // namespace

size_t window_lds_bytes(const gl_operator* op, int K, size_t acc) {
    return 2 * (size_t)K * window_region(op->wr) * acc;
}

size_t window_part_bytes(const gl_operator* op, int K, size_t acc) {
    if (op->layout != LAYOUT_WINDOW) return 0;
    return (size_t)op->nblocks * window_region(op->wr) * K * acc;
}

template <typename TW>
static void window_power_t(const WinPowerArgs& a, const gl_operator* op, hipStream_t s) {
    WinPartArgs<float> pa;
    pa.op = a.op;
    pa.v = a.x;
    pa.part = const_cast<float*>(a.part);
    const dim3 grid((unsigned)op->nblocks), block(256);
    hipLaunchKernelGGL((window_part_kernel<1, TW, float>), grid, block, window_lds_bytes(op, 1, 4), s, pa);
    hipLaunchKernelGGL(window_power_kernel<TW>, grid, block, 0, s, a);
}

hipError_t launch_window_power(const gl_operator* op, const float* x, float* y, int mode, float gain, const float* scale,
                               float* partials, float* part, hipStream_t s) {
    WinPowerArgs a;
    a.op.w = op->w;
    a.op.height = op->wheight;
    a.op.width = op->wwidth;
    a.op.r = op->wr;
    a.op.M = op->wM;
    a.op.tiles_x = op->wtiles_x;
    a.part = part;
    a.x = x;
    a.y = y;
    a.scale = scale;
    a.partials = partials;
    a.dd = (const float*)op->dd;
    a.mode = mode;
    a.gain = gain;
    switch (op->store_w) {
        case GL_F32: window_power_t<float>(a, op, s); break;
        case GL_BF16: window_power_t<bf16>(a, op, s); break;
        case GL_F16: window_power_t<f16>(a, op, s); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace gl

extern "C" gl_status gl_window_operator_create(const gl_window_graph* g, gl_dtype store_w, void* stream,
                                               gl_operator** out) {
    using namespace gl;
    if (!g || !out) return wfail(GL_E_INVALID_ARG, "graph and out must not be NULL");
    *out = nullptr;
    if (!g->image) return wfail(GL_E_INVALID_ARG, "image must not be NULL");
    if (((uintptr_t)g->image) % 4) return wfail(GL_E_INVALID_ARG, "image must be 4-byte aligned");
    if (g->height < 1 || g->width < 1 || (int64_t)g->height * g->width >= ((int64_t)1 << 31))
        return wfail(GL_E_INVALID_ARG, "height and width must be >= 1 with height * width < 2^31");
    if (g->channels < 1 || g->channels > 4) return wfail(GL_E_INVALID_ARG, "channels must lie in [1, 4]");
    if (g->window_radius < 1 || g->window_radius > kWinMaxR)
        return wfail(GL_E_INVALID_ARG, "window_radius must lie in [1, 27]");
    if (g->patch_radius < 0 || g->patch_radius > kWinMaxRp)
        return wfail(GL_E_INVALID_ARG, "patch_radius must lie in [0, 4]");
    if (!(g->sigma > 0.0) || !std::isfinite(g->sigma)) return wfail(GL_E_INVALID_ARG, "sigma must be finite and > 0");
    if (g->laplacian != GL_LAP_NORMALIZED && g->laplacian != GL_LAP_UNNORMALIZED)
        return wfail(GL_E_INVALID_ARG, "unknown laplacian");
    if (g->reserved != 0) return wfail(GL_E_INVALID_ARG, "reserved must be 0");
    if (wdtype_size(store_w) == 0) return wfail(GL_E_DTYPE, "unknown weight storage type");
    hipStream_t s = (hipStream_t)stream;

    const int32_t h = g->height, w = g->width, r = g->window_radius, rp = g->patch_radius;
    const int32_t side = 2 * r + 1, M = side * side - 1;
    const int32_t tiles_x = (w + kWinTX - 1) / kWinTX, tiles_y = (h + kWinTY - 1) / kWinTY;
    const int64_t ntiles = (int64_t)tiles_x * tiles_y;
    const int64_t n = (int64_t)h * w;
    const int GS = 16 / (int)wdtype_size(store_w);
    const int64_t stored = ntiles * 256 * window_groups(M, GS) * GS;  // first half of each window, padded

    gl_operator* op = new gl_operator();
    op->n = n;
    op->store_w = store_w;
    op->layout = LAYOUT_WINDOW;
    op->lap = g->laplacian;
    op->G = 1;
    op->wheight = h;
    op->wwidth = w;
    op->wr = r;
    op->wM = M;
    op->wtiles_x = tiles_x;
    op->nblocks = ntiles;
    op->stored = stored;
    // edges: the window clipped to the image, minus the pixel itself
    int64_t sy = 0, sx = 0;
    for (int32_t y = 0; y < h; ++y) sy += std::min(y + r, h - 1) - std::max(y - r, 0) + 1;
    for (int32_t x = 0; x < w; ++x) sx += std::min(x + r, w - 1) - std::max(x - r, 0) + 1;
    op->nnz = sy * sx - n;
    (void)hipGetDevice(&op->device);

    // patch weights: separable Gaussian normalised to sum 1
    WinBuild build = {};
    build.rp = rp;
    build.c4 = g->channels == 4;
    build.inv_s2 = 1.0 / (g->sigma * g->sigma);
    {
        double gs = 0.0;
        for (int t = 0; t <= rp; ++t) {
            build.al.g[t] = rp > 0 ? std::exp(-(double)t * t / (2.0 * rp * rp)) : 1.0;
            gs += (t ? 2.0 : 1.0) * build.al.g[t];
        }
        for (int t = 0; t <= rp; ++t) build.al.g[t] /= gs;
    }

    const size_t wbytes = (size_t)stored * wdtype_size(store_w);
    const size_t Jn = (size_t)(h + 2 * rp) * (size_t)(w + 2 * rp);
    float4* J = nullptr;
    double* root = nullptr;  // sqrt of the degrees
    int32_t* flags = nullptr;
    std::string what;
    hipError_t e = hipMalloc(&op->w, wbytes);
    if (e == hipSuccess) e = hipMalloc((void**)&op->degree, (size_t)n * 8);
    if (e == hipSuccess) e = hipMalloc((void**)&J, Jn * sizeof(float4));
    if (e == hipSuccess) e = hipMalloc((void**)&root, (size_t)n * 8);
    if (e == hipSuccess) e = hipMalloc((void**)&flags, 16);
    if (e != hipSuccess) {
        (void)hipFree(J);
        (void)hipFree(root);
        (void)hipFree(flags);
        gl_operator_destroy(op);
        (void)hipGetLastError();
        return wfail(GL_E_NOMEM, "device allocation for the window operator failed");
    }
    op->bytes = wbytes + (size_t)n * 8;
    unsigned long long* first_bad = (unsigned long long*)(flags + 2);
    const unsigned long long none = ~0ull;
    int32_t hflags[4] = {0, 0, 0, 0};
    __builtin_memcpy(&hflags[2], &none, 8);

    e = hipMemcpyAsync(flags, hflags, 16, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(window_pad_kernel, dim3((unsigned)((Jn + 255) / 256)), dim3(256), 0, s, g->image, h, w,
                           g->channels, rp, J);
        e = hipGetLastError();
    }
    build.J = J;
    build.root = root;
    if (e == hipSuccess) {
        switch (rp) {
            case 0: e = launch_degree_t<0>(build, op, root, flags, first_bad, s); break;
            case 1: e = launch_degree_t<1>(build, op, root, flags, first_bad, s); break;
            case 2: e = launch_degree_t<2>(build, op, root, flags, first_bad, s); break;
            case 3: e = launch_degree_t<3>(build, op, root, flags, first_bad, s); break;
            default: e = launch_degree_t<4>(build, op, root, flags, first_bad, s); break;
        }
    }
    if (e == hipSuccess) e = hipMemcpyAsync(hflags, flags, 16, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    gl_status st = GL_OK;
    if (e != hipSuccess) {
        st = wfail(GL_E_HIP, std::string("window weights: ") + hipGetErrorString(e));
    } else if (hflags[0]) {
        unsigned long long bad = 0;
        __builtin_memcpy(&bad, &hflags[2], 8);
        st = wfail(GL_E_BAD_GRAPH, "window graph: pixel (" + std::to_string(bad / (unsigned long long)w) + ", " +
                                       std::to_string(bad % (unsigned long long)w) +
                                       ") has degree 0 (no neighbour, or every weight underflows)");
    }
    if (st == GL_OK) {
        const int raw_mode = op->lap == GL_LAP_UNNORMALIZED ? 1 : 0;
        switch (rp) {
            case 0: e = launch_fill<0>(build, op, raw_mode, s); break;
            case 1: e = launch_fill<1>(build, op, raw_mode, s); break;
            case 2: e = launch_fill<2>(build, op, raw_mode, s); break;
            case 3: e = launch_fill<3>(build, op, raw_mode, s); break;
            default: e = launch_fill<4>(build, op, raw_mode, s); break;
        }
        if (e == hipSuccess && raw_mode) {
            const size_t es = store_w == GL_F64 ? 8 : 4;
            e = hipMalloc(&op->dd, (size_t)n * es);
            if (e == hipSuccess) {
                op->bytes += (size_t)n * es;
                switch (store_w) {
                    case GL_F64: e = launch_rowsum_t<double, double>(op, s); break;
                    case GL_F32: e = launch_rowsum_t<float, float>(op, s); break;
                    case GL_BF16: e = launch_rowsum_t<bf16, float>(op, s); break;
                    default: e = launch_rowsum_t<f16, float>(op, s); break;
                }
            }
            double mx = 0.0;
            bool bad = false;
            if (e == hipSuccess) e = check_diagonal(op->dd, es == 8, n, flags, s, mx, bad);
            if (e == hipSuccess && bad)
                st = wfail(GL_E_BAD_GRAPH, "window graph: a stored row sums to a non-positive degree");
            op->dmax = mx;
        }
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess && st == GL_OK) st = wfail(GL_E_HIP, std::string("window fill: ") + hipGetErrorString(e));
    }
    (void)hipStreamSynchronize(s);
    (void)hipFree(J);
    (void)hipFree(root);
    (void)hipFree(flags);
    if (st != GL_OK) {
        gl_operator_destroy(op);
        return st;
    }
    *out = op;
    return GL_OK;
}
