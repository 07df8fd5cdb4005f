// Second eigenpair of the operator's Laplacian, the start of the unsupervised
// runs (Section 5.2 initialises them with the second eigenvector of the
// normalized graph Laplacian).
//
// Lanczos with full reorthogonalisation on the operator's own sparse product,
// deflated against the known null vector (D^{1/2} 1 for L_s, 1 for L):
//   q_0 = x_0 - (z.x_0) z, normalised; for j = 0 .. m-1:
//   w = L q_j; alpha_j = q_j.w; w -= [z, q_0 .. q_j] c twice (classical
//   Gram-Schmidt, c = [z, q_0 .. q_j]^T w); beta_j = |w|; q_{j+1} = w / beta_j.
// The smallest eigenpair (theta, y) of the tridiagonal T_m (bisection on the
// Sturm count, then inverse iteration) gives the Ritz vector x = Q y; the run
// restarts from x until |L x - theta x| <= tol.  Vectors are float in the
// operator's position order; every inner product is summed in double in a
// fixed order, so results are reproducible.
//
// A step is six launches (product, twice inner products and subtraction,
// normalisation) and no copy: alpha and beta stay on the device until the m
// steps are queued.  At 20 000 rows the vectors are a few MB and a launch is
// bound by its latency, so the inner products are spread over row tiles of 256
// and groups of 32 vectors (237 workgroups; a workgroup per 2048 rows looping
// over the vectors took 19 us of a step's 240), and the subtraction's
// workgroups add up the tiles' partial sums themselves.  64 steps on 20 011 rows:
// 15.4 ms before, 1.9 to 2.0 so.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <string>
#include <vector>

#include "gl_internal.hpp"
#include "gl_kernels.hpp"

namespace gl {

// z_p = sqrt(d_i) (L_s) or 1 (L), i the node of position p.
__global__ void null_vector_kernel(int64_t n, const double* __restrict__ degree, const int32_t* __restrict__ order,
                                   int32_t normalized, float* __restrict__ z) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const int64_t i = order ? (int64_t)order[p] : p;
    z[p] = normalized ? (float)sqrt(degree[i]) : 1.0f;
}

// Rows of one tile: a wavefront covers it with R float4 per lane.
template <int R> constexpr int tile_rows() { return 256 * R; }

// A lane's rows of a vector of n floats (16-byte aligned, readable up to the
// next multiple of 64): rows base + 256 r + 4 lane .. + 3; zero beyond n.
template <int R>
__device__ __forceinline__ void load_tile(const float* __restrict__ v, int64_t base, int64_t n, int lane,
                                          float4 (&out)[R]) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t i = base + 256 * r + 4 * lane;
        float4 x = {0.f, 0.f, 0.f, 0.f};
        if (i < n) {
            x = *reinterpret_cast<const float4*>(v + i);
            if (i + 1 >= n) x.y = 0.f;
            if (i + 2 >= n) x.z = 0.f;
            if (i + 3 >= n) x.w = 0.f;
        }
        out[r] = x;
    }
}

constexpr int kDotVecs = 8;  // vectors per wavefront

// partials[j * nb + b] = V_j . w over the rows of tile b, for the cnt vectors V_j =
// V + j * ldv: four groups of kDotVecs vectors per workgroup (one per wavefront).
template <int R>
__global__ __launch_bounds__(kBlock) void dots_kernel(int64_t n, const float* __restrict__ V, int64_t ldv, int32_t cnt,
                                                      const float* __restrict__ w, double* __restrict__ partials,
                                                      int64_t nb) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t b = blockIdx.x, base = b * tile_rows<R>();
    float4 wv[R];
    load_tile<R>(w, base, n, lane, wv);
    const int j0 = ((int)blockIdx.y * 4 + wave) * kDotVecs;
#pragma unroll
    for (int u = 0; u < kDotVecs; ++u) {
        const int j = j0 + u;
        if (j >= cnt) break;
        float4 v[R];
        load_tile<R>(V + (int64_t)j * ldv, base, n, lane, v);
        double acc = 0.0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            acc += (double)v[r].x * (double)wv[r].x;
            acc += (double)v[r].y * (double)wv[r].y;
            acc += (double)v[r].z * (double)wv[r].z;
            acc += (double)v[r].w * (double)wv[r].w;
        }
        acc = wave_sum63(acc);
        if (lane == 63) partials[(int64_t)j * nb + b] = acc;
    }
}

// out[j] = sum of partials[j * nb .. j * nb + nb) in a fixed order (block j).
__global__ __launch_bounds__(kBlock) void sum_partials_kernel(const double* __restrict__ partials, int64_t nb,
                                                              double* __restrict__ out) {
    const double v = block_sum(partials + (int64_t)blockIdx.x * nb, nb);
    if (threadIdx.x == 0) out[blockIdx.x] = v;
}

constexpr int64_t kSumTiles = 8192;
constexpr int kMaxVecs = 514;  // z and up to 513 Lanczos vectors

// out = w - sum_j c_j V_j (or + sum_j c_j V_j where w is NULL) over the rows of
// tile b, sums in double; c_j = sum of coef[j * nc .. j * nc + nc) in a fixed
// order.  norm[b] = the tile's |out|^2.  keep: receives c_{cnt-1} (or NULL).
// Wavefront v takes the vectors v, v + 4, ..; the four sums are added in order.
template <int R>
__global__ __launch_bounds__(kBlock) void combine_kernel(int64_t n, const float* __restrict__ V, int64_t ldv,
                                                         int32_t cnt, const double* __restrict__ coef, int32_t nc,
                                                         const float* w, float* out, double* __restrict__ norm,
                                                         double* __restrict__ keep) {
    __shared__ double c[kMaxVecs];
    __shared__ double part[4][tile_rows<R>()];
    __shared__ double sn[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t b = blockIdx.x, base = b * tile_rows<R>();
    // eight lanes per coefficient
    for (int j = threadIdx.x >> 3; j < (cnt + 31) / 32 * 32; j += kBlock / 8) {
        double s = 0.0;
        if (j < cnt)
#pragma unroll 8
            for (int i = threadIdx.x & 7; i < nc; i += 8) s += coef[(int64_t)j * nc + i];
        s += xor_partner<1>(s);
        s += xor_partner<2>(s);
        s += xor_partner<4>(s);
        if (j < cnt && (threadIdx.x & 7) == 0) c[j] = s;
    }
    __syncthreads();
    if (keep && b == 0 && threadIdx.x == 0) *keep = c[cnt - 1];
    double acc[R][4];
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r][0] = acc[r][1] = acc[r][2] = acc[r][3] = 0.0;
#pragma unroll 4
    for (int j = wave; j < cnt; j += 4) {
        float4 v[R];
        load_tile<R>(V + (int64_t)j * ldv, base, n, lane, v);
        const double cj = c[j];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            acc[r][0] += cj * (double)v[r].x;
            acc[r][1] += cj * (double)v[r].y;
            acc[r][2] += cj * (double)v[r].z;
            acc[r][3] += cj * (double)v[r].w;
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int e = 0; e < 4; ++e) part[wave][256 * r + 4 * lane + e] = acc[r][e];
    __syncthreads();
    double sq = 0.0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int at = 256 * r + (int)threadIdx.x;
        const int64_t i = base + at;
        if (i < n) {
            const double s = ((part[0][at] + part[1][at]) + part[2][at]) + part[3][at];
            const float o = (float)(w ? (double)w[i] - s : s);
            out[i] = o;
            sq += (double)o * (double)o;
        }
    }
    sq = wave_sum63(sq);
    if (lane == 63) sn[wave] = sq;
    __syncthreads();
    if (threadIdx.x == 0) norm[b] = ((sn[0] + sn[1]) + sn[2]) + sn[3];
}

// y = x / |x|, |x|^2 = the sum of norm[0 .. nb) in a fixed order; length (or
// NULL) receives |x|.
__global__ __launch_bounds__(kBlock) void normalise_kernel(int64_t n, const float* __restrict__ x, float* __restrict__ y,
                                                           const double* __restrict__ norm, int64_t nb,
                                                           double* __restrict__ length) {
    const double len = sqrt(block_sum(norm, nb));
    const double s = 1.0 / len;
    if (length && blockIdx.x == 0 && threadIdx.x == 0) *length = len;
    const int64_t i = ((int64_t)blockIdx.x * kBlock + threadIdx.x) * 4;
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (i + e < n) y[i + e] = (float)((double)x[i + e] * s);
}

// Largest |x_i| of tile b (256 rows) and the lowest i that has it.
__global__ __launch_bounds__(kBlock) void argmax_kernel(int64_t n, const float* __restrict__ x, float* __restrict__ best,
                                                        int64_t* __restrict__ where) {
    __shared__ float sv[kBlock];
    __shared__ int32_t si[kBlock];
    const int t = threadIdx.x;
    const int64_t i = (int64_t)blockIdx.x * kBlock + t;
    sv[t] = i < n ? fabsf(x[i]) : -1.0f;
    si[t] = t;
    __syncthreads();
    for (int off = kBlock / 2; off > 0; off >>= 1) {
        if (t < off && (sv[t + off] > sv[t] || (sv[t + off] == sv[t] && si[t + off] < si[t]))) {
            sv[t] = sv[t + off];
            si[t] = si[t + off];
        }
        __syncthreads();
    }
    if (t == 0) {
        best[blockIdx.x] = sv[0];
        where[blockIdx.x] = (int64_t)blockIdx.x * kBlock + si[0];
    }
}

// sign[0] = -1 where the first entry of largest magnitude is negative, else 1.
__global__ __launch_bounds__(kBlock) void sign_kernel(const float* __restrict__ x, const float* __restrict__ best,
                                                      const int64_t* __restrict__ where, int64_t nb,
                                                      float* __restrict__ sign) {
    __shared__ float sv[kBlock];
    __shared__ int64_t si[kBlock];
    const int t = threadIdx.x;
    float v = -1.0f;
    int64_t at = INT64_MAX;
    for (int64_t b = t; b < nb; b += kBlock)
        if (best[b] > v) {
            v = best[b];
            at = where[b];
        }
    sv[t] = v;
    si[t] = at;
    __syncthreads();
    for (int off = kBlock / 2; off > 0; off >>= 1) {
        if (t < off && (sv[t + off] > sv[t] || (sv[t + off] == sv[t] && si[t + off] < si[t]))) {
            sv[t] = sv[t + off];
            si[t] = si[t + off];
        }
        __syncthreads();
    }
    if (t == 0) sign[0] = si[0] < INT64_MAX && x[si[0]] < 0.0f ? -1.0f : 1.0f;
}

// y = sign x at the node of each position.
__global__ void output_kernel(int64_t n, const float* __restrict__ x, float* __restrict__ y,
                              const float* __restrict__ sign, const int32_t* __restrict__ order) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    y[order ? (int64_t)order[i] : i] = sign[0] * x[i];
}

// y = x gathered from node order into position order.
__global__ void gather_kernel(int64_t n, const float* __restrict__ x, const int32_t* __restrict__ order,
                              float* __restrict__ y) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    y[p] = x[order ? (int64_t)order[p] : p];
}

// r = w - theta x.
__global__ void residual_kernel(int64_t n, const float* __restrict__ w, const float* __restrict__ x, double theta,
                                float* __restrict__ r) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    r[i] = (float)((double)w[i] - theta * (double)x[i]);
}

}  // namespace gl

namespace {

gl_status efail(gl_status st, const std::string& m) {
    gl::set_last_error(m);
    return st;
}

size_t al256(size_t b) { return (b + 255) & ~(size_t)255; }

struct EigWs {
    int64_t ldv = 0, nb = 0;     // vector pitch; row tiles
    int R = 1;                   // float4 per lane and tile
    float* z = nullptr;          // null vector (unit), followed by
    float* Q = nullptr;          // [m + 1] Lanczos vectors
    float* w = nullptr;
    float* x = nullptr;
    double* partials = nullptr;  // [(m + 2) * nb]
    double* norm = nullptr;      // [nb]
    double* sums = nullptr;      // [m + 2]
    double* out = nullptr;       // alpha [m], beta [m], |x|^2 before and after, |residual|^2
    double* y = nullptr;         // [m]
    float* best = nullptr;       // [rows / 256], the sign, and their places
    int64_t* where = nullptr;
    float* wpart = nullptr;      // window layout: region sums of one product
    size_t bytes = 0;
};

EigWs carve(const gl_operator* op, int32_t m, char* base) {
    EigWs e;
    e.ldv = (op->n + 63) / 64 * 64;
    // small tiles while the workgroups of the subtraction can add up their partial sums
    e.R = op->n <= 256 * 128 ? 1 : 4;
    e.nb = (op->n + 256 * e.R - 1) / (256 * e.R);
    const size_t vec = al256((size_t)e.ldv * 4), nm = (size_t)((op->n + gl::kBlock - 1) / gl::kBlock);
    size_t o = 0;
    auto take = [&](size_t b) {
        char* p = base ? base + o : nullptr;
        o += al256(b);
        return p;
    };
    e.z = (float*)take((size_t)(m + 2) * e.ldv * 4);
    e.Q = e.z ? e.z + e.ldv : nullptr;
    e.w = (float*)take(vec);
    e.x = (float*)take(vec);
    e.partials = (double*)take((size_t)(m + 2) * e.nb * 8);
    e.norm = (double*)take((size_t)e.nb * 8);
    e.sums = (double*)take((size_t)(m + 2) * 8);
    e.out = (double*)take((size_t)(2 * m + 4) * 8);
    e.y = (double*)take((size_t)m * 8);
    e.best = (float*)take((nm + 1) * 4);
    e.where = (int64_t*)take(nm * 8);
    e.wpart = (float*)take(gl::window_part_bytes(op, 1, 4));
    e.bytes = o;
    return e;
}

// Smallest eigenpair of the symmetric tridiagonal matrix (a, b): bisection on
// the Sturm count for the eigenvalue, inverse iteration for the unit eigenvector.
void tridiag_smallest(const std::vector<double>& a, const std::vector<double>& b, double& theta,
                      std::vector<double>& y) {
    const int m = (int)a.size();
    double lo = a[0], hi = a[0];
    for (int i = 0; i < m; ++i) {
        const double r = (i > 0 ? std::fabs(b[i - 1]) : 0.0) + (i + 1 < m ? std::fabs(b[i]) : 0.0);
        lo = std::min(lo, a[i] - r);
        hi = std::max(hi, a[i] + r);
    }
    const double scale = std::max(std::fabs(lo), std::fabs(hi)) + 1e-300;
    auto count_below = [&](double x) {  // eigenvalues < x
        int c = 0;
        double d = 1.0;
        for (int i = 0; i < m; ++i) {
            d = a[i] - x - (i > 0 ? b[i - 1] * b[i - 1] / d : 0.0);
            if (d == 0.0) d = -1e-300;
            if (d < 0.0) ++c;
        }
        return c;
    };
    for (int it = 0; it < 200 && hi - lo > 1e-15 * scale; ++it) {
        const double mid = 0.5 * (lo + hi);
        if (count_below(mid) >= 1) hi = mid;
        else lo = mid;
    }
    theta = 0.5 * (lo + hi);
    // inverse iteration on T - (theta - tiny) I
    const double shift = theta - 1e-12 * scale;
    y.assign(m, 1.0 / std::sqrt((double)m));
    // (Gaussian elimination with partial pivoting: one row below, so up to two
    // entries above the diagonal)
    std::vector<double> d0(m), d1(m), d2(m), lo_(m), rhs(m);
    for (int it = 0; it < 3; ++it) {
        for (int i = 0; i < m; ++i) {
            d0[i] = a[i] - shift;
            d1[i] = i + 1 < m ? b[i] : 0.0;
            d2[i] = 0.0;
            lo_[i] = i > 0 ? b[i - 1] : 0.0;
            rhs[i] = y[i];
        }
        for (int k = 0; k + 1 < m; ++k) {
            if (std::fabs(lo_[k + 1]) > std::fabs(d0[k])) {
                std::swap(d0[k], lo_[k + 1]);
                std::swap(d1[k], d0[k + 1]);
                std::swap(d2[k], d1[k + 1]);
                std::swap(rhs[k], rhs[k + 1]);
            }
            if (d0[k] == 0.0) d0[k] = 1e-300;
            const double f = lo_[k + 1] / d0[k];
            d0[k + 1] -= f * d1[k];
            d1[k + 1] -= f * d2[k];
            rhs[k + 1] -= f * rhs[k];
        }
        if (d0[m - 1] == 0.0) d0[m - 1] = 1e-300;
        for (int i = m - 1; i >= 0; --i) {
            double s = rhs[i];
            if (i + 1 < m) s -= d1[i] * y[i + 1];
            if (i + 2 < m) s -= d2[i] * y[i + 2];
            y[i] = s / d0[i];
        }
        double nrm = 0.0;
        for (double v : y) nrm += v * v;
        nrm = std::sqrt(nrm);
        for (double& v : y) v /= nrm;
    }
}

}  // namespace

extern "C" {

gl_status gl_second_eigenpair_workspace_size(const gl_operator* op, int32_t krylov, size_t* bytes) {
    if (!gl::valid(op) || !bytes) return efail(GL_E_INVALID_ARG, "operator (a live operator handle) and bytes must not be NULL");
    if (krylov < 2 || krylov > 512) return efail(GL_E_INVALID_ARG, "krylov must lie in [2, 512]");
    *bytes = carve(op, krylov, nullptr).bytes;
    return GL_OK;
}

gl_status gl_second_eigenpair(const gl_operator* op, int32_t krylov, int32_t max_restarts, double tol,
                              const float* x0, float* v_out, void* ws, size_t ws_bytes, double* lambda2,
                              double* residual, int32_t* restarts_used, void* stream) {
    if (!gl::valid(op) || !x0 || !v_out || !ws || !lambda2 || !residual)
        return efail(GL_E_INVALID_ARG, "operator, x0, v_out, workspace and outputs must not be NULL");
    if (krylov < 2 || krylov > 512) return efail(GL_E_INVALID_ARG, "krylov must lie in [2, 512]");
    if (max_restarts < 0) return efail(GL_E_INVALID_ARG, "max_restarts must be >= 0");
    if (!(tol > 0.0) || !std::isfinite(tol)) return efail(GL_E_INVALID_ARG, "tol must be finite and > 0");
    if (op->store_w == GL_F64) return efail(GL_E_DTYPE, "the eigen-solver runs on F32/BF16/F16 weights");
    if ((uintptr_t)ws % 256) return efail(GL_E_INVALID_ARG, "workspace must be 256-byte aligned");
    const int32_t m = (int32_t)std::min<int64_t>(krylov, op->n - 1);
    if (m < 2) return efail(GL_E_INVALID_ARG, "the graph is too small");
    EigWs e = carve(op, m, (char*)ws);
    if (ws_bytes < e.bytes) return efail(GL_E_INVALID_ARG, "workspace too small");
    hipStream_t s = (hipStream_t)stream;
    const int64_t n = op->n;
    const unsigned g256 = (unsigned)((n + 255) / 256);
    gl::RowLaunch rows = gl::operator_rows(op);
    rows.wpart = e.wpart;
    hipError_t err = hipSuccess;
#define GE_CHECK(what)                                                                  \
    do {                                                                                \
        if (err == hipSuccess) err = hipGetLastError();                                 \
        if (err != hipSuccess)                                                          \
            return efail(GL_E_HIP, std::string(what) + ": " + hipGetErrorString(err)); \
    } while (0)

    // c = V^T w for the cnt vectors from z on, then w -= V c; norm <- |w|^2 per
    // tile.  Where a tile count is large, the partial sums are added up first.
    auto dots = [&](const float* V, int32_t cnt, const float* w) {
        const dim3 grid((unsigned)e.nb, (unsigned)((cnt + 4 * gl::kDotVecs - 1) / (4 * gl::kDotVecs)));
        if (e.R == 1)
            hipLaunchKernelGGL(gl::dots_kernel<1>, grid, dim3(gl::kBlock), 0, s, n, V, e.ldv, cnt, w, e.partials, e.nb);
        else
            hipLaunchKernelGGL(gl::dots_kernel<4>, grid, dim3(gl::kBlock), 0, s, n, V, e.ldv, cnt, w, e.partials, e.nb);
    };
    auto combine = [&](const float* V, int32_t cnt, const double* c, int32_t nc, const float* w, float* out,
                       double* keep) {
        const dim3 grid((unsigned)e.nb);
        if (e.R == 1)
            hipLaunchKernelGGL(gl::combine_kernel<1>, grid, dim3(gl::kBlock), 0, s, n, V, e.ldv, cnt, c, nc, w, out,
                               e.norm, keep);
        else
            hipLaunchKernelGGL(gl::combine_kernel<4>, grid, dim3(gl::kBlock), 0, s, n, V, e.ldv, cnt, c, nc, w, out,
                               e.norm, keep);
    };
    auto orthogonalise = [&](float* w, int32_t cnt, double* first_pass_last) {
        for (int pass = 0; pass < 2; ++pass) {
            double* keep = pass == 0 ? first_pass_last : nullptr;
            dots(e.z, cnt, w);
            if (e.nb <= 128) {
                combine(e.z, cnt, e.partials, (int32_t)e.nb, w, w, keep);
            } else {
                hipLaunchKernelGGL(gl::sum_partials_kernel, dim3((unsigned)cnt), dim3(gl::kBlock), 0, s, e.partials,
                                   e.nb, e.sums);
                combine(e.z, cnt, e.sums, 1, w, w, keep);
            }
        }
    };
    const unsigned g1024 = (unsigned)((n + 4 * gl::kBlock - 1) / (4 * gl::kBlock));
    // Every workgroup adds up the tiles' sums itself, which is nb^2 reads in all: beyond
    // kSumTiles tiles (8 M rows) a launch of its own does it first (32 steps on 2 M rows
    // 17.4 ms without and 17.5 with it, on 16 M 209 and 206).
    auto normalise = [&](const float* x, float* y, const double* norm, int64_t nb, double* length) {
        if (nb > gl::kSumTiles) {
            hipLaunchKernelGGL(gl::sum_partials_kernel, dim3(1), dim3(gl::kBlock), 0, s, norm, nb, e.sums);
            norm = e.sums;
            nb = 1;
        }
        hipLaunchKernelGGL(gl::normalise_kernel, dim3(g1024), dim3(gl::kBlock), 0, s, n, x, y, norm, nb, length);
    };
    auto norm2 = [&](const float* v, double* out) {  // |v|^2 to *out
        dots(v, 1, v);
        hipLaunchKernelGGL(gl::sum_partials_kernel, dim3(1), dim3(gl::kBlock), 0, s, e.partials, e.nb, out);
    };
    double *d_alpha = e.out, *d_beta = e.out + m, *d_scal = e.out + 2 * m;

    // null vector z, unit norm
    hipLaunchKernelGGL(gl::null_vector_kernel, dim3(g256), dim3(256), 0, s, n, op->degree, op->order,
                       op->lap == GL_LAP_NORMALIZED ? 1 : 0, e.z);
    dots(e.z, 1, e.z);
    normalise(e.z, e.z, e.partials, e.nb, nullptr);
    // start vector in position order
    hipLaunchKernelGGL(gl::gather_kernel, dim3(g256), dim3(256), 0, s, n, x0, op->order, e.x);
    GE_CHECK("start vector");

    double theta = 0.0, res = INFINITY;
    int32_t restart = 0;
    std::vector<double> host(2 * m + 4), a, b, y;
    for (;; ++restart) {
        // q_0 = x - (z.x) z, normalised
        norm2(e.x, d_scal);
        orthogonalise(e.x, 1, nullptr);
        hipLaunchKernelGGL(gl::sum_partials_kernel, dim3(1), dim3(gl::kBlock), 0, s, e.norm, e.nb, d_scal + 1);
        normalise(e.x, e.Q, e.norm, e.nb, nullptr);
        GE_CHECK("start vector");
        for (int32_t j = 0; j < m; ++j) {
            err = gl::launch_laplacian_f32(1, rows, e.Q + (int64_t)j * e.ldv, e.w, s);
            GE_CHECK("Lanczos product");
            orthogonalise(e.w, j + 2, d_alpha + j);
            if (j + 1 < m) normalise(e.w, e.Q + (int64_t)(j + 1) * e.ldv, e.norm, e.nb, d_beta + j);
            GE_CHECK("Lanczos step");
        }
        err = hipMemcpyAsync(host.data(), e.out, (size_t)(2 * m + 2) * 8, hipMemcpyDeviceToHost, s);
        if (err == hipSuccess) err = hipStreamSynchronize(s);
        GE_CHECK("Lanczos coefficients");
        const double before = host[2 * m], after = host[2 * m + 1];
        if (!(before > 0.0) || !std::isfinite(before))
            return efail(GL_E_NONFINITE, "the start vector is zero or not finite");
        if (!(after > 1e-10 * before))
            return efail(GL_E_INVALID_ARG, "the start vector is parallel to the null vector");
        // up to an invariant subspace: |w| at the rounding of L q_j itself (2^-24 of its
        // entries; |L q_j|^2 = beta_{j-1}^2 + alpha_j^2 + beta_j^2).  Below it, the second
        // Gram-Schmidt pass works on rounding errors and its result is no longer
        // orthogonal to the vectors before it (a graph with few distinct eigenvalues
        // gets there).  No multiple of dmax: a restart begins with beta_0 = the last
        // residual, which L q_0 = lambda q_0 lets go far below 2^-24 dmax; one direction
        // at that rounding does no harm yet, so the first step is cut at a quarter.
        a.clear();
        b.clear();
        for (int32_t j = 0; j < m; ++j) {
            a.push_back(host[j]);
            const double product = std::hypot(host[j], j > 0 ? host[m + j - 1] : 0.0);
            if (j + 1 == m || !(host[m + j] > (j > 0 ? 4.0 : 1.0) * 0x1p-24 * product)) break;
            b.push_back(host[m + j]);
        }
        tridiag_smallest(a, b, theta, y);
        const int32_t k = (int32_t)a.size();
        err = hipMemcpyAsync(e.y, y.data(), (size_t)k * 8, hipMemcpyHostToDevice, s);
        GE_CHECK("Ritz coefficients");
        combine(e.Q, k, e.y, 1, nullptr, e.x, nullptr);
        normalise(e.x, e.x, e.norm, e.nb, nullptr);
        // residual |L x - theta x| of the unit Ritz vector
        err = gl::launch_laplacian_f32(1, rows, e.x, e.w, s);
        GE_CHECK("residual product");
        hipLaunchKernelGGL(gl::residual_kernel, dim3(g256), dim3(256), 0, s, n, e.w, e.x, theta, e.w);
        norm2(e.w, d_scal + 2);
        double r2 = 0.0;
        err = hipMemcpyAsync(&r2, d_scal + 2, 8, hipMemcpyDeviceToHost, s);
        if (err == hipSuccess) err = hipStreamSynchronize(s);
        GE_CHECK("residual norm");
        res = std::sqrt(std::max(r2, 0.0));
        if (res <= tol || restart >= max_restarts || k == 1) break;  // k == 1: x is what it was
    }
    // sign: the entry of largest magnitude is positive
    float* sign = e.best + g256;
    hipLaunchKernelGGL(gl::argmax_kernel, dim3(g256), dim3(gl::kBlock), 0, s, n, e.x, e.best, e.where);
    hipLaunchKernelGGL(gl::sign_kernel, dim3(1), dim3(gl::kBlock), 0, s, e.x, e.best, e.where, (int64_t)g256, sign);
    hipLaunchKernelGGL(gl::output_kernel, dim3(g256), dim3(256), 0, s, n, e.x, v_out, sign, op->order);
    GE_CHECK("eigenvector output");
    err = hipStreamSynchronize(s);
    GE_CHECK("eigen-solver");
#undef GE_CHECK
    *lambda2 = theta;
    *residual = res;
    if (restarts_used) *restarts_used = restart;
    return GL_OK;
}

}  // extern "C"
