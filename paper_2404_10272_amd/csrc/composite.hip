// Volume-rendering composite over packed samples and its backward pass.
//
// The paper only says a ray's sample colours and densities are accumulated
// into the pixel colour (Sec. 1); the emission-absorption quadrature is
// used: per ray, tau_i = sigma_i (t1_i - t0_i), alpha_i = 1 - exp(-tau_i),
// T_i = exp(-sum_{j<i} tau_j), w_i = T_i alpha_i, C = sum w_i c_i,
// A = sum w_i.  The backward pass gives
//   dL/dc_i     = w_i g_C
//   dL/dsigma_i = dt_i (g_C . (T_{i+1} c_i - sum_{k>i} w_k c_k) + g_A T_n),
// with the suffix sum accumulated in a reverse pass (not as C minus a
// prefix) and T rebuilt from the exponent sum, whose absolute error stays
// at the level of one rounding of the ray's total optical depth.  One 16-lane
// row (a DPP row) handles one ray, four consecutive samples a lane.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "internal.hpp"

namespace ogv {
namespace {

constexpr int kBlock = 256;
constexpr int kRow = 16;                    // lanes per ray: one DPP row
constexpr int kRaysPerBlock = kBlock / kRow;

// Row-local data movement on the VALU (DPP): lane j of a 16-lane row reads
// lane j - n (row_shr) or j + n (row_shl) of the same row; lanes whose
// source falls outside the row read 0.
template <int kCtrl>
__device__ __forceinline__ float dpp(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), kCtrl, 0xF, 0xF, true));
}
// inclusive prefix sum over the row (lane 15 ends with the row total)
__device__ __forceinline__ float row_prefix(float x) {
    x += dpp<0x111>(x);
    x += dpp<0x112>(x);
    x += dpp<0x114>(x);
    x += dpp<0x118>(x);
    return x;
}
// inclusive suffix sum over the row (lane 0 ends with the row total)
__device__ __forceinline__ float row_suffix(float x) {
    x += dpp<0x101>(x);
    x += dpp<0x102>(x);
    x += dpp<0x104>(x);
    x += dpp<0x108>(x);
    return x;
}
// value of lane kLane (0..15) of this lane's row
template <int kLane>
__device__ __forceinline__ float row_bcast(float x) {
    return dpp<0x150 + kLane>(x);
}

// Each lane takes kPer consecutive samples of its row's ray, so a row covers
// kChunk samples per pass and reads them with 16-byte loads (three for t0, t1
// and sigma, three for the colours), where one sample a lane took six 4-byte
// loads each.  A group starts wherever the ray does: the loads are aligned to
// 4 bytes, not 16, which global memory takes at full rate.
constexpr int kPer = 4;
constexpr int kChunk = kPer * kRow;

struct __attribute__((packed, aligned(4))) Quad {
    float v[4];
};
__device__ __forceinline__ void load4(const float *p, float v[4]) {
    const Quad q = *reinterpret_cast<const Quad *>(p);
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = q.v[k];
}
__device__ __forceinline__ void store4(float *p, float a, float b, float c, float d) {
    *reinterpret_cast<Quad *>(p) = Quad{{a, b, c, d}};
}

// Step lengths and optical depths of samples i .. i+3 of a ray ending at b
// (zero past it), and their colours when rgb is given.  A group may run past
// the ray into the next one's samples, whose values are dropped; only past
// `total`, the end of all rays' samples, is nothing read.
template <bool kColour>
__device__ __forceinline__ void load_group(int64_t i, int64_t b, int64_t total, const float *__restrict__ t0,
                                           const float *__restrict__ t1, const float *__restrict__ sigma,
                                           const float *__restrict__ rgb, float dt[kPer], float tau[kPer],
                                           float c[3 * kPer]) {
#pragma unroll
    for (int k = 0; k < kPer; ++k) dt[k] = tau[k] = 0.f;
#pragma unroll
    for (int k = 0; k < 3 * kPer; ++k) c[k] = 0.f;
    if (i >= b) return;
    float u[kPer], v[kPer], s[kPer];
    if (i + kPer <= total) {
        load4(t0 + i, u);
        load4(t1 + i, v);
        load4(sigma + i, s);
        if (kColour) {
            load4(rgb + 3 * i, c);
            load4(rgb + 3 * i + 4, c + 4);
            load4(rgb + 3 * i + 8, c + 8);
        }
    } else {
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            u[k] = v[k] = s[k] = 0.f;
            if (i + k < b) {
                u[k] = t0[i + k];
                v[k] = t1[i + k];
                s[k] = sigma[i + k];
                if (kColour) {
                    c[3 * k] = rgb[3 * (i + k)];
                    c[3 * k + 1] = rgb[3 * (i + k) + 1];
                    c[3 * k + 2] = rgb[3 * (i + k) + 2];
                }
            }
        }
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const bool ok = i + k < b;
        dt[k] = ok ? v[k] - u[k] : 0.f;
        tau[k] = ok ? s[k] * dt[k] : 0.f;
        if (kColour) {
#pragma unroll
            for (int q = 0; q < 3; ++q) c[3 * k + q] = ok ? c[3 * k + q] : 0.f;
        }
    }
}

// exp(-x), by the hardware's base-2 exponential of a product kept to twice
// the precision of a float (x up to a few hundred otherwise loses bits there)
__device__ __forceinline__ float exp_neg(float x) {
    constexpr float L = 1.44269502f, l = 1.92596303e-8f;   // log2(e) = L + l
    const float y = -x * L;
    const float e = fmaf(-x, L, -y) - x * l;
    const float p = __builtin_amdgcn_exp2f(y);
    return __builtin_isfinite(y) ? fmaf(p, e * 0.693147181f, p) : p;
}

// alpha = 1 - exp(-tau) of four samples.  Up to half an optical depth it is
// tau - tau^2 (1/2 - tau/6 + ...), the series truncated below 1.1e-8 of it and
// rounded once at the end; 1 - exp(-tau) would cancel there.  Thicker samples
// are rare enough that a wave mostly skips their exponential.
__device__ __forceinline__ void alphas(const float tau[kPer], float alpha[kPer]) {
    bool thick = false;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const float x = tau[k];
        float s = fmaf(x, -1.f / 40320.f, 1.f / 5040.f);
        s = fmaf(x, -s, 1.f / 720.f);
        s = fmaf(x, -s, 1.f / 120.f);
        s = fmaf(x, -s, 1.f / 24.f);
        s = fmaf(x, -s, 1.f / 6.f);
        s = fmaf(x, -s, 0.5f);
        alpha[k] = fmaf(x, -(x * s), x);
        thick = thick || !(fabsf(x) <= 0.5f);
    }
    if (thick) {
#pragma unroll
        for (int k = 0; k < kPer; ++k)
            if (!(fabsf(tau[k]) <= 0.5f)) alpha[k] = 1.f - exp_neg(tau[k]);
    }
}

// One 16-lane row per ray.  The optical depth before a lane's samples is a
// row prefix sum of the lanes' depths plus the carry of earlier chunks; every
// sample's transmittance is an exponential of its own (multiplying one on
// along the lane costs less and rounds more).  Rows past the last ray do
// nothing, but stay in their wave so that every DPP source lane is active.
//
// Bound by HBM reads, whose latency the resident waves (5.9 a SIMD on average)
// and the arithmetic (74 us of VALU issue) do not hide in full: 640,000 rays
// with 25.4 M samples, 614 MB, take 128 us, 4.8 TB/s; one sample a lane took
// 158 us, and a bare read of as many bytes takes 85.  Measured no better: two
// chunks loaded together (139 us), eight lanes a ray (140 us; 20.7 against
// 27.9 us where rays average 8 samples), a persistent grid that loads the next
// ray's offsets ahead (138 to 159 us).
__global__ void __launch_bounds__(kBlock) composite_fwd_kernel(const int64_t *__restrict__ offsets, int64_t n_rays,
                                                              const float *__restrict__ t0,
                                                              const float *__restrict__ t1,
                                                              const float *__restrict__ sigma,
                                                              const float *__restrict__ rgb, float *__restrict__ out_rgb,
                                                              float *__restrict__ out_opacity) {
    const int l = threadIdx.x & (kRow - 1);
    const int64_t r = (int64_t)blockIdx.x * kRaysPerBlock + (threadIdx.x / kRow);
    const bool live = r < n_rays;
    const int64_t a = live ? offsets[r] : 0, b = live ? offsets[r + 1] : 0, total = offsets[n_rays];
    float cr = 0.f, cg = 0.f, cb = 0.f, acc = 0.f, carry = 0.f;
    for (int64_t g0 = a; g0 < b; g0 += kChunk) {   // row-uniform
        float dt[kPer], tau[kPer], c[3 * kPer], alpha[kPer];
        load_group<true>(g0 + kPer * l, b, total, t0, t1, sigma, rgb, dt, tau, c);
        alphas(tau, alpha);
        const float incl = row_prefix((tau[0] + tau[1]) + (tau[2] + tau[3]));
        float depth = carry + dpp<0x111>(incl);
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const float w = exp_neg(depth) * alpha[k];
            cr = fmaf(w, c[3 * k], cr);
            cg = fmaf(w, c[3 * k + 1], cg);
            cb = fmaf(w, c[3 * k + 2], cb);
            acc += w;
            depth += tau[k];
        }
        carry += row_bcast<kRow - 1>(incl);
    }
    cr = row_prefix(cr);
    cg = row_prefix(cg);
    cb = row_prefix(cb);
    acc = row_prefix(acc);
    if (live && l == kRow - 1) {
        out_rgb[3 * r + 0] = cr;
        out_rgb[3 * r + 1] = cg;
        out_rgb[3 * r + 2] = cb;
        if (out_opacity) out_opacity[r] = acc;
    }
}

// One 16-lane row per ray, in spans of kKeep chunks.  Pass 1: the optical
// depth before the ray's last span, which stays in registers.  Pass 2, spans
// from the back: T_i from the depth before it (the span's, less a span at each
// step back, plus row prefix sums), and S_i = sum_{k>i} w_k q_k by a row
// suffix sum plus the carry -- never as C minus a prefix.  The upstream
// gradient is constant along a ray, so a sample's colour enters only as
// q_i = g_C . c_i + g_A, the opacity being
// one more channel of colour one (T_n = T_{i+1} - sum_{k>i} w_k):
//   dL/dsigma_i = dt_i (T_{i+1} q_i - S_i).
// One suffix sum instead of three, and one register a sample instead of three;
// the products of q are summed in 64 bits, as they may cancel.
//
// Bound by HBM: 640,000 rays with 25.4 M samples, 614 MB in and 407 MB out,
// take 263 us, 3.9 TB/s; one sample a lane took 375 us.  kKeep = 1: with two
// chunks a span 270 us (170 against 164 at 24 samples a ray, 65 against 54 at
// 8, 287 against 292 at 96), with three 302 and with four 351, as more
// registers leave fewer waves.
constexpr int kKeep = 1;
__global__ void __launch_bounds__(kBlock) composite_bwd_kernel(
    const int64_t *__restrict__ offsets, int64_t n_rays, int64_t n_samples, const float *__restrict__ t0,
    const float *__restrict__ t1,
    const float *__restrict__ sigma, const float *__restrict__ rgb, const float *__restrict__ g_rgb,
    const float *__restrict__ g_opacity, float *__restrict__ d_sigma, float *__restrict__ d_rgb) {
    const int l = threadIdx.x & (kRow - 1);
    const int64_t r = (int64_t)blockIdx.x * kRaysPerBlock + (threadIdx.x / kRow);
    const bool live = r < n_rays;
    const int64_t a = live ? offsets[r] : 0, b = live ? offsets[r + 1] : 0, hi = offsets[n_rays];
    const float gr = live ? g_rgb[3 * r + 0] : 0.f, gg = live ? g_rgb[3 * r + 1] : 0.f;
    const float gb = live ? g_rgb[3 * r + 2] : 0.f;
    const double dr = gr, dg = gg, db = gb, da = live && g_opacity ? g_opacity[r] : 0.f;
    constexpr int kSpan = kKeep * kChunk;
    // first sample of the last span (the ray's spans start at a)
    const int64_t last = b > a ? a + ((b - a - 1) / kSpan) * kSpan : a;

    float dt[kKeep][kPer], tau[kKeep][kPer], q[kKeep][kPer];
    const auto load_span = [&](int64_t g0) {
#pragma unroll
        for (int h = 0; h < kKeep; ++h) {
            float c[3 * kPer];
            load_group<true>(g0 + h * kChunk + kPer * l, b, hi, t0, t1, sigma, rgb, dt[h], tau[h], c);
#pragma unroll
            for (int k = 0; k < kPer; ++k) 
                q[h][k] = (float)fma(db, (double)c[3 * k + 2], fma(dg, (double)c[3 * k + 1], fma(dr, (double)c[3 * k], da)));
        }
    };
    float part = 0.f;
    for (int64_t g0 = a; g0 < last; g0 += kChunk) {   // the spans before the last
        float u[kPer], v[kPer], none[3 * kPer];
        load_group<false>(g0 + kPer * l, b, hi, t0, t1, sigma, rgb, u, v, none);
        part += (v[0] + v[1]) + (v[2] + v[3]);
    }
    load_span(last);
    float depth = row_bcast<kRow - 1>(row_prefix(part));   // before the span
    float later = 0.f;                                     // sum of w q over the later chunks
    for (int64_t g0 = last; g0 >= a; g0 -= kSpan) {   // row-uniform
        if (g0 != last) load_span(g0);
        float before[kKeep], all[kKeep];   // depth before the lane in its chunk, of the chunk
#pragma unroll
        for (int h = 0; h < kKeep; ++h) {
            const float incl = row_prefix((tau[h][0] + tau[h][1]) + (tau[h][2] + tau[h][3]));
            before[h] = dpp<0x111>(incl);
            all[h] = row_bcast<kRow - 1>(incl);
        }
        if (g0 != last) {
#pragma unroll
            for (int h = 0; h < kKeep; ++h) depth -= all[h];
        }
        if (g0 == a) depth = 0.f;
        float at[kKeep];
        at[0] = depth;
#pragma unroll
        for (int h = 1; h < kKeep; ++h) at[h] = at[h - 1] + all[h - 1];
#pragma unroll
        for (int h = kKeep - 1; h >= 0; --h) {
            if (g0 + h * kChunk >= b) continue;   // row-uniform
            const int64_t i = g0 + h * kChunk + kPer * l;
            float alpha[kPer], w[kPer], next[kPer];   // next: T_{i+1}
            alphas(tau[h], alpha);
            float d = at[h] + before[h];
            float T = exp_neg(d);
            float wq = 0.f;
#pragma unroll
            for (int k = 0; k < kPer; ++k) {
                w[k] = T * alpha[k];
                d += tau[h][k];
                next[k] = T = exp_neg(d);
                wq = fmaf(w[k], q[h][k], wq);
            }
            const float qs = row_suffix(wq);
            float S = dpp<0x101>(qs) + later;   // sum over the samples of later lanes and chunks
            float ds[kPer];
#pragma unroll
            for (int k = kPer - 1; k >= 0; --k) {
                ds[k] = dt[h][k] * fmaf(next[k], q[h][k], -S);
                S = fmaf(w[k], q[h][k], S);
            }
            if (i + kPer <= b) {
                store4(d_sigma + i, ds[0], ds[1], ds[2], ds[3]);
                store4(d_rgb + 3 * i, w[0] * gr, w[0] * gg, w[0] * gb, w[1] * gr);
                store4(d_rgb + 3 * i + 4, w[1] * gg, w[1] * gb, w[2] * gr, w[2] * gg);
                store4(d_rgb + 3 * i + 8, w[2] * gb, w[3] * gr, w[3] * gg, w[3] * gb);
            } else {
#pragma unroll
                for (int k = 0; k < kPer; ++k)
                    if (i + k < b) {
                        d_sigma[i + k] = ds[k];
                        d_rgb[3 * (i + k) + 0] = w[k] * gr;
                        d_rgb[3 * (i + k) + 1] = w[k] * gg;
                        d_rgb[3 * (i + k) + 2] = w[k] * gb;
                    }
            }
            later += row_bcast<0>(qs);
        }
        if (g0 == a) break;
    }
    // samples no ray owns (before offsets[0], from offsets[n_rays] on) get zero gradient
    const int64_t lo = offsets[0];
    const int64_t before = lo < n_samples ? lo : n_samples, after = hi < n_samples ? n_samples - hi : 0;
    for (int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x; k < before + after; k += (int64_t)gridDim.x * kBlock) {
        const int64_t i = k < before ? k : hi + (k - before);
        d_sigma[i] = 0.f;
        d_rgb[3 * i + 0] = 0.f;
        d_rgb[3 * i + 1] = 0.f;
        d_rgb[3 * i + 2] = 0.f;
    }
}

constexpr int kGroup = 4;
constexpr int kSpan = kGroup * kRow;
__device__ __forceinline__ float row_lane(float x, int src) {
    return __shfl(x, ((int)threadIdx.x & 63 & ~(kRow - 1)) | src, 64);
}

// ------------------------------------------------------------------ blob field

// Blob parameters as the kernel takes them (a by-value argument, so they sit
// in scalar registers): nk = -log2(e) / (2 radius^2), so that
// g = exp2(|x - c|^2 nk) is one hardware exp2.
struct BlobArgs {
    int n;
    float cx[OGV_MAX_BLOBS], cy[OGV_MAX_BLOBS], cz[OGV_MAX_BLOBS], nk[OGV_MAX_BLOBS];
    float a[OGV_MAX_BLOBS], r[OGV_MAX_BLOBS], g[OGV_MAX_BLOBS], b[OGV_MAX_BLOBS];
};

// One 16-lane row per ray, the composite forward's structure, with sigma and
// colour computed in registers from the field at each sample's midpoint
// instead of being read.
__global__ void __launch_bounds__(kBlock) render_blobs_kernel(const int64_t *__restrict__ offsets, int64_t n_rays,
                                                             const float *__restrict__ origins,
                                                             const float *__restrict__ dirs,
                                                             const float *__restrict__ t0,
                                                             const float *__restrict__ t1, BlobArgs f,
                                                             float *__restrict__ out_rgb,
                                                             float *__restrict__ out_opacity) {
    const int l = threadIdx.x & (kRow - 1);
    const int64_t r = (int64_t)blockIdx.x * kRaysPerBlock + (threadIdx.x / kRow);
    const bool live = r < n_rays;
    const int64_t a = live ? offsets[r] : 0, b = live ? offsets[r + 1] : 0;
    float o[3] = {0.f, 0.f, 0.f}, d[3] = {0.f, 0.f, 0.f};
    if (live && b > a) {
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            o[q] = origins[3 * r + q];
            d[q] = dirs[3 * r + q];
        }
    }
    float cr = 0.f, cg = 0.f, cb = 0.f, acc = 0.f, carry = 0.f;
    for (int64_t g0 = a; g0 < b; g0 += kSpan) {   // row-uniform
        float mid[kGroup], dt[kGroup];
#pragma unroll
        for (int c = 0; c < kGroup; ++c) {
            const int64_t i = g0 + c * kRow + l;
            mid[c] = dt[c] = 0.f;
            if (i < b) {
                const float u = t0[i], v = t1[i];
                mid[c] = 0.5f * (u + v);
                dt[c] = v - u;
            }
        }
#pragma unroll
        for (int c = 0; c < kGroup; ++c) {
            if (g0 + c * kRow >= b) break;   // row-uniform
            const bool ok = g0 + c * kRow + l < b;
            const float x = fmaf(d[0], mid[c], o[0]), y = fmaf(d[1], mid[c], o[1]), z = fmaf(d[2], mid[c], o[2]);
            float sig = 0.f, nr = 0.f, ng = 0.f, nb = 0.f;
            for (int k = 0; k < f.n; ++k) {
                const float ex = x - f.cx[k], ey = y - f.cy[k], ez = z - f.cz[k];
                const float d2 = fmaf(ex, ex, fmaf(ey, ey, ez * ez));
                const float w = f.a[k] * __builtin_amdgcn_exp2f(d2 * f.nk[k]);
                sig += w;
                nr = fmaf(w, f.r[k], nr);
                ng = fmaf(w, f.g[k], ng);
                nb = fmaf(w, f.b[k], nb);
            }
            const float inv = sig > 0.f ? 1.0f / sig : 0.f;
            const float tau = ok ? sig * dt[c] : 0.f;
            const float incl = row_prefix(tau);
            const float T = expf(-(carry + incl - tau));
            const float w = ok ? T * (-expm1f(-tau)) : 0.f;
            const float wi = w * inv;
            cr = fmaf(wi, nr, cr);
            cg = fmaf(wi, ng, cg);
            cb = fmaf(wi, nb, cb);
            acc += w;
            carry += row_lane(incl, kRow - 1);
        }
    }
    cr = row_prefix(cr);
    cg = row_prefix(cg);
    cb = row_prefix(cb);
    acc = row_prefix(acc);
    if (live && l == kRow - 1) {
        out_rgb[3 * r + 0] = cr;
        out_rgb[3 * r + 1] = cg;
        out_rgb[3 * r + 2] = cb;
        if (out_opacity) out_opacity[r] = acc;
    }
}

}  // namespace
}  // namespace ogv

using namespace ogv;

extern "C" ogv_status ogv_composite_fwd(const int64_t *offsets, int64_t n_rays, const float *t0, const float *t1,
                                        const float *sigma, const float *rgb, float *out_rgb, float *out_opacity,
                                        void *stream) {
    if (n_rays < 0) OGV_FAIL(OGV_ERR_INVALID, "n_rays < 0");
    if (n_rays == 0) return OGV_OK;
    if (!offsets || !out_rgb || !t0 || !t1 || !sigma || !rgb) OGV_FAIL(OGV_ERR_INVALID, "null argument");
    hipStream_t s = (hipStream_t)stream;
    const unsigned blocks = (unsigned)((n_rays + kRaysPerBlock - 1) / kRaysPerBlock);
    composite_fwd_kernel<<<blocks, kBlock, 0, s>>>(offsets, n_rays, t0, t1, sigma, rgb, out_rgb, out_opacity);
    OGV_CHECK_LAUNCH();
    return OGV_OK;
}

extern "C" ogv_status ogv_composite_bwd(const int64_t *offsets, int64_t n_rays, int64_t n_samples, const float *t0,
                                        const float *t1,
                                        const float *sigma, const float *rgb, const float *g_rgb,
                                        const float *g_opacity, float *d_sigma, float *d_rgb, void *stream) {
    if (n_rays < 0) OGV_FAIL(OGV_ERR_INVALID, "n_rays < 0");
    if (n_samples < 0) OGV_FAIL(OGV_ERR_INVALID, "n_samples < 0");
    if (n_rays == 0 && n_samples == 0) return OGV_OK;
    if (!offsets || !t0 || !t1 || !sigma || !rgb || !g_rgb || !d_sigma || !d_rgb)
        OGV_FAIL(OGV_ERR_INVALID, "null argument");
    hipStream_t s = (hipStream_t)stream;
    // at least one block, so that an empty ray range still zeroes the samples
    const unsigned blocks = (unsigned)std::max<int64_t>((n_rays + kRaysPerBlock - 1) / kRaysPerBlock, 1);
    composite_bwd_kernel<<<blocks, kBlock, 0, s>>>(offsets, n_rays, n_samples, t0, t1, sigma, rgb, g_rgb, g_opacity,
                                                   d_sigma, d_rgb);
    OGV_CHECK_LAUNCH();
    return OGV_OK;
}

extern "C" ogv_status ogv_render_blobs(const int64_t *offsets, int64_t n_rays, const float *origins, const float *dirs,
                                       const float *t0, const float *t1, const ogv_blob_field *field, float *out_rgb,
                                       float *out_opacity, void *stream) {
    if (n_rays < 0) OGV_FAIL(OGV_ERR_INVALID, "n_rays < 0");
    if (!field) OGV_FAIL(OGV_ERR_INVALID, "null field");
    if (field->n < 1 || field->n > OGV_MAX_BLOBS) OGV_FAIL(OGV_ERR_INVALID, "blob count outside 1..16");
    BlobArgs f{};
    f.n = field->n;
    for (int k = 0; k < field->n; ++k) {
        const float rad = field->radius[k], den = field->density[k];
        if (!(rad > 0.f) || !(den >= 0.f) || !std::isfinite(rad) || !std::isfinite(den))
            OGV_FAIL(OGV_ERR_INVALID, "blob radius must be > 0 and density >= 0, both finite");
        f.cx[k] = field->centre[k][0];
        f.cy[k] = field->centre[k][1];
        f.cz[k] = field->centre[k][2];
        f.nk[k] = (float)(-1.4426950408889634 / (2.0 * (double)rad * (double)rad));   // -log2(e) / (2 r^2)
        f.a[k] = den;
        f.r[k] = field->colour[k][0];
        f.g[k] = field->colour[k][1];
        f.b[k] = field->colour[k][2];
    }
    if (n_rays == 0) return OGV_OK;
    if (!offsets || !origins || !dirs || !t0 || !t1 || !out_rgb) OGV_FAIL(OGV_ERR_INVALID, "null argument");
    hipStream_t s = (hipStream_t)stream;
    const unsigned blocks = (unsigned)((n_rays + kRaysPerBlock - 1) / kRaysPerBlock);
    render_blobs_kernel<<<blocks, kBlock, 0, s>>>(offsets, n_rays, origins, dirs, t0, t1, f, out_rgb, out_opacity);
    OGV_CHECK_LAUNCH();
    return OGV_OK;
}
