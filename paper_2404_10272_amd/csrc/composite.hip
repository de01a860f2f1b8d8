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
// prefix) and T from the optical depth before the sample: that before its
// chunk of 64, kept in 64 bits, and float sums within the chunk.  One 16-lane
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
// the lane whose place differs in the bits a permutation of four lanes exchanges
template <int kCtrl>
__device__ __forceinline__ int32_t lane_xor(int32_t x) {
    return __builtin_amdgcn_update_dpp(0, x, kCtrl, 0xF, 0xF, true);
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
// smallest value of the row, in every lane (a lane whose source falls outside
// the row keeps its own)
template <int kCtrl>
__device__ __forceinline__ float dpp_min(float x) {
    return fminf(x, __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(x), __float_as_int(x), kCtrl, 0xF, 0xF, false)));
}
// value of lane kLane (0..15) of this lane's row
template <int kLane>
__device__ __forceinline__ float row_bcast(float x) {
    return dpp<0x150 + kLane>(x);
}
__device__ __forceinline__ float row_min(float x) {
    return row_bcast<kRow - 1>(dpp_min<0x118>(dpp_min<0x114>(dpp_min<0x112>(dpp_min<0x111>(x)))));
}

// sum over the row in 64 bits, in every lane
template <int kCtrl>
__device__ __forceinline__ double dpp64(double x) {
    const int64_t b = __double_as_longlong(x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)b, kCtrl, 0xF, 0xF, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(b >> 32), kCtrl, 0xF, 0xF, true);
    return __longlong_as_double((int64_t)((uint64_t)hi << 32 | lo));
}
__device__ __forceinline__ double row_sum64(double x) {
    x += dpp64<0x111>(x);
    x += dpp64<0x112>(x);
    x += dpp64<0x114>(x);
    x += dpp64<0x118>(x);
    return dpp64<0x150 + kRow - 1>(x);
}
// value of lane kLane (0..3) of this lane's four
template <int kLane>
__device__ __forceinline__ float quad_bcast(float x) {
    return dpp<kLane * 0x55>(x);
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

// Step lengths and optical depths (kDepths) of samples i .. i+3 of a ray ending at
// b, and their colours (kColours); zero past it.  A group may run past the ray into
// the next one's samples, whose values are dropped; only past `total`, the end of
// all rays' samples, is nothing read.
template <bool kDepths, bool kColours>
__device__ __forceinline__ void load_group(int64_t i, int64_t b, int64_t total, const float *__restrict__ t0,
                                           const float *__restrict__ t1, const float *__restrict__ sigma,
                                           const float *__restrict__ rgb, float dt[kPer], float tau[kPer],
                                           float c[3 * kPer]) {
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        if (kDepths) dt[k] = tau[k] = 0.f;
        if (kColours) c[3 * k] = c[3 * k + 1] = c[3 * k + 2] = 0.f;
    }
    if (i >= b) return;
    float u[kPer], v[kPer], s[kPer];
    if (i + kPer <= total) {
        if (kDepths) {
            load4(t0 + i, u);
            load4(t1 + i, v);
            load4(sigma + i, s);
        }
        if (kColours) {
            load4(rgb + 3 * i, c);
            load4(rgb + 3 * i + 4, c + 4);
            load4(rgb + 3 * i + 8, c + 8);
        }
    } else {
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            u[k] = v[k] = s[k] = 0.f;
            if (i + k < b) {
                if (kDepths) {
                    u[k] = t0[i + k];
                    v[k] = t1[i + k];
                    s[k] = sigma[i + k];
                }
                if (kColours) {
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
        if (kDepths) {
            dt[k] = ok ? v[k] - u[k] : 0.f;
            tau[k] = ok ? s[k] * dt[k] : 0.f;
        }
        if (kColours) {
#pragma unroll
            for (int q = 0; q < 3; ++q) c[3 * k + q] = ok ? c[3 * k + q] : 0.f;
        }
    }
}

// One sample of a ray ending at b (zero past it).
struct Sample {
    float dt, tau, c[3];
};
__device__ __forceinline__ Sample load_one(int64_t i, int64_t b, const float *__restrict__ t0,
                                           const float *__restrict__ t1, const float *__restrict__ sigma,
                                           const float *__restrict__ rgb) {
    Sample x{};
    if (i < b) {
        x.dt = t1[i] - t0[i];
        x.tau = sigma[i] * x.dt;
#pragma unroll
        for (int q = 0; q < 3; ++q) x.c[q] = rgb[3 * i + q];
    }
    return x;
}

// exp(-x), by the hardware's base-2 exponential of a product kept to twice
// the precision of a float (x up to a few hundred otherwise loses bits there);
// beyond the range of the result the power alone, 0 or infinity (or NaN)
__device__ __forceinline__ float exp_neg(float x) {
    constexpr float L = 1.44269502f, l = 1.92596303e-8f;   // log2(e) = L + l
    const float y = -x * L;
    const float e = fmaf(-x, L, -y) - x * l;
    const float p = __builtin_amdgcn_exp2f(y);
    return fabsf(y) < 128.f ? fmaf(p, e * 0.693147181f, p) : p;
}

// alpha = 1 - exp(-tau).  Up to an optical depth of one it is
// tau - tau^2 (1/2 - tau/6 + ...), the series truncated below 2.1e-9 of it and
// rounded once at the end; 1 - exp(-tau) would cancel there.  Thicker samples
// are rare enough that a wave mostly skips their exponential.
__device__ __forceinline__ float alpha_series(float x) {
    float s = fmaf(x, -1.f / 39916800.f, 1.f / 3628800.f);
    s = fmaf(x, -s, 1.f / 362880.f);
    s = fmaf(x, -s, 1.f / 40320.f);
    s = fmaf(x, -s, 1.f / 5040.f);
    s = fmaf(x, -s, 1.f / 720.f);
    s = fmaf(x, -s, 1.f / 120.f);
    s = fmaf(x, -s, 1.f / 24.f);
    s = fmaf(x, -s, 1.f / 6.f);
    s = fmaf(x, -s, 0.5f);
    return fmaf(x, -(x * s), x);
}
__device__ __forceinline__ float alpha_of(float tau) {
    float alpha = alpha_series(tau);
    if (!(fabsf(tau) <= 1.f)) alpha = 1.f - exp_neg(tau);
    return alpha;
}
__device__ __forceinline__ void alphas(const float tau[kPer], float alpha[kPer]) {
    bool thick = false;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        alpha[k] = alpha_series(tau[k]);
        thick = thick || !(fabsf(tau[k]) <= 1.f);
    }
    if (thick) {
#pragma unroll
        for (int k = 0; k < kPer; ++k)
            if (!(fabsf(tau[k]) <= 1.f)) alpha[k] = 1.f - exp_neg(tau[k]);
    }
}

// T alpha; 0 for an opacity of 0, as past a ray's end, whatever the transmittance
// (with negative densities it may be infinite)
__device__ __forceinline__ float weight(float T, float alpha) { return alpha == 0.f ? 0.f : T * alpha; }

// Four samples a lane cost four samples' arithmetic however few a ray has, so a
// wave none of whose rays has more than 16 takes one sample a lane: 640,000 rays
// of 8 samples each 35 us forward and 60 backward, against 54 and 83.  A ray's
// result does not depend on the rays that share its wave: four lanes then do the
// sums of the one lane, in its order, and the steps that only add zeros are left
// out.  (To choose for each ray by its own length, and add in any order, makes
// waves of long and short rays run both forms: 139 us where 130 were, over
// 640,000 rays of 40 samples on average.  Two samples a lane, for rays of up to 32,
// measured no better than four.)
//
// Optical depth before a lane's sample, and (all, in the last lane) of the ray:
// the quads' sums first, their prefix, then the quad's samples one by one.
__device__ __forceinline__ float depth_of_one(float tau, float &all) {
    const int k = threadIdx.x & 3;
    float s = tau + dpp<0xb1>(tau);   // of two, then of four lanes
    s += dpp<0x4e>(s);
    s += dpp<0x114>(s);
    s += dpp<0x118>(s);
    all = s;
    float d = dpp<0x114>(s);
    // read by all lanes, before any of them is left out
    const float tau0 = quad_bcast<0>(tau), tau1 = quad_bcast<1>(tau), tau2 = quad_bcast<2>(tau);
    d += k > 0 ? tau0 : 0.f;
    d += k > 1 ? tau1 : 0.f;
    d += k > 2 ? tau2 : 0.f;
    return d;
}
// sum of w c over a quad's lanes, one after the other (in its last lane)
__device__ __forceinline__ float quad_chain(float w, float c) {
    float x = fmaf(w, c, 0.f);
#pragma unroll
    for (int step = 1; step < kPer; ++step) {
        const float y = fmaf(w, c, dpp<0x111>(x));
        x = (threadIdx.x & 3) == step ? y : x;
    }
    return x;
}
// sum over the row's quads of their last lane's value (in the row's last lane)
__device__ __forceinline__ float quads_total(float x) {
    x += dpp<0x114>(x);
    x += dpp<0x118>(x);
    return x;
}

__device__ __forceinline__ void write_pixel(float *out_rgb, float *out_opacity, int64_t r, float cr, float cg, float cb,
                                            float acc) {
    out_rgb[3 * r + 0] = cr;
    out_rgb[3 * r + 1] = cg;
    out_rgb[3 * r + 2] = cb;
    if (out_opacity) out_opacity[r] = acc;
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
    if (!__any(b - a > kRow)) {   // wave-uniform: one sample a lane
        const Sample x = load_one(a + l, b, t0, t1, sigma, rgb);
        float all;
        const float w = weight(exp_neg(depth_of_one(x.tau, all)), alpha_of(x.tau));
        cr = quads_total(quad_chain(w, x.c[0]));
        cg = quads_total(quad_chain(w, x.c[1]));
        cb = quads_total(quad_chain(w, x.c[2]));
        acc = quads_total(quad_chain(w, 1.f));
        if (live && l == kRow - 1) write_pixel(out_rgb, out_opacity, r, cr, cg, cb, acc);
        return;
    }
    for (int64_t g0 = a; g0 < b; g0 += kChunk) {   // row-uniform
        float dt[kPer], tau[kPer], c[3 * kPer], alpha[kPer];
        load_group<true, true>(g0 + kPer * l, b, total, t0, t1, sigma, rgb, dt, tau, c);
        alphas(tau, alpha);
        const float incl = row_prefix((tau[0] + tau[1]) + (tau[2] + tau[3]));
        float depth = carry + dpp<0x111>(incl);
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const float w = weight(exp_neg(depth), alpha[k]);
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
    if (live && l == kRow - 1) write_pixel(out_rgb, out_opacity, r, cr, cg, cb, acc);
}

// Samples no ray owns (before offsets[0] = lo, from offsets[n_rays] = hi on) get
// zero gradient; the launch's threads share them.
__device__ __forceinline__ void zero_unowned(int64_t lo, int64_t hi, int64_t n_samples, float *__restrict__ d_sigma,
                                             float *__restrict__ d_rgb) {
    const int64_t before = lo < n_samples ? lo : n_samples, after = hi < n_samples ? n_samples - hi : 0;
    for (int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x; k < before + after; k += (int64_t)gridDim.x * kBlock) {
        const int64_t i = k < before ? k : hi + (k - before);
        d_sigma[i] = 0.f;
        d_rgb[3 * i + 0] = 0.f;
        d_rgb[3 * i + 1] = 0.f;
        d_rgb[3 * i + 2] = 0.f;
    }
}

// One 16-lane row per ray.  Pass 1: the optical depth before the ray's last chunk,
// which stays in registers, as do the depths of the chunk before it.  Pass 2,
// chunks from the back: T_i from the depth before the chunk (at each step back less
// the chunk's, both in 64 bits, so that a thick chunk leaves no rounding in those
// before it) plus row prefix sums, and S_i = sum_{k>i} w_k q_k by a row suffix
// sum plus the carry -- never as C minus a prefix.  The upstream gradient is
// constant along a ray, so a sample's colour enters only as q_i = g_C . c_i:
//   dL/dsigma_i = dt_i (T_{i+1} q_i - S_i + g_A T_n).
// One suffix sum instead of three, and one register a sample instead of three;
// the products of q are summed in 64 bits, as they may cancel.  T_n is the
// exponential of the ray's whole optical depth: taken as T_{i+1} less the
// weights behind i (the opacity as one more channel of colour one) it would be
// a small difference of numbers near one on every opaque ray.
//
// Bound by HBM: 640,000 rays with 25.4 M samples, 614 MB in and 407 MB out,
// take 255 us, 4.0 TB/s; one sample a lane took 375 us.  The depths kept from
// pass 1 took 5 to 10% off rays of more than 64 samples (640,000 of 100 each 565 us
// against 616).  Two chunks kept whole took 270 us, three 302 and four 351, as more
// registers leave fewer waves.
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
    const double dr = gr, dg = gg, db = gb;
    const float ga = live && g_opacity ? g_opacity[r] : 0.f;
    if (!__any(b - a > kRow)) {   // wave-uniform: one sample a lane, as in the forward pass
        const int64_t i = a + l;
        const Sample x = load_one(i, b, t0, t1, sigma, rgb);
        const float q = (float)fma(db, (double)x.c[2], fma(dg, (double)x.c[1], dr * (double)x.c[0]));
        float all;
        const float d = depth_of_one(x.tau, all), w = weight(exp_neg(d), alpha_of(x.tau)), next = exp_neg(d + x.tau);
        const float end = ga * expf(-row_bcast<kRow - 1>(all));
        // sum over the later quads, then over the quad's later lanes, one after the other
        float qs = quad_bcast<kPer - 1>(quad_chain(w, q));
        qs += dpp<0x104>(qs);
        qs += dpp<0x108>(qs);
        float S = dpp<0x104>(qs);
#pragma unroll
        for (int step = kPer - 2; step >= 0; --step) {
            const float later = fmaf(dpp<0x101>(w), dpp<0x101>(q), dpp<0x101>(S));
            S = (threadIdx.x & 3) == step ? later : S;
        }
        if (i < b) {
            d_sigma[i] = x.dt * (fmaf(next, q, -S) + end);
            d_rgb[3 * i + 0] = w * gr;
            d_rgb[3 * i + 1] = w * gg;
            d_rgb[3 * i + 2] = w * gb;
        }
        zero_unowned(offsets[0], hi, n_samples, d_sigma, d_rgb);
        return;
    }
    const int64_t last = b > a ? a + (b - a - 1) / kChunk * kChunk : a;   // first sample of the last chunk
    float dt[kPer], tau[kPer], q[kPer], c[3 * kPer];
    float dt_before[kPer] = {}, tau_before[kPer] = {};   // of the chunk before it
    const auto sum64 = [](const float v[kPer]) { return ((double)v[0] + v[1]) + ((double)v[2] + v[3]); };
    double part = 0.;
    for (int64_t g0 = a; g0 < last; g0 += kChunk) {   // the chunks before the last
        load_group<true, false>(g0 + kPer * l, b, hi, t0, t1, sigma, rgb, dt_before, tau_before, c);
        part += sum64(tau_before);
    }
    load_group<true, true>(last + kPer * l, b, hi, t0, t1, sigma, rgb, dt, tau, c);
    double depth = row_sum64(part);   // before the chunk
    float later = 0.f;                                     // sum of w q over the later chunks
    float end = 0.f;                                       // g_A T_n
    for (int64_t g0 = last; g0 >= a; g0 -= kChunk) {   // row-uniform
        const int64_t i = g0 + kPer * l;
        if (g0 == last - kChunk) {
            load_group<false, true>(i, b, hi, t0, t1, sigma, rgb, dt, tau, c);
#pragma unroll
            for (int k = 0; k < kPer; ++k) {
                dt[k] = dt_before[k];
                tau[k] = tau_before[k];
            }
        } else if (g0 != last) {
            load_group<true, true>(i, b, hi, t0, t1, sigma, rgb, dt, tau, c);
        }
#pragma unroll
        for (int k = 0; k < kPer; ++k)
            q[k] = (float)fma(db, (double)c[3 * k + 2], fma(dg, (double)c[3 * k + 1], dr * (double)c[3 * k]));
        const float incl = row_prefix((tau[0] + tau[1]) + (tau[2] + tau[3])), all = row_bcast<kRow - 1>(incl);
        if (g0 == a) depth = 0.;
        else if (g0 != last) depth -= row_sum64(sum64(tau));
        if (g0 == last) end = ga * expf(-((float)depth + all));
        float alpha[kPer], w[kPer], next[kPer];   // next: T_{i+1}
        alphas(tau, alpha);
        float d = (float)depth + dpp<0x111>(incl);
        float T = exp_neg(d);
        float wq = 0.f;
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            w[k] = weight(T, alpha[k]);
            d += tau[k];
            next[k] = T = exp_neg(d);
            wq = fmaf(w[k], q[k], wq);
        }
        const float qs = row_suffix(wq);
        float S = dpp<0x101>(qs) + later;   // sum over the samples of later lanes and chunks
        float ds[kPer];
#pragma unroll
        for (int k = kPer - 1; k >= 0; --k) {
            ds[k] = dt[k] * (fmaf(next[k], q[k], -S) + end);
            S = fmaf(w[k], q[k], S);
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
        if (g0 == a) break;
    }
    zero_unowned(offsets[0], hi, n_samples, d_sigma, d_rgb);
}

// ------------------------------------------------------------------ blob field

// Blob parameters as the kernel takes them (a by-value argument; entries past
// the field's blobs are zero): nk = -log2(e) / (2 radius^2), so that
// g = exp2(|x - c|^2 nk) is one hardware exp2; channels of a blob: 1, r, g, b.
struct BlobArgs {
    double nk64[OGV_MAX_BLOBS];
    float cx[OGV_MAX_BLOBS], cy[OGV_MAX_BLOBS], cz[OGV_MAX_BLOBS], nk[OGV_MAX_BLOBS], a[OGV_MAX_BLOBS];
    float channel[OGV_MAX_BLOBS][4];
};

// 2^x for x <= 0, within 1e-9 of itself: the weights' common factors are rounded
// to a float once.
__device__ __forceinline__ double exp2_64(double x) {
    x = fmax(x, -1000.);
    const double n = rint(x), z = (x - n) * 0.69314718055994531;   // |z| <= 0.347
    double p = fma(z, 1. / 40320., 1. / 5040.);
    p = fma(z, p, 1. / 720.);
    p = fma(z, p, 1. / 120.);
    p = fma(z, p, 1. / 24.);
    p = fma(z, p, 1. / 6.);
    p = fma(z, p, 0.5);
    p = fma(z, p, 1.);
    p = fma(z, p, 1.);
    return ldexp(p, (int)n);
}

typedef float Acc __attribute__((ext_vector_type(4)));

// a_k exp2(nk |x - c_k|^2) at the ray's samples, from the distance along the
// ray to its point nearest c_k: with s the length from a reference point,
// |x - c_k|^2 = (s - u_k)^2 + perp_k^2, so a blob's value at a sample is
// exp2(nk (s - u_k)^2) W_k, W_k = a_k exp2(nk perp_k^2) once per ray.  Lane k of
// a row holds u_k and W_k of its ray, in 64 bits up to their rounding, and every
// lane of the row reads them with the instruction that uses them (DPP).  The
// reference point lies among the blobs: s and u_k are small there and lose
// nothing to the camera's distance, which o + d t rounded at does.  It is the
// mean of the nearest parameters of the blobs that the ray meets (W_k > 0), those
// behind the origin or beyond twice the first one's left out: a blob far from the
// others, or one without density, takes no bits from them, and samples near any
// blob are no further from the reference than from the origin.
template <int kK, int kN>
struct Blobs {
    static __device__ __forceinline__ void add(const BlobArgs &f, const float channel[kN], float s, float u, float W,
                                               Acc &acc) {
        const float v = s - dpp<0x150 + kK>(u);
        const float w = __builtin_amdgcn_exp2f(v * v * f.nk[kK]) * dpp<0x150 + kK>(W);
        // four lanes a block: row i (channel i of lane i) times column j (the
        // weight of lane j's sample), added to lane j's acc[i]
        acc = __builtin_amdgcn_mfma_f32_4x4x1f32(channel[kK], w, acc, 0, 0, 0);
        if constexpr (kK + 1 < kN) Blobs<kK + 1, kN>::add(f, channel, s, u, W, acc);
    }
};

// The same from the sample's place, which needs nothing per ray and blob, but
// seven more instructions per sample and blob.  A loop that loads each blob's
// parameters to scalar registers as it comes to it: unrolled, they would take the
// other form's registers and waves.
template <int kN>
__device__ __forceinline__ void add_at(const BlobArgs &f, float x, float y, float z, Acc &acc) {
    constexpr int kUnroll = kN <= 4 ? kN : 2;
#pragma unroll kUnroll
    for (int k = 0; k < kN; ++k) {
        const float ex = x - f.cx[k], ey = y - f.cy[k], ez = z - f.cz[k];
        const float w = f.a[k] * __builtin_amdgcn_exp2f(fmaf(ex, ex, fmaf(ey, ey, ez * ez)) * f.nk[k]);
        acc[0] += w;
#pragma unroll
        for (int q = 1; q < 4; ++q) acc[q] = fmaf(w, f.channel[k][q], acc[q]);
    }
}

// Sums of a ray, or of its part in a row's range: the lane's own samples, and the
// depth before the row's next ones.
struct RaySums {
    float r, g, b, opacity, depth;
};
// adds one sample a lane (sum: its sigma and sigma times colour; ok: it is one)
__device__ __forceinline__ void composite_row(RaySums &q, const Acc &sum, float dt, bool ok) {
    const float sig = sum[0];
    // the hardware's reciprocal, refined; it gives 0 where that would be no normal number
    float inv = __builtin_amdgcn_rcpf(sig);
    inv = sig >= 0x1p-126f ? fmaf(fmaf(-sig, inv, 1.f), inv, inv) : 0.f;
    if (__any(sig > 0x1p125f)) inv = sig > 0x1p125f ? 1.f / sig : inv;
    const float tau = ok ? sig * dt : 0.f;
    const float incl = row_prefix(tau);
    const float wt = exp_neg(q.depth + dpp<0x111>(incl)) * alpha_of(tau);
    const float wi = wt * inv;
    q.r = fmaf(wi, sum[1], q.r);
    q.g = fmaf(wi, sum[2], q.g);
    q.b = fmaf(wi, sum[3], q.b);
    q.opacity += wt;
    q.depth += row_bcast<kRow - 1>(incl);
}

// A wave renders `per` consecutive rays (at most kWaveRays), whose samples are
// cut into chunks of 16, one sample a lane of a row, in one of two ways.
//
// A ray a row, four rays at a time: nothing is prepared, and a turn evaluates the
// blobs at the samples' places (add_at).  Rows wait for the longest of four.
//
// Dealt: the chunks of the wave's rays, in order, go to its four rows in four
// contiguous ranges of equal length, and the blobs are evaluated along the ray
// (Blobs).  A ray cut by a range's end is rendered in parts, each as if it began
// with transmittance one, and the parts are put together at the end
// (C = C_1 + T_1 (C_2 + T_2 ...), T_k = exp(-depth of part k)).  A turn costs
// less, but every wave pays for the rays' blobs and for the parts about as much
// as for two turns of twelve blobs.
//
// So short rays, rays of like lengths and fields of few blobs take the first way.
// 640,000 rays, the way taken (always dealt): 8 samples each and 1 blob 37 us
// (84), 12 blobs 67 (106); 40 each, 12 blobs 155 (185); 800x800 rays of one
// object, 1 blob 71 (109), 12 blobs 164 (174); random lengths of 40 on average
// are dealt: 193, and 290 with a ray a row.
//
// Sigma and colour are computed in registers from the field at each sample's
// midpoint.  Along the ray, the sums over blobs of the weight and of its three
// colour products are a contraction of the blobs' channels with the sample's
// weights, one matrix instruction (4x4x1, 16 blocks) a blob, which leaves each
// lane its own sample's four sums and runs beside the vector ALU.  The loops are
// wave-uniform, as matrix instructions ignore the lane mask.
//
// Bound by VALU issue: 640,000 rays of 25.4 M samples through 12 blobs take 193 us,
// of which the blobs' own instructions are about two fifths.  At the 64 registers
// of eight waves a SIMD; at seven 200 us.
constexpr int kWaveRays = 8;
struct RenderLds {
    float2 uw[kWaveRays][kRow];        // u_k, W_k of each ray with samples
    float2 ref_scale[kWaveRays];       // its reference parameter and |d|
    double inv_dd[kWaveRays];
    double len[kWaveRays];
    int64_t from[kWaveRays], to[kWaveRays];   // its samples
    int32_t start[kWaveRays + 1];      // its first chunk among the wave's
    int32_t ray[kWaveRays];            // its index among the wave's rays
    float part[kWaveRays][4][5];       // depth, r, g, b, opacity of its part in each row's range
};
// LDS written by a lane is read by others of the same wave after this.
__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int kN>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(8))) render_blobs_kernel(const int64_t *__restrict__ offsets, int64_t n_rays,
                                                             int per, const float *__restrict__ origins,
                                                             const float *__restrict__ dirs,
                                                             const float *__restrict__ t0,
                                                             const float *__restrict__ t1, BlobArgs f,
                                                             float *__restrict__ out_rgb,
                                                             float *__restrict__ out_opacity) {
    __shared__ RenderLds lds[kBlock / 64];
    RenderLds &w = lds[threadIdx.x >> 6];
    const int lane = threadIdx.x & 63, l = lane & (kRow - 1), row = lane / kRow;
    const int64_t r0 = ((int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6)) * per;

    // lane i: ray r0 + i; the rays with samples are packed to the front
    const bool live = lane < per && r0 + lane < n_rays;
    const int64_t a = live ? offsets[r0 + lane] : 0, b = live ? offsets[r0 + lane + 1] : 0;
    const int32_t chunks = b > a ? (int32_t)((b - a + kRow - 1) / kRow) : 0;
    // a ray a row where that costs less: a turn (16 samples a row) by either way
    // and the dealing, in twelfths of a microsecond for every wave of 640,000
    // rays, from equal lengths of 40 and 96 samples through 1 to 16 blobs
    constexpr int kTurnAt = 100 + 17 * kN, kTurnAlong = 114 + 12 * kN, kDeal = 500;
    int32_t most = max(chunks, lane_xor<0xb1>(chunks));   // of the ray's four
    most = max(most, lane_xor<0x4e>(most));
    int32_t all = chunks + lane_xor<0xb1>(chunks);
    all += lane_xor<0x4e>(all);
    const int32_t turns[2] = {__builtin_amdgcn_readlane(most, 0), __builtin_amdgcn_readlane(most, 4)};
    const int32_t dealt = (__builtin_amdgcn_readlane(all, 0) + __builtin_amdgcn_readlane(all, 4) + 3) / 4;
    if ((int64_t)(turns[0] + turns[1]) * kTurnAt <= (int64_t)dealt * kTurnAlong + kDeal) {
        for (int h = 0; 4 * h < per; ++h) {
            const int64_t r = r0 + 4 * h + row;
            if (r0 + 4 * h >= n_rays) break;   // wave-uniform
            const int64_t from = __shfl(a, 4 * h + row, 64), to = __shfl(b, 4 * h + row, 64);
            float o[3] = {0.f, 0.f, 0.f}, d[3] = {0.f, 0.f, 0.f};
            if (to > from) {
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    o[k] = origins[3 * r + k];
                    d[k] = dirs[3 * r + k];
                }
            }
            RaySums q{};
            int64_t g = from + l;
            for (int32_t k = 0; k < turns[h]; ++k, g += kRow) {   // wave-uniform
                const bool ok = g < to;
                float m = 0.f, dt = 0.f;
                if (ok) {
                    const float t_a = t0[g], t_b = t1[g];
                    m = 0.5f * (t_a + t_b);
                    dt = t_b - t_a;
                }
                Acc sum = {0.f, 0.f, 0.f, 0.f};
                add_at<kN>(f, fmaf(d[0], m, o[0]), fmaf(d[1], m, o[1]), fmaf(d[2], m, o[2]), sum);
                composite_row(q, sum, dt, ok);
            }
            const float sr = row_prefix(q.r), sg = row_prefix(q.g), sb = row_prefix(q.b), sa = row_prefix(q.opacity);
            if (l == kRow - 1 && r < n_rays) {
                out_rgb[3 * r + 0] = sr;
                out_rgb[3 * r + 1] = sg;
                out_rgb[3 * r + 2] = sb;
                if (out_opacity) out_opacity[r] = sa;
            }
        }
        return;
    }

    const uint64_t some = __ballot(chunks > 0);
    const int rays = __popcll(some), slot = __popcll(some & ((1ull << lane) - 1));
    int32_t last = chunks;   // inclusive scan over the first kWaveRays lanes
#pragma unroll
    for (int off = 1; off < kWaveRays; off <<= 1) {
        const int32_t y = __shfl_up(last, off, 64);
        if (lane >= off) last += y;
    }
    if (chunks > 0) {
        w.ray[slot] = lane;
        w.from[slot] = a;
        w.to[slot] = b;
        w.start[slot] = last - chunks;
        const int64_t r = r0 + lane;
        const double dx = dirs[3 * r], dy = dirs[3 * r + 1], dz = dirs[3 * r + 2];
        const double dd = dx * dx + dy * dy + dz * dz;
        w.inv_dd[slot] = dd > 0. ? 1. / dd : 0.;   // a ray that stays at o has no nearest point
        w.len[slot] = sqrt(dd);
    }
    const int32_t total = __shfl(last, kWaveRays - 1, 64);
    if (lane == 0) w.start[rays] = total;
    wave_fence();

    // row by row: ray i = row, row + 4, ..., blob l
    for (int i0 = 0; i0 < rays; i0 += 4) {
        const int i = i0 + row;
        const bool ok = i < rays;
        float tc_f = 0.f, u = 0.f, W = 0.f, ref = 0.f;
        double tc = 0., len = 0.;
        if (ok) {
            const int64_t r = r0 + w.ray[i];
            const double ex = (double)origins[3 * r] - f.cx[l], ey = (double)origins[3 * r + 1] - f.cy[l];
            const double ez = (double)origins[3 * r + 2] - f.cz[l];
            const double dx = dirs[3 * r], dy = dirs[3 * r + 1], dz = dirs[3 * r + 2];
            len = w.len[i];
            tc = -fma(dx, ex, fma(dy, ey, dz * ez)) * w.inv_dd[i];
            const double px = fma(dx, tc, ex), py = fma(dy, tc, ey), pz = fma(dz, tc, ez);
            const double arg = fma(px, px, fma(py, py, pz * pz)) * f.nk64[l];
            W = l < kN ? (float)(f.a[l] * exp2_64(arg)) : 0.f;
            tc_f = W > 0.f ? (float)tc : 0.f;
        }
        const float first = row_min(tc_f > 0.f ? tc_f : __builtin_huge_valf());
        const bool counts = tc_f > 0.f && tc_f <= 2.f * first;
        const int met = __popcll(__ballot(counts) >> (lane & 48) & 0xffff);
        ref = row_bcast<kRow - 1>(row_prefix(counts ? tc_f : 0.f)) * __builtin_amdgcn_rcpf((float)max(met, 1));
        if (!__builtin_isfinite(ref)) ref = 0.f;   // a direction so short that the blobs are nowhere near in t
        u = (float)((tc - (double)ref) * len);
        if (ok) {
            w.uw[i][l] = make_float2(u, W);
            if (l == 0) w.ref_scale[i] = make_float2(ref, (float)len);
        }
    }
    wave_fence();

    float channel[kN];
#pragma unroll
    for (int k = 0; k < kN; ++k) channel[k] = f.channel[k][l & 3];
    // this row's chunks [c, end)
    int32_t c = (int32_t)((int64_t)total * row / 4);
    const int32_t end = (int32_t)((int64_t)total * (row + 1) / 4);
    int i = -1;              // current ray
    int32_t next = c;        // first chunk past it
    int64_t g = 0, to = 0;   // first sample of the current chunk, end of the ray's samples
    float u = 0.f, W = 0.f, ref = 0.f, scale = 0.f;
    RaySums q{};
    while (__any(c < end)) {
        if (c < end && c == next) {   // row-uniform: on to the next ray
            if (i < 0) {
                while (w.start[i + 1] <= c) {
                    if (++i + 1 == rays) break;
                }
            } else {
                ++i;
            }
            const float2 uw = w.uw[i][l], rs = w.ref_scale[i];
            u = uw.x;
            W = uw.y;
            ref = rs.x;
            scale = rs.y;
            next = w.start[i + 1];
            to = w.to[i];
            g = w.from[i] + (int64_t)(c - w.start[i]) * kRow;
            q = RaySums{};
        }
        const bool ok = c < end && g + l < to;
        float s = 0.f, dt = 0.f;
        if (ok) {
            const float t_a = t0[g + l], t_b = t1[g + l];
            s = 0.5f * ((t_a - ref) + (t_b - ref)) * scale;
            dt = t_b - t_a;
        }
        Acc sum = {0.f, 0.f, 0.f, 0.f};
        Blobs<0, kN>::add(f, channel, s, u, W, sum);
        composite_row(q, sum, dt, ok);
        const bool mine = c < end;
        ++c;
        g += kRow;
        if (mine && (c == next || c == end)) {   // row-uniform: the ray, or its part here, ends
            const float sr = row_prefix(q.r), sg = row_prefix(q.g), sb = row_prefix(q.b), sa = row_prefix(q.opacity);
            if (l == kRow - 1) {
                float *p = w.part[i][row];
                p[0] = q.depth;
                p[1] = sr;
                p[2] = sg;
                p[3] = sb;
                p[4] = sa;
            }
        }
    }
    wave_fence();
    if (!live) return;
    // lane i again: its ray's parts, from the back, in 64 bits so that a cut
    // costs no rounding of its own
    double C[4] = {0., 0., 0., 0.};
    if (chunks > 0) {
#pragma unroll
        for (int q = 3; q >= 0; --q) {
            const int32_t from = (int32_t)((int64_t)total * q / 4), upto = (int32_t)((int64_t)total * (q + 1) / 4);
            if (max(from, last - chunks) >= min(upto, last)) continue;
            const float *p = w.part[slot][q];
            if (upto >= last) {   // the ray's last part
#pragma unroll
                for (int k = 0; k < 4; ++k) C[k] = p[1 + k];
            } else {
                const double T = exp2_64(fmin(-1.4426950408889634 * (double)p[0], 1000.));
#pragma unroll
                for (int k = 0; k < 4; ++k) C[k] = fma(T, C[k], (double)p[1 + k]);
            }
        }
    }
    const int64_t r = r0 + lane;
    out_rgb[3 * r + 0] = (float)C[0];
    out_rgb[3 * r + 1] = (float)C[1];
    out_rgb[3 * r + 2] = (float)C[2];
    if (out_opacity) out_opacity[r] = (float)C[3];
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
    for (int k = 0; k < field->n; ++k) {
        const float rad = field->radius[k], den = field->density[k];
        if (!(rad > 0.f) || !(den >= 0.f) || !std::isfinite(rad) || !std::isfinite(den))
            OGV_FAIL(OGV_ERR_INVALID, "blob radius must be > 0 and density >= 0, both finite");
        f.cx[k] = field->centre[k][0];
        f.cy[k] = field->centre[k][1];
        f.cz[k] = field->centre[k][2];
        f.nk64[k] = -1.4426950408889634 / (2.0 * (double)rad * (double)rad);   // -log2(e) / (2 r^2)
        f.nk[k] = (float)f.nk64[k];
        f.a[k] = den;
        f.channel[k][0] = 1.f;
        for (int q = 0; q < 3; ++q) f.channel[k][1 + q] = field->colour[k][q];
    }
    if (n_rays == 0) return OGV_OK;
    if (!offsets || !origins || !dirs || !t0 || !t1 || !out_rgb) OGV_FAIL(OGV_ERR_INVALID, "null argument");
    hipStream_t s = (hipStream_t)stream;
    // 8 rays a wave even their lengths out (640,000 rays of random lengths, all
    // dealt, 191 us against 215 with 4) and still part the long rays of an image's
    // middle (800x800 rays of one object 170 us, with 4 rays 175; 16 take 187 on the
    // random lengths and 190 here).  Calls of fewer rays need the waves instead:
    // half that image 96 us with 4 against 101 with 8, a quarter 57 against 68,
    // 300,000 random rays 108 against 99
    const int per = n_rays >= 524288 ? kWaveRays : 4;
    const int64_t per_block = (int64_t)per * (kBlock / 64);
    const unsigned blocks = (unsigned)((n_rays + per_block - 1) / per_block);
    // one instantiation per number of blobs: a blob's row broadcast is part of
    // the instructions' encoding
#define OGV_BLOBS(N)                                                                                             \
    case N:                                                                                                      \
        render_blobs_kernel<N><<<blocks, kBlock, 0, s>>>(offsets, n_rays, per, origins, dirs, t0, t1, f, out_rgb, \
                                                         out_opacity);                                           \
        break;
    switch (field->n) {
        OGV_BLOBS(1) OGV_BLOBS(2) OGV_BLOBS(3) OGV_BLOBS(4) OGV_BLOBS(5) OGV_BLOBS(6) OGV_BLOBS(7) OGV_BLOBS(8)
        OGV_BLOBS(9) OGV_BLOBS(10) OGV_BLOBS(11) OGV_BLOBS(12) OGV_BLOBS(13) OGV_BLOBS(14) OGV_BLOBS(15) OGV_BLOBS(16)
    }
#undef OGV_BLOBS
    OGV_CHECK_LAUNCH();
    return OGV_OK;
}
