// Thread-per-output bodies that run alone or as members of a region: depthwise convolutions and window pools
// (the kernels and their launchers are in kernels_misc.hip).
#pragma once

#include <type_traits>

#include <hip/hip_runtime.h>

#include "device_common.h"

namespace clg {

// (i: the output of this thread)
// Depthwise convolution (one input channel per output channel), square filter KS: one output per
// thread, taps unrolled, loads without branches (clamped addresses, masked values) so that they all
// go out together; optional relu on the input, fused tail.
template <int KS>
__device__ __forceinline__ void depthwise_body(const DirectConvArgs &a, const uint32_t i) {
    const uint32_t npix = (uint32_t)(a.HO * a.WO);
    const uint32_t total = (uint32_t)(a.N * a.C) * npix;
    if (i >= total) return;
    const uint32_t nc = i / npix, p = i - nc * npix;
    const uint32_t c = nc % (uint32_t)a.C;
    const int oh = (int)(p / (uint32_t)a.WO), ow = (int)(p - (uint32_t)oh * a.WO);
    const int ih0 = oh * a.sh - a.ph, iw0 = ow * a.sw - a.pw;
    const float *xc = a.x + (int64_t)nc * a.H * a.W;
    const float *wc = a.w + c * (KS * KS);
    const float lo = a.pro_relu ? 0.f : -INFINITY;
    int ro[KS], co[KS];
    bool vr[KS], vc[KS];
#pragma unroll
    for (int t = 0; t < KS; ++t) {
        const int ih = ih0 + t, iw = iw0 + t;
        vr[t] = ih >= 0 && ih < a.H;
        vc[t] = iw >= 0 && iw < a.W;
        ro[t] = (ih < 0 ? 0 : (ih >= a.H ? a.H - 1 : ih)) * a.W;
        co[t] = iw < 0 ? 0 : (iw >= a.W ? a.W - 1 : iw);
    }
    float xv[KS * KS], wv[KS * KS];
#pragma unroll
    for (int kh = 0; kh < KS; ++kh)
#pragma unroll
        for (int kw = 0; kw < KS; ++kw) {
            xv[kh * KS + kw] = xc[ro[kh] + co[kw]];
            wv[kh * KS + kw] = wc[kh * KS + kw];
        }
    // bias and residual of this output, fetched with the taps
    const int f = a.ef.flags;
    const bool fast = !(f & EF_GENERIC);
    float bias_v = 0.f, add_v = 0.f;
    if (fast && (f & EF_BIAS)) bias_v = a.ef.bias[c];
    if (fast && (f & EF_ADD)) add_v = a.ef.add[i];
    float v = 0.f;
#pragma unroll
    for (int kh = 0; kh < KS; ++kh)
#pragma unroll
        for (int kw = 0; kw < KS; ++kw) {
            const float t = (vr[kh] && vc[kw]) ? fmaxf(xv[kh * KS + kw], lo) : 0.f;
            v = fmaf(wv[kh * KS + kw], t, v);
        }
    if (fast) {
        if (f & EF_SCALE) v *= a.ef.scale;
        v += bias_v;
        v += add_v;
        if (f & EF_RELU) v = v > 0.f ? v : 0.f;
        else if (f & EF_GELU) v = gelu_erf(v);
        else if (f & EF_TANH) v = tanhf(v);
    } else {
        v = apply_steps(a.epi, v, i, (int)c);
    }
    a.y[i] = v;
}

// One output pixel per thread.  AVG: mean over the window's pixels inside the image.
template <bool AVG>
__device__ __forceinline__ void window_pool_body(const PoolArgs &a, const uint32_t i) {
    // 32-bit index arithmetic (the launcher checks the sizes): a 64-bit division is a long routine
    const uint32_t total = (uint32_t)(a.NC * a.DO * a.HO * a.WO);
    if (i >= total) return;
    const uint32_t q1 = i / (uint32_t)a.WO, q2 = q1 / (uint32_t)a.HO;
    const int ow = (int)(i - q1 * a.WO), oh = (int)(q1 - q2 * a.HO);
    int od = 0;
    uint32_t nc = q2;
    if (a.DO > 1) {
        nc = q2 / (uint32_t)a.DO;
        od = (int)(q2 - nc * a.DO);
    }
    const float *xp = a.x + (int64_t)nc * a.D * a.H * a.W;
    float acc = AVG ? 0.f : -INFINITY;
    int cnt = 0;
    // 3x3 windows (planes of a 3x3x3 one): all loads at once, from clamped addresses, and taken or not in the order of the loops below.  One after the
    // other, each behind its test, they made the kernel nine round trips long: 3x3 stride 2 over 112x112, 64 channels, 4.35 us instead of
    // 3.44, batch 32 52 instead of 36 (155 MB).
    auto planes = [&](auto kds) {
        constexpr int KD = decltype(kds)::value;
        float v[KD][9];
        bool in[KD][9];
#pragma unroll
        for (int kd = 0; kd < KD; ++kd)
#pragma unroll
            for (int t = 0; t < 9; ++t) {
                const int id = od * a.sd - a.pd + kd, ih = oh * a.sh - a.ph + t / 3, iw = ow * a.sw - a.pw + t % 3;
                in[kd][t] = id >= 0 && id < a.D && ih >= 0 && ih < a.H && iw >= 0 && iw < a.W;
                v[kd][t] = xp[(uint32_t)((min(max(id, 0), a.D - 1) * a.H + min(max(ih, 0), a.H - 1)) * a.W + min(max(iw, 0), a.W - 1))];
            }
#pragma unroll
        for (int kd = 0; kd < KD; ++kd)
#pragma unroll
            for (int t = 0; t < 9; ++t) {
                acc = !in[kd][t] ? acc : (AVG ? acc + v[kd][t] : fmaxf(acc, v[kd][t]));
                cnt += in[kd][t] ? 1 : 0;
            }
    };
    const bool three = a.KH == 3 && a.KW == 3;
    if (three && a.KD == 1) planes(std::integral_constant<int, 1>{});
    else if (three && a.KD == 3) planes(std::integral_constant<int, 3>{});
    else for (int kd = 0; kd < a.KD; ++kd) {
        const int id = od * a.sd - a.pd + kd;
        if (id < 0 || id >= a.D) continue;
        for (int kh = 0; kh < a.KH; ++kh) {
            const int ih = oh * a.sh - a.ph + kh;
            if (ih < 0 || ih >= a.H) continue;
            for (int kw = 0; kw < a.KW; ++kw) {
                const int iw = ow * a.sw - a.pw + kw;
                if (iw < 0 || iw >= a.W) continue;
                const float v = xp[(id * a.H + ih) * a.W + iw];
                acc = AVG ? acc + v : fmaxf(acc, v);
                ++cnt;
            }
        }
    }
    if (AVG) acc = cnt ? acc / (float)cnt : 0.f;
    if (a.epi.n) acc = apply_steps(a.epi, acc, i, a.epi.bias_c ? (int)((i / (uint32_t)a.epi.bias_inner) % (uint32_t)a.epi.bias_c) : 0);
    a.y[i] = acc;
}

}  // namespace clg
