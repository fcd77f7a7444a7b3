// The end of a small classifier in one kernel: [global average pool] -> dense -> softmax, a workgroup per image.
//
// Each of the three is a few microseconds of launch and one memory round trip, and together they are one workgroup's work where the weights are a
// few kilobytes.  What bounds it is that round trip and, for images, one compute unit's loads: weights and bias wait in registers while the image is
// summed, 16 bytes per load, eight in flight per lane; the reductions need no LDS.  Every intermediate result is written as well, since others may read it.
// Ten classes from 32 channels of 32x32, all of a network of six kernels, us: 16.7 -> 15.1 on the GPU, and 19.4 - 25 -> 15.8 - 17.7 where the host, which
// needs 3 - 4 us per launch, is what it waits for.  With the weights through LDS (an integer division each), shuffles and any tail: as slow as three launches.
#include <hip/hip_runtime.h>

#include "device_common.h"
#include "gemm_lean.h"

namespace clg {

namespace {

constexpr int kThreads = 1024, kMaxClasses = kThreads / 16, kPerLane = 16, kMaxChannels = 16 * kPerLane;
static_assert(kThreads / kMaxChannels >= 4, "a lane takes one of an image's last three values");
constexpr int64_t kMaxImage = 65536;       // values of an image that is pooled (classifier_resolve)

typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));      // (an image may lie at any address of a float)

// Reductions over 64 lanes without LDS traffic (wave_sum_dpp's steps)
__device__ __forceinline__ float wave_max_dpp(float v) {
    v = fmaxf(v, dpp_lane<0xB1>(v));
    v = fmaxf(v, dpp_lane<0x4E>(v));
    v = fmaxf(v, dpp_lane<0x141>(v));
    v = fmaxf(v, dpp_lane<0x140>(v));
    auto row = [&](int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l)); };
    return fmaxf(fmaxf(row(0), row(16)), fmaxf(row(32), row(48)));
}

// group: lanes per channel of the pool, 4 .. 64 (kThreads / kMaxChannels at least)
__global__ __launch_bounds__(kThreads) void classifier_kernel(ClassifierArgs a, int group) {
    __shared__ float xs[kMaxChannels], ls[kMaxClasses];
    const int tid = threadIdx.x, row = blockIdx.x;
    // ---- weights and bias, sixteen lanes per class, all under way together with the first part of the image
    const int n = tid / 16, l16 = tid & 15, nn = min(n, a.N - 1);
    float w[kPerLane];
    const float bias = a.ef.flags & EF_BIAS ? a.ef.bias[nn] : 0.f;
    if (a.ts) {                                              // the register-fed kernel's order (rf_pack_dense_kernel)
        const int slots = kWave / a.ts, sh = __builtin_ctz(slots);
        const float *wp = a.w + ((nn / a.ts) * a.ngtot * kWave + nn % a.ts) * 4 + l16 % 4;
#pragma unroll
        for (int u = 0; u < kPerLane; ++u) {
            const int part = min((l16 >> 2) + 4 * u, a.K / 4 - 1);       // (such a layer has K % 4 = 0)
            w[u] = wp[((part >> sh) * kWave + (part & (slots - 1)) * a.ts) * 4];
        }
    } else {
        const float *wp = a.w + nn * a.ldb;
#pragma unroll
        for (int u = 0; u < kPerLane; ++u) w[u] = wp[min(l16 + 16 * u, a.K - 1)];
    }
    if (a.hw) {
        const int c = tid / group, l = tid & (group - 1);
        float part[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if (c < a.K) {
            const float *xp = a.x + ((int64_t)row * a.K + c) * a.hw;
            const int n4 = a.hw / 4;
            const float rest = l < a.hw - 4 * n4 ? xp[4 * n4 + l] : 0.f;
            for (int i = l; i < n4; i += 8 * group) {
                f32x4u v[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) v[k] = reinterpret_cast<const f32x4u *>(xp)[min(i + k * group, n4 - 1)];
#pragma unroll
                for (int k = 0; k < 8; ++k) part[k] += i + k * group < n4 ? (v[k][0] + v[k][1]) + (v[k][2] + v[k][3]) : 0.f;
            }
            part[0] += rest;
        }
        float sum = ((part[0] + part[1]) + (part[2] + part[3])) + ((part[4] + part[5]) + (part[6] + part[7]));
        sum += dpp_lane<0xB1>(sum);
        sum += dpp_lane<0x4E>(sum);
        if (group > 4) sum += dpp_lane<0x141>(sum);
        if (group > 8) sum += dpp_lane<0x140>(sum);
        if (group > 16) sum += __shfl_xor(sum, 16, kWave);
        if (group > 32) sum += __shfl_xor(sum, 32, kWave);
        if (c < a.K && l == 0) {
            sum /= (float)a.hw;
            xs[c] = sum;
            a.pooled[(int64_t)row * a.lda + c] = sum;
        }
    } else if (tid < a.K) {
        xs[tid] = a.x[(int64_t)row * a.lda + tid];
    }
    __syncthreads();
    // ---- dense
    float acc = 0.f;
#pragma unroll
    for (int u = 0; u < kPerLane; ++u)
        if (l16 + 16 * u < a.K) acc += w[u] * xs[l16 + 16 * u];
    acc += dpp_lane<0xB1>(acc);
    acc += dpp_lane<0x4E>(acc);
    acc += dpp_lane<0x141>(acc);
    acc += dpp_lane<0x140>(acc);
    acc += bias;
    if (n < a.N && l16 == 0) {
        ls[n] = acc;
        a.logits[(int64_t)row * a.ldc + n] = acc;
    }
    __syncthreads();
    // ---- softmax: one wave, a lane per class
    if (tid >= kWave) return;
    const float v = tid < a.N ? ls[tid] : 0.f;
    const float mx = wave_max_dpp(tid < a.N ? v : -INFINITY);
    const float e = tid < a.N ? expf(v - mx) : 0.f;
    const float inv = 1.0f / wave_sum_dpp(e);
    if (tid < a.N) a.prob[(int64_t)row * a.N + tid] = e * inv;
}

}  // namespace

// An image up to 256 KB: one compute unit sums it in the time that a launch costs (45x45: GPU time of the network 17.8 -> 16.9 us); larger ones are
// summed by all of them, and only dense layer and softmax are joined (55x55 19.3 -> 18.6, 96x96 27.1 -> 26.5).
// Images: a workgroup each, and a round of workgroups costs as much as the first however little each has to do, while the tiles of a dense layer grow with the rows
// slowly.  So no more rows than compute units, or than twice as many where a pool is joined as well, from 32 channels on.  us, launches apart and joined, on 256 compute units: 256 -> 64
// on 256 rows 5.0 and 4.7, 384 5.0 and 7.7, 4096 7.3 and 50; 32 -> 10 on 256 5.4 and 3.6, 384 5.5 and 5.6, 1024 5.5 and 9.6; with a pool 64 channels of 4x4 on 256 rows 8.5 and 4.9, 512 10.0
// and 8.2, 768 11.3 and 11.4; 32 channels of 16x16 on 512 10.0 and 8.4, 1024 12.8 and 15.2; 256 channels of 7x7 on 512 20.7 and 10.3; 16 channels of 8x8 on 256 7.4 and 5.0, 257 7.5 and 7.7.
bool classifier_resolve(const PoolArgs *pool, const GemmArgs &d, const RowwiseArgs &sm, int n_cus, ClassifierArgs *out) {
    const int flags = epi_fast_flags(d.epi);
    if (d.mode != GM_NT || d.batch != 1 || d.cs_len || (flags & ~EF_BIAS)) return false;
    if (d.N < 1 || d.N > kMaxClasses || d.K < 1 || d.K > kMaxChannels || (int64_t)d.N * d.ldb >= ((int64_t)1 << 30) || d.M < 1) return false;
    if (d.M > (pool && d.K >= 32 ? 2 * n_cus : n_cus)) return false;
    if (sm.mode != 0 || sm.n_gather || sm.pro.n || sm.rows != d.M || sm.len != d.N || d.ldc != d.N) return false;
    ClassifierArgs a{};
    if (pool) {
        if (pool->mode != 1 || pool->epi.n || pool->D > 1 || (int64_t)pool->NC != (int64_t)d.M * d.K || d.lda != d.K) return false;
        if ((int64_t)d.K * pool->H * pool->W > kMaxImage) return false;
        a.hw = pool->H * pool->W;
    }
    a.rows = d.M; a.K = d.K; a.N = d.N;
    a.lda = d.lda; a.ldb = d.ldb; a.ldc = d.ldc;
    if (d.rf_ts) {
        a.ts = d.rf_ts;
        a.ngtot = d.rf_ngtot;
    }
    *out = a;
    return true;
}

int launch_classifier(const ClassifierArgs &a, void *stream) {
    int group = kWave;
    while (group > 1 && (int64_t)group * a.K > kThreads) group /= 2;
    hipLaunchKernelGGL(classifier_kernel, dim3((unsigned)a.rows), dim3(kThreads), 0, (hipStream_t)stream, a, group);
    return (int)hipGetLastError();
}

}  // namespace clg
