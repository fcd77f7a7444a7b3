// Memory-bound kernels of the fused-operator set for gfx950: elementwise
// chains and embedding gather, softmax / layer norm with a fused prologue
// (wavefront shuffle reductions, one 64-lane wave per row), direct convolution
// for grouped and small-channel layers, pooling, layout copies.
//
// These operators move O(1) flops per byte (paper Sec. 5.1 lists them as the
// non-contraction part of the workloads), so the design rule is: every tensor
// is read once and written once, with consecutive lanes on consecutive
// addresses; anything elementwise rides along in registers.
#include <algorithm>
#include <type_traits>

#include <hip/hip_runtime.h>

#include "device_common.h"
#include "plane.h"

namespace clg {

// ------------------------------------------------------------------ elementwise
// y = steps(x) (or steps(table[ids])).  VEC = 4: numel % 4 == 0, and the four
// elements of a float4 share a bias channel layout the kernel can index:
// inner % 4 == 0 (same channel) or inner == 1 with C % 4 == 0 (four channels).
template <int VEC>
__global__ __launch_bounds__(256) void eltwise_kernel(EltwiseArgs a) {
    const int64_t n = a.numel / VEC;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const int64_t off = i * VEC;
        float v[VEC];
        const float *src = a.x + off;
        if (a.ids) {
            const int64_t row = off / a.row_len, col = off % a.row_len;
            int id = a.ids[row];
            id = id < 0 ? 0 : (id >= a.table_rows ? a.table_rows - 1 : id);
            src = a.x + (int64_t)id * a.row_len + col;
        }
        if constexpr (VEC == 4) {
            const float4 t = *reinterpret_cast<const float4 *>(src);
            v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
        } else {
            v[0] = src[0];
        }
#pragma unroll
        for (int q = 0; q < VEC; ++q) v[q] = apply_steps(a.epi, v[q], off + q, chan_of(a.epi, off + q));
        if constexpr (VEC == 4) {
            *reinterpret_cast<float4 *>(a.y + off) = make_float4(v[0], v[1], v[2], v[3]);
        } else {
            a.y[off] = v[0];
        }
    }
}

static bool aligned16(const void *p) { return ((uintptr_t)p & 15) == 0; }

int launch_eltwise(const EltwiseArgs &a, void *stream) {
    bool vec = a.numel % 4 == 0 && aligned16(a.x) && aligned16(a.y) && (!a.ids || a.row_len % 4 == 0);
    for (int s = 0; s < a.epi.n; ++s)
        if (a.epi.s[s].op == EPI_ADD && !aligned16(a.epi.s[s].ptr)) vec = false;
    const int64_t items = vec ? a.numel / 4 : a.numel;
    const int block = 256;
    const int grid = (int)std::min<int64_t>((items + block - 1) / block, 256 * 16);
    if (vec)
        hipLaunchKernelGGL(eltwise_kernel<4>, dim3(grid), dim3(block), 0, (hipStream_t)stream, a);
    else
        hipLaunchKernelGGL(eltwise_kernel<1>, dim3(grid), dim3(block), 0, (hipStream_t)stream, a);
    return (int)hipGetLastError();
}

// --------------------------------------------------------------- softmax / LN
// One wave per row; the row (after the fused prologue) is held in registers:
// ITEMS values per lane, element c = lane + 64 * t.  Reads x once, writes y
// once.  Softmax: max, sum of exp, normalise.  Layer norm: mean, then the
// biased variance of the centred values, then scale and shift.
template <int ITEMS>
__global__ __launch_bounds__(256) void rowwise_kernel(RowwiseArgs a) {
    const int lane = threadIdx.x & (kWave - 1);
    const int row = blockIdx.x * (blockDim.x / kWave) + (threadIdx.x / kWave);
    if (row >= a.rows) return;
    const float *xr = a.x + (int64_t)row * a.len;
    float *yr = a.y + (int64_t)row * a.len;
    float v[ITEMS];
#pragma unroll
    for (int t = 0; t < ITEMS; ++t) {
        const int c = lane + kWave * t;
        v[t] = 0.f;
        if (c < a.len) v[t] = apply_steps(a.pro, xr[c], (int64_t)row * a.len + c, c);
    }
    if (a.mode == 0) {
        float mx = -INFINITY;
#pragma unroll
        for (int t = 0; t < ITEMS; ++t)
            if (lane + kWave * t < a.len) mx = fmaxf(mx, v[t]);
        mx = wave_max(mx);
        float sum = 0.f;
#pragma unroll
        for (int t = 0; t < ITEMS; ++t) {
            v[t] = (lane + kWave * t < a.len) ? expf(v[t] - mx) : 0.f;
            sum += v[t];
        }
        sum = wave_sum(sum);
        const float inv = 1.0f / sum;
#pragma unroll
        for (int t = 0; t < ITEMS; ++t)
            if (lane + kWave * t < a.len) yr[lane + kWave * t] = v[t] * inv;
    } else {
        float sum = 0.f;
#pragma unroll
        for (int t = 0; t < ITEMS; ++t) sum += v[t];          // padding lanes hold 0
        const float mean = wave_sum(sum) / (float)a.len;
        float sq = 0.f;
#pragma unroll
        for (int t = 0; t < ITEMS; ++t) {
            const float d = (lane + kWave * t < a.len) ? v[t] - mean : 0.f;
            v[t] = d;
            sq += d * d;
        }
        const float var = wave_sum(sq) / (float)a.len;
        const float inv = 1.0f / sqrtf(var + a.eps);
#pragma unroll
        for (int t = 0; t < ITEMS; ++t) {
            const int c = lane + kWave * t;
            if (c < a.len) yr[c] = v[t] * inv * a.gamma[c] + a.beta[c];
        }
    }
}

// One workgroup (four waves) per row: for few, long rows (layer norm over 128 x 768,
// the 1 x 1000 softmax of a classifier) a wave per row leaves most of the chip
// idle and strings ITEMS dependent loads and exponentials behind each other.
// Each reduction is a wave reduction plus four partial values through LDS, added
// in wave order.  gamma / beta are fetched before the reductions.
template <int ITEMS>
__global__ __launch_bounds__(256) void rowwise_block_kernel(RowwiseArgs a) {
    __shared__ float part[2][4];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int row = blockIdx.x;
    const float *xr = a.x + (int64_t)row * a.len;
    float *yr = a.y + (int64_t)row * a.len;
    float v[ITEMS], ga[ITEMS], be[ITEMS];
#pragma unroll
    for (int t = 0; t < ITEMS; ++t) {
        const int c = tid + 256 * t;
        v[t] = 0.f;
        ga[t] = 0.f;
        be[t] = 0.f;
        if (c < a.len) {
            v[t] = apply_steps(a.pro, xr[c], (int64_t)row * a.len + c, c);
            if (a.mode == 1) {
                ga[t] = a.gamma[c];
                be[t] = a.beta[c];
            }
        }
    }
    auto block_sum = [&](float x, int slot) {
        x = wave_sum(x);
        if (lane == 0) part[slot][wave] = x;
        __syncthreads();
        return (part[slot][0] + part[slot][1]) + (part[slot][2] + part[slot][3]);
    };
    if (a.mode == 0) {
        float mx = -INFINITY;
#pragma unroll
        for (int t = 0; t < ITEMS; ++t)
            if (tid + 256 * t < a.len) mx = fmaxf(mx, v[t]);
        mx = wave_max(mx);
        if (lane == 0) part[0][wave] = mx;
        __syncthreads();
        mx = fmaxf(fmaxf(part[0][0], part[0][1]), fmaxf(part[0][2], part[0][3]));
        float sum = 0.f;
#pragma unroll
        for (int t = 0; t < ITEMS; ++t) {
            v[t] = (tid + 256 * t < a.len) ? expf(v[t] - mx) : 0.f;
            sum += v[t];
        }
        const float inv = 1.0f / block_sum(sum, 1);
#pragma unroll
        for (int t = 0; t < ITEMS; ++t)
            if (tid + 256 * t < a.len) yr[tid + 256 * t] = v[t] * inv;
    } else {
        float sum = 0.f;
#pragma unroll
        for (int t = 0; t < ITEMS; ++t) sum += v[t];          // padding lanes hold 0
        const float mean = block_sum(sum, 0) / (float)a.len;
        float sq = 0.f;
#pragma unroll
        for (int t = 0; t < ITEMS; ++t) {
            const float d = (tid + 256 * t < a.len) ? v[t] - mean : 0.f;
            v[t] = d;
            sq += d * d;
        }
        const float var = block_sum(sq, 1) / (float)a.len;
        const float inv = 1.0f / sqrtf(var + a.eps);
#pragma unroll
        for (int t = 0; t < ITEMS; ++t) {
            const int c = tid + 256 * t;
            if (c < a.len) yr[c] = v[t] * inv * ga[t] + be[t];
        }
    }
}

// Layer norm, a wave per row and a row per workgroup, for the transformer's shapes (128 rows of 768):
// every load of the row - the value, the fused bias and residual, gamma and beta, 16 bytes per lane
// each - is issued before anything is computed, so the kernel pays one memory round trip; the two
// reductions stay inside the wave (no LDS, no barrier).  The row comes from x with an optional
// [bias] [residual add] in front (the common form of a fused prologue), or is the sum of two or three
// gathered table rows (an embedding).  Same arithmetic as above: mean, biased variance of the centred
// values, scale and shift.  len % 4 == 0, len <= 256 * V4, all pointers 16-byte aligned.
// R: Ahead (the first kAheadWaves workgroups read ahead; a constant, so that the others wait for nothing to know that they do not) or NoAhead.
// P: SplitSum (x is the sum of a split contraction's partial results, in slice order, and its bias and residual, which saves the launch that would
// add them: 4.8 us between two kernels on 389 rows of 768) or NoSum.
template <int V4, class R, class P>
__global__ __launch_bounds__(64) void ln_wave_kernel(RowwiseArgs a, EpiFast ef, R ra, P parts) {
    constexpr bool SUM = std::is_same_v<P, SplitSum>;
    const int lane = threadIdx.x;
    int row = blockIdx.x;
    if constexpr (std::is_same_v<R, Ahead>) {
        row -= kAheadWaves;
        if (row < 0) return read_ahead(ra, (uint32_t)(blockIdx.x * kWave + lane), kAheadWaves * kWave);
    }
    const int len4 = a.len >> 2;
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    float4 v[V4], t1[V4], t2[V4], ga[V4], be[V4];
    const float4 *p0, *p1 = nullptr, *p2 = nullptr;
    if (a.n_gather) {
        auto row_of = [&](int k) {
            int id = a.gid[k][row];
            id = id < 0 ? 0 : (id >= a.tab_rows[k] ? a.tab_rows[k] - 1 : id);
            return reinterpret_cast<const float4 *>(a.tab[k] + (int64_t)id * a.len);
        };
        p0 = row_of(0);
        p1 = row_of(1);
        if (a.n_gather > 2) p2 = row_of(2);
    } else {
        if constexpr (SUM) p0 = reinterpret_cast<const float4 *>(parts.partial + (int64_t)row * a.len);
        else p0 = reinterpret_cast<const float4 *>(a.x + (int64_t)row * a.len);
        if (ef.flags & EF_BIAS) p1 = reinterpret_cast<const float4 *>(ef.bias);
        if (ef.flags & EF_ADD) p2 = reinterpret_cast<const float4 *>(ef.add + (int64_t)row * a.len);
    }
    const float4 *g4 = reinterpret_cast<const float4 *>(a.gamma), *b4 = reinterpret_cast<const float4 *>(a.beta);
#pragma unroll
    for (int q = 0; q < V4; ++q) {
        const int c = lane + kWave * q;
        const bool in = c < len4;
        const int cc = in ? c : 0;
        if constexpr (!SUM) v[q] = p0[cc];
        t1[q] = p1 ? p1[cc] : zero;
        t2[q] = p2 ? p2[cc] : zero;
        ga[q] = g4[cc];
        be[q] = b4[cc];
        if (!in) v[q] = t1[q] = t2[q] = zero;
    }
    if constexpr (SUM) {                                     // the reduction's own order: slice after slice, then bias, then residual
        float4 db[V4], da[V4];
        const float4 *d1 = reinterpret_cast<const float4 *>(parts.bias), *d2 = parts.add ? reinterpret_cast<const float4 *>(parts.add + (int64_t)row * a.len) : nullptr;
#pragma unroll
        for (int q = 0; q < V4; ++q) {
            const int cc = lane + kWave * q < len4 ? lane + kWave * q : 0;
            db[q] = d1 ? d1[cc] : zero;
            da[q] = d2 ? d2[cc] : zero;
            v[q] = zero;
        }
        constexpr int F = V4 <= 4 ? 4 : 2;                   // slices in flight
        const uint32_t step = (uint32_t)parts.numel / 4;
        for (int k = 0; k < parts.splitk; k += F) {
            float4 s[F][V4];
#pragma unroll
            for (int e = 0; e < F; ++e)
#pragma unroll
                for (int q = 0; q < V4; ++q) {
                    const int c = lane + kWave * q;
                    s[e][q] = p0[(uint32_t)min(k + e, parts.splitk - 1) * step + (uint32_t)(c < len4 ? c : 0)];
                }
#pragma unroll
            for (int e = 0; e < F; ++e)
#pragma unroll
                for (int q = 0; q < V4; ++q)
                    if (k + e < parts.splitk) { v[q].x += s[e][q].x; v[q].y += s[e][q].y; v[q].z += s[e][q].z; v[q].w += s[e][q].w; }
        }
#pragma unroll
        for (int q = 0; q < V4; ++q) {
            v[q].x = v[q].x + db[q].x + da[q].x; v[q].y = v[q].y + db[q].y + da[q].y;
            v[q].z = v[q].z + db[q].z + da[q].z; v[q].w = v[q].w + db[q].w + da[q].w;
            if (lane + kWave * q >= len4) v[q] = zero;
        }
    }
    float sum = 0.f;
#pragma unroll
    for (int q = 0; q < V4; ++q) {
        // the operators' own order, one rounding each: (x + bias) + residual, or (row0 + row1) + row2
        if (p1) { v[q].x += t1[q].x; v[q].y += t1[q].y; v[q].z += t1[q].z; v[q].w += t1[q].w; }
        if (p2) { v[q].x += t2[q].x; v[q].y += t2[q].y; v[q].z += t2[q].z; v[q].w += t2[q].w; }
        sum += (v[q].x + v[q].y) + (v[q].z + v[q].w);
    }
    const float mean = wave_sum_dpp(sum) / (float)a.len;
    float sq = 0.f;
#pragma unroll
    for (int q = 0; q < V4; ++q) {
        if (lane + kWave * q < len4) {
            v[q].x -= mean; v[q].y -= mean; v[q].z -= mean; v[q].w -= mean;
        }
        sq += (v[q].x * v[q].x + v[q].y * v[q].y) + (v[q].z * v[q].z + v[q].w * v[q].w);
    }
    const float inv = 1.0f / sqrtf(wave_sum_dpp(sq) / (float)a.len + a.eps);
    float4 *y4 = reinterpret_cast<float4 *>(a.y + (int64_t)row * a.len);
#pragma unroll
    for (int q = 0; q < V4; ++q) {
        const int c = lane + kWave * q;
        if (c < len4)
            y4[c] = make_float4(v[q].x * inv * ga[q].x + be[q].x, v[q].y * inv * ga[q].y + be[q].y,
                                v[q].z * inv * ga[q].z + be[q].z, v[q].w * inv * ga[q].w + be[q].w);
    }
}

// Whether the one-round-trip layer norm takes the shape and the prologue; fills *ef with the prologue's common form.
static bool ln_wave_shape_ok(const RowwiseArgs &a, EpiFast *ef) {
    if (a.mode != 1 || a.len % 4 || a.len > 256 * 8 || a.len < 64 || a.rows > 4096) return false;
    ef->flags = 0;
    if (a.n_gather) {
        for (int k = 0; k < a.n_gather; ++k)
            if (a.tab_rows[k] < 1) return false;
        return a.n_gather == 2 || a.n_gather == 3;
    }
    *ef = make_epi_fast(a.pro);
    if (ef->flags & ~(EF_BIAS | EF_ADD)) return false;
    return !(ef->flags & EF_BIAS) || (a.pro.bias_inner == 1 && a.pro.bias_c == a.len);
}

// ... and, with every pointer bound, the alignment.
static bool ln_wave_ok(const RowwiseArgs &a, EpiFast *ef) {
    if (!ln_wave_shape_ok(a, ef)) return false;
    auto al = [](const void *p) { return ((uintptr_t)p & 15) == 0; };
    if (!al(a.y) || !al(a.gamma) || !al(a.beta)) return false;
    if (a.n_gather) {
        for (int k = 0; k < a.n_gather; ++k)
            if (!al(a.tab[k])) return false;
        return true;
    }
    return al(a.x) && (!(ef->flags & EF_BIAS) || al(ef->bias)) && (!(ef->flags & EF_ADD) || al(ef->add));
}

bool rowwise_reads_ahead(const RowwiseArgs &a) {
    EpiFast ef{};
    return ln_wave_shape_ok(a, &ef);
}

// Rows longer than 64 * 32: same arithmetic, the row is re-read per pass.
__global__ __launch_bounds__(256) void rowwise_long_kernel(RowwiseArgs a) {
    const int lane = threadIdx.x & (kWave - 1);
    const int row = blockIdx.x * (blockDim.x / kWave) + (threadIdx.x / kWave);
    if (row >= a.rows) return;
    const float *xr = a.x + (int64_t)row * a.len;
    float *yr = a.y + (int64_t)row * a.len;
    auto val = [&](int c) { return apply_steps(a.pro, xr[c], (int64_t)row * a.len + c, c); };
    if (a.mode == 0) {
        float mx = -INFINITY;
        for (int c = lane; c < a.len; c += kWave) mx = fmaxf(mx, val(c));
        mx = wave_max(mx);
        float sum = 0.f;
        for (int c = lane; c < a.len; c += kWave) sum += expf(val(c) - mx);
        sum = wave_sum(sum);
        const float inv = 1.0f / sum;
        for (int c = lane; c < a.len; c += kWave) yr[c] = expf(val(c) - mx) * inv;
    } else {
        float sum = 0.f;
        for (int c = lane; c < a.len; c += kWave) sum += val(c);
        const float mean = wave_sum(sum) / (float)a.len;
        float sq = 0.f;
        for (int c = lane; c < a.len; c += kWave) {
            const float d = val(c) - mean;
            sq += d * d;
        }
        const float inv = 1.0f / sqrtf(wave_sum(sq) / (float)a.len + a.eps);
        for (int c = lane; c < a.len; c += kWave) yr[c] = (val(c) - mean) * inv * a.gamma[c] + a.beta[c];
    }
}

template <class R, class P>
static void launch_ln_wave(const RowwiseArgs &a, const EpiFast &ef, const R &r, const P &p, int waves, hipStream_t s) {
    const int v4 = (a.len / 4 + kWave - 1) / kWave;
    if (v4 <= 1) hipLaunchKernelGGL((ln_wave_kernel<1, R, P>), dim3(waves), dim3(kWave), 0, s, a, ef, r, p);
    else if (v4 <= 2) hipLaunchKernelGGL((ln_wave_kernel<2, R, P>), dim3(waves), dim3(kWave), 0, s, a, ef, r, p);
    else if (v4 <= 4) hipLaunchKernelGGL((ln_wave_kernel<4, R, P>), dim3(waves), dim3(kWave), 0, s, a, ef, r, p);
    else hipLaunchKernelGGL((ln_wave_kernel<8, R, P>), dim3(waves), dim3(kWave), 0, s, a, ef, r, p);
}

bool rowwise_sums_shape_ok(const RowwiseArgs &a) {
    EpiFast ef{};
    return !a.n_gather && ln_wave_shape_ok(a, &ef);
}

bool rowwise_sums_ok(const RowwiseArgs &a, const SplitSum &s) {
    RowwiseArgs b = a;
    b.x = s.partial;
    EpiFast ef{};
    return !a.n_gather && ln_wave_ok(b, &ef) && ((uintptr_t)s.bias & 15) == 0 && ((uintptr_t)s.add & 15) == 0;
}

int launch_rowwise_sum(const RowwiseArgs &a, const SplitSum &sum, const Ahead *ahead, void *stream) {
    const EpiFast ef = make_epi_fast(a.pro);
    if (!rowwise_sums_ok(a, sum)) return (int)hipErrorInvalidValue;
    if (ahead && ahead->n) launch_ln_wave(a, ef, *ahead, sum, a.rows + kAheadWaves, (hipStream_t)stream);
    else launch_ln_wave(a, ef, NoAhead{}, sum, a.rows, (hipStream_t)stream);
    return (int)hipGetLastError();
}

int launch_rowwise(const RowwiseArgs &a, const Ahead *ahead, void *stream) {
    const int block = 256, rows_per_block = block / kWave;
    const dim3 grid((a.rows + rows_per_block - 1) / rows_per_block);
    const int items = (a.len + kWave - 1) / kWave;
    hipStream_t s = (hipStream_t)stream;
    EpiFast ef{};
    if (ln_wave_ok(a, &ef)) {                                      // layer norm in one memory round trip
        // (read-ahead waves first, so that theirs are the first loads to leave: behind the rows all of BERT-base, 200 rows, took 797 instead of 785 us)
        if (ahead && ahead->n) launch_ln_wave(a, ef, *ahead, NoSum{}, a.rows + kAheadWaves, s);
        else launch_ln_wave(a, ef, NoAhead{}, NoSum{}, a.rows, s);
        return (int)hipGetLastError();
    }
    if (a.n_gather) return (int)hipErrorInvalidValue;              // only the kernel above gathers
    if (a.len > 256 && a.len <= 2048 && a.rows <= 1024) {          // few long rows: a workgroup per row
        const int bi = (a.len + 255) / 256;
        if (bi <= 2) hipLaunchKernelGGL(rowwise_block_kernel<2>, dim3(a.rows), dim3(256), 0, s, a);
        else if (bi <= 4) hipLaunchKernelGGL(rowwise_block_kernel<4>, dim3(a.rows), dim3(256), 0, s, a);
        else hipLaunchKernelGGL(rowwise_block_kernel<8>, dim3(a.rows), dim3(256), 0, s, a);
        return (int)hipGetLastError();
    }
    if (items <= 1) hipLaunchKernelGGL(rowwise_kernel<1>, grid, dim3(block), 0, s, a);
    else if (items <= 2) hipLaunchKernelGGL(rowwise_kernel<2>, grid, dim3(block), 0, s, a);
    else if (items <= 4) hipLaunchKernelGGL(rowwise_kernel<4>, grid, dim3(block), 0, s, a);
    else if (items <= 8) hipLaunchKernelGGL(rowwise_kernel<8>, grid, dim3(block), 0, s, a);
    else if (items <= 16) hipLaunchKernelGGL(rowwise_kernel<16>, grid, dim3(block), 0, s, a);
    else if (items <= 32) hipLaunchKernelGGL(rowwise_kernel<32>, grid, dim3(block), 0, s, a);
    else hipLaunchKernelGGL(rowwise_long_kernel, grid, dim3(block), 0, s, a);
    return (int)hipGetLastError();
}

// ------------------------------------------------------------ direct convolution
// One thread per output pixel and COB consecutive output channels of one group:
// every input value loaded is used COB times; the weights of those channels are
// wave-uniform (scalar loads).  blockIdx.y = channel block, blockIdx.z = image.
template <int COB>
__global__ __launch_bounds__(256) void direct_conv_kernel(DirectConvArgs a) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    const int npix = a.HO * a.WO;
    const int Cg = a.C / a.G, Og = a.O / a.G;
    const int co0 = blockIdx.y * COB;
    const int g = co0 / Og;
    const int n = blockIdx.z;
    if (p >= npix) return;
    const int oh = p / a.WO, ow = p % a.WO;
    float acc[COB];
#pragma unroll
    for (int j = 0; j < COB; ++j) acc[j] = 0.f;
    const float *xg = a.x + ((int64_t)n * a.C + (int64_t)g * Cg) * a.H * a.W;
    const float *wg = a.w + (int64_t)co0 * Cg * a.KH * a.KW;
    const int wstride = Cg * a.KH * a.KW;
    for (int ci = 0; ci < Cg; ++ci) {
        for (int kh = 0; kh < a.KH; ++kh) {
            const int ih = oh * a.sh - a.ph + kh;
            if (ih < 0 || ih >= a.H) continue;
            for (int kw = 0; kw < a.KW; ++kw) {
                const int iw = ow * a.sw - a.pw + kw;
                if (iw < 0 || iw >= a.W) continue;
                const float xv = xg[((int64_t)ci * a.H + ih) * a.W + iw];
                const float *wp = wg + (ci * a.KH + kh) * a.KW + kw;
#pragma unroll
                for (int j = 0; j < COB; ++j) acc[j] = fmaf(xv, wp[j * wstride], acc[j]);
            }
        }
    }
#pragma unroll
    for (int j = 0; j < COB; ++j) {
        const int co = co0 + j;
        const int64_t off = ((int64_t)n * a.O + co) * npix + p;
        a.y[off] = apply_steps(a.epi, acc[j], off, co);
    }
}

// 3x3 convolutions of a few channels per group (ResNeXt's): four output rows at one column and COB output channels per
// thread, so that an input value is loaded once for 3 COB .. 9 COB products and neighbouring lanes read neighbouring
// columns.  On the matrix cores a group of four fills an eighth of a 32x32 tile's products and a quarter of a 16x16
// one's; the vector units do no work for other groups.  The products of an output are added in the order of
// direct_conv_kernel.  Bounds: 9 Cg fused multiply-adds per output at 39 T/s (12 us for a layer of ResNeXt-50 at batch 32),
// and the traffic.  Batch 32, 128 channels in groups of four at 56x56: 28 us, on the matrix cores 64; 256 in groups of
// eight at 28x28: 29, 36; from groups of 16 on the matrix cores are faster (21 us).
constexpr int kGroupRows = 4;
template <int COB, int S>
__global__ __launch_bounds__(256) void grouped3_kernel(DirectConvArgs a, uint32_t items, uint32_t quads) {
    constexpr int R = (kGroupRows - 1) * S + 3;              // input rows
    constexpr uint32_t kOut = 0x80000000u;                   // beyond the buffer: loaded as zero
    const uint32_t t = blockIdx.x * 256u + threadIdx.x;
    const bool live = t < items;
    const uint32_t tt = live ? t : 0;
    const int n = (int)(tt / quads), q = (int)(tt - (uint32_t)n * quads);
    const int qr = q / a.WO, ow = q - qr * a.WO, oh0 = qr * kGroupRows;
    const int Cg = a.C / a.G, co0 = blockIdx.y * COB, g = co0 / (a.O / a.G);
    const int HW = a.H * a.W, ih0 = oh0 * S - a.ph, iw0 = ow * S - a.pw;
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.x), (short)0, (int)((int64_t)a.N * a.C * HW * 4), 0x00020000);
    uint32_t off[R][3];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const int ih = ih0 + r, iw = iw0 + k;
            off[r][k] = ih >= 0 && ih < a.H && iw >= 0 && iw < a.W ? (uint32_t)(n * a.C * HW + ih * a.W + iw) * 4u : kOut;
        }
    float acc[kGroupRows][COB];
#pragma unroll
    for (int r = 0; r < kGroupRows; ++r)
#pragma unroll
        for (int j = 0; j < COB; ++j) acc[r][j] = 0.f;
    const float *w = a.w + (int64_t)co0 * Cg * 9;            // wave-uniform: scalar loads
    const int wstride = Cg * 9;
    for (int ci = 0; ci < Cg; ++ci) {
        const int so = (g * Cg + ci) * HW * 4;
        float x[R][3];
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int k = 0; k < 3; ++k) x[r][k] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)off[r][k], so, 0));
#pragma unroll
        for (int f = 0; f < 9; ++f)
#pragma unroll
            for (int j = 0; j < COB; ++j)
#pragma unroll
                for (int r = 0; r < kGroupRows; ++r) acc[r][j] = fmaf(x[r * S + f / 3][f % 3], w[j * wstride + ci * 9 + f], acc[r][j]);
    }
    const int npix = a.HO * a.WO, bytes = (int)((int64_t)a.N * a.O * npix * 4);
    const auto ydst = __builtin_amdgcn_make_buffer_rsrc(a.y, (short)0, bytes, 0x00020000);
    const auto rsum = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.ef.add), (short)0, bytes, 0x00020000);
    float v[kGroupRows * COB], bv[kGroupRows * COB], av[kGroupRows * COB];
    uint32_t ob[kGroupRows];
#pragma unroll
    for (int r = 0; r < kGroupRows; ++r) {
        ob[r] = live && oh0 + r < a.HO ? (uint32_t)(n * a.O * npix + (oh0 + r) * a.WO + ow) * 4u : kOut;
#pragma unroll
        for (int j = 0; j < COB; ++j) {
            v[r * COB + j] = acc[r][j];
            bv[r * COB + j] = (a.ef.flags & EF_BIAS) ? a.ef.bias[co0 + j] : 0.f;
            av[r * COB + j] = 0.f;
        }
    }
    if (a.ef.flags & EF_ADD) {
#pragma unroll
        for (int r = 0; r < kGroupRows; ++r)
#pragma unroll
            for (int j = 0; j < COB; ++j)
                av[r * COB + j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsum, (int)ob[r], (co0 + j) * npix * 4, 0));
    }
    fused_tail<kGroupRows * COB>(a.ef, v, bv, av);
#pragma unroll
    for (int r = 0; r < kGroupRows; ++r)
#pragma unroll
        for (int j = 0; j < COB; ++j) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v[r * COB + j]), ydst, (int)ob[r], (co0 + j) * npix * 4, 0);
}

// Groups of 2 .. 32 channels with a multiple of four outputs each; 31-bit byte offsets.  At every size: over 370 layers of 8 - 1024
// channels, 4x4 to 56x56 and 1 to 32 images it takes 0.16 to 0.98 of the general direct kernel's time (64 channels in
// groups of four at 7x7, one image, where 14 lanes of a workgroup have work: 5.2 instead of 8.7 us).
static bool grouped3_ok(const DirectConvArgs &a) {
    const int Cg = a.C / a.G, Og = a.O / a.G;
    return !a.transposed && !a.pro_relu && !(a.ef.flags & EF_GENERIC) && a.G > 1 && Cg > 1 && Cg <= 32 && Og % 4 == 0 && a.KH == 3 && a.KW == 3 && a.sh == a.sw &&
           a.sh <= 2 && (int64_t)a.N * a.C * a.H * a.W < ((int64_t)1 << 29) && (int64_t)a.N * a.O * a.HO * a.WO < ((int64_t)1 << 29) && a.O / 4 <= 65535;
}

template <int COB>
static void launch_grouped3(const DirectConvArgs &a, hipStream_t s) {
    const uint32_t quads = (uint32_t)((a.HO + kGroupRows - 1) / kGroupRows * a.WO), items = quads * (uint32_t)a.N;
    const dim3 grid((items + 255) / 256, (unsigned)(a.O / COB));
    if (a.sh == 1) hipLaunchKernelGGL((grouped3_kernel<COB, 1>), grid, dim3(256), 0, s, a, items, quads);
    else hipLaunchKernelGGL((grouped3_kernel<COB, 2>), grid, dim3(256), 0, s, a, items, quads);
}

// One output of a transposed convolution in gather form (w is [C][O][KH][KW]): output row oh takes
// filter row kh from input row (oh + ph - kh) / sh where that division is exact and the row exists;
// the same along the width.
__device__ __forceinline__ float convt_gather(const DirectConvArgs &a, int n, int co, int oh, int ow) {
    const float *xn = a.x + (int64_t)n * a.C * a.H * a.W;
    const float *wo = a.w + (int64_t)co * a.KH * a.KW;
    const int64_t xstride = (int64_t)a.H * a.W, wstride = (int64_t)a.O * a.KH * a.KW;
    float acc = 0.f;
    for (int kh = 0; kh < a.KH; ++kh) {
        const int th = oh + a.ph - kh;
        if (th < 0 || th % a.sh != 0 || th / a.sh >= a.H) continue;
        const int ih = th / a.sh;
        for (int kw = 0; kw < a.KW; ++kw) {
            const int tw = ow + a.pw - kw;
            if (tw < 0 || tw % a.sw != 0 || tw / a.sw >= a.W) continue;
            const float *xp = xn + (int64_t)ih * a.W + tw / a.sw;
            const float *wp = wo + kh * a.KW + kw;
            for (int ci = 0; ci < a.C; ++ci) acc = fmaf(xp[ci * xstride], wp[ci * wstride], acc);
        }
    }
    return acc;
}

// Transposed convolution of any filter size, stride and pad: one thread per output pixel, blockIdx.y =
// output channel, blockIdx.z = image.  The kernel that runs what the phase-decomposed MFMA kernels refuse
// (a filter size that the stride does not divide).
__global__ __launch_bounds__(256) void direct_convt_kernel(DirectConvArgs a) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    const int npix = a.HO * a.WO;
    const int co = blockIdx.y, n = blockIdx.z;
    if (p >= npix) return;
    const int64_t off = ((int64_t)n * a.O + co) * npix + p;
    a.y[off] = apply_steps(a.epi, convt_gather(a, n, co, p / a.WO, p % a.WO), off, co);
}

// 4x4 filters, stride 2, pad 1, one to four output channels (the layer that makes an image): a lane owns the 2x2 outputs around
// each of R input positions, one above the other, which need R + 2 rows of three inputs, so 3 R + 6 loads feed 16 R O products, all of them useful; the 16 O
// weights of an input channel are wave-uniform (scalar loads).  The matrix cores do this layer with 3 of 16 or 12 of 16 rows filled and
// nine taps of which a phase uses four.  The WK waves of a workgroup share its 64 lanes' positions and split the input channels; they meet in
// LDS, and each finishes whole rows of pixel pairs.  Bounds: the products at 39 T/s (5 us for 64 -> 3 channels at 32x32, 64 images), and for few images
// the weights' round trips, one behind the other.  That layer on the fp32 matrix cores and here: 16 images 7.0 and 6.5 us, 32 images
// 12.0 and 8.7, 64 images 21.2 and 12.6, 256 images 74 and 38; up to eight images the matrix cores are faster (3.8 - 4.9 us).
// Error against 64 bits, rms, 0.82 - 0.86 of theirs: a sum is eight chains (five layers of 33 - 256 channels).
template <int O, int R, int WK>
__global__ __launch_bounds__(WK * kWave) void few_convt_kernel(DirectConvArgs a, uint32_t items) {
    constexpr uint32_t kOut = 0x80000000u;                   // beyond the buffer: loaded as zero, not stored
    constexpr int X = 3 * (R + 2);
    __shared__ float red[WK][4 * R * O][kWave];
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const uint32_t t = blockIdx.x * (uint32_t)kWave + lane;
    const bool live = t < items;
    const uint32_t tt = live ? t : 0;
    const int HW = a.H * a.W, per_image = (a.H + R - 1) / R * a.W;
    const int n = (int)(tt / (uint32_t)per_image), q = (int)(tt - (uint32_t)n * per_image);
    const int i = q / a.W * R, j = q - i / R * a.W;
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.x), (short)0, (int)((int64_t)a.N * a.C * HW * 4), 0x00020000);
    uint32_t off[X];
#pragma unroll
    for (int k = 0; k < X; ++k) {
        const int ih = i - 1 + k / 3, iw = j - 1 + k % 3;
        off[k] = live && ih >= 0 && ih < a.H && iw >= 0 && iw < a.W ? (uint32_t)(n * a.C * HW + ih * a.W + iw) * 4u : kOut;
    }
    float acc[2 * R][2][O];                                  // output row, column
#pragma unroll
    for (int r = 0; r < 2 * R; ++r)
#pragma unroll
        for (int o = 0; o < O; ++o) acc[r][0][o] = acc[r][1][o] = 0.f;
    const int per = (a.C + WK - 1) / WK, c0 = wave * per, c1 = min(c0 + per, a.C);
    float x[2][X];
    auto load = [&](int set, int c) {
#pragma unroll
        for (int k = 0; k < X; ++k) x[set][k] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)off[k], min(c, a.C - 1) * HW * 4, 0));
    };
    // Weights: 16 at a time (an output channel), the next ones on their way while these are used.  Scalar loads return out of order, so a wait is for all
    // of them: the next load leaves behind the first product of this one's.  (All of a channel's loaded where they are used: 64 images 13.0 instead of 12.6 us.)
    float wv[2][16];
    auto load_w = [&](int set, int k) {
        const float *w = a.w + (int64_t)min(k, a.C * O - 1) * 16;
#pragma unroll
        for (int f = 0; f < 16; ++f) wv[set][f] = w[f];
    };
    auto step = [&](int set, int c) {
#pragma unroll
        for (int o = 0; o < O; ++o) {
            const int ring = (set * O + o) & 1;
#pragma unroll
            for (int f = 0; f < 16; ++f) {
                // filter rows 0 and 2 make the lower output row, from the input row below and this one; 1 and 3 the upper one, from this one and the one above
                const int kh = f >> 2, kw = f & 3, r = kh & 1 ? 0 : 1, s = kw & 1 ? 0 : 1, ih = kh == 0 ? 2 : (kh == 3 ? 0 : 1), iw = kw == 0 ? 2 : (kw == 3 ? 0 : 1);
#pragma unroll
                for (int y = 0; y < R; ++y) acc[2 * y + r][s][o] = fmaf(x[set][(y + ih) * 3 + iw], wv[ring][f], acc[2 * y + r][s][o]);
                if (f == 0) {
                    __builtin_amdgcn_sched_barrier(0);
                    load_w(ring ^ 1, c * O + o + 1);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    load_w(0, c0 * O);
    load(0, c0);
    for (int c = c0; c < c1; c += 2) {
        load(1, c + 1);
        step(0, c);
        load(0, c + 2);
        if (c + 1 < c1) step(1, c + 1);
    }
#pragma unroll
    for (int r = 0; r < 2 * R; ++r)
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int o = 0; o < O; ++o) red[wave][(2 * r + s) * O + o][lane] = acc[r][s][o];
    __syncthreads();
    const int npix = a.HO * a.WO, bytes = (int)((int64_t)a.N * O * npix * 4);
    const auto ydst = __builtin_amdgcn_make_buffer_rsrc(a.y, (short)0, bytes, 0x00020000);
    const auto rsum = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.ef.add), (short)0, bytes, 0x00020000);
#pragma unroll 1
    for (int e = wave; e < 2 * R * O; e += WK) {             // (channel, output row)
        const int r = e & (2 * R - 1), o = e / (2 * R);
        const bool in = live && 2 * i + r < a.HO;
        float v[2] = {0.f, 0.f}, bv[2], av[2] = {0.f, 0.f};
#pragma unroll
        for (int k = 0; k < WK; ++k) {
            v[0] += red[k][2 * r * O + o][lane];
            v[1] += red[k][(2 * r + 1) * O + o][lane];
        }
        // taps outside the image were multiplied as zeros, which an infinite weight makes a NaN: such outputs are gathered
        if (in && !(fabsf(v[0]) < INFINITY)) v[0] = convt_gather(a, n, o, 2 * i + r, 2 * j);
        if (in && !(fabsf(v[1]) < INFINITY)) v[1] = convt_gather(a, n, o, 2 * i + r, 2 * j + 1);
        const uint32_t ob = in ? (uint32_t)((n * O + o) * npix + (2 * i + r) * a.WO + 2 * j) * 4u : kOut;
        bv[0] = bv[1] = (a.ef.flags & EF_BIAS) ? a.ef.bias[o] : 0.f;
        if (a.ef.flags & EF_ADD) {
            av[0] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsum, (int)ob, 0, 0));
            av[1] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsum, (int)ob, 4, 0));
        }
        fused_tail<2>(a.ef, v, bv, av);
        typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
        __builtin_amdgcn_raw_buffer_store_b64(u32x2{__float_as_uint(v[0]), __float_as_uint(v[1])}, ydst, (int)ob, 0, 0);
    }
}

// 31-bit byte offsets.  At every size: over 26 layers 1.3 (one channel of one value) to 35 times as fast as the general kernel (512 channels at 2x2: 19 us, 663).
static bool few_convt_ok(const DirectConvArgs &a) {
    return a.transposed && !(a.ef.flags & EF_GENERIC) && a.G == 1 && a.O >= 1 && a.O <= 4 && a.C >= 1 && a.KH == 4 && a.KW == 4 && a.sh == 2 && a.sw == 2 && a.ph == 1 && a.pw == 1 &&
           a.HO == 2 * a.H && a.WO == 2 * a.W && (int64_t)a.N * a.C * a.H * a.W < ((int64_t)1 << 29) && (int64_t)a.N * a.O * a.HO * a.WO < ((int64_t)1 << 29);
}

template <int O, int R, int WK>
static void launch_few_convt_as(const DirectConvArgs &a, hipStream_t s) {
    const uint32_t items = (uint32_t)(a.N * ((a.H + R - 1) / R) * a.W), groups = (items + kWave - 1) / kWave;
    hipLaunchKernelGGL((few_convt_kernel<O, R, WK>), dim3(groups), dim3(WK * kWave), 0, s, a, items);
}

// One position per lane while that makes no more than two workgroups per compute unit, two above (64 -> 3 channels at 32x32, us with one and
// two: 16 images 6.5 and 8.7, 32 images 8.7 and 9.0, 64 images 14.0 and 12.6, 256 images 47 and 39; 16 -> 1 at 256x256, four images, 17.2 and 12.0).
// Four waves and sixteen instead of eight, one position: 16 images 9.0 and 6.4, 32 images 9.4 and 8.9.
template <int O>
static void launch_few_convt(const DirectConvArgs &a, hipStream_t s) {
    constexpr int kCUs = 256;                                // of an MI355X
    if (((int64_t)a.N * a.H * a.W + kWave - 1) / kWave <= 2 * kCUs) launch_few_convt_as<O, 1, 8>(a, s);
    else launch_few_convt_as<O, 2, 8>(a, s);
}

template <int KS>
__global__ __launch_bounds__(256) void depthwise_kernel(DirectConvArgs a) {
    depthwise_body<KS>(a, blockIdx.x * 256u + threadIdx.x);
}

bool depthwise_fast_ok(const DirectConvArgs &a) {
    return !a.transposed && a.G == a.C && a.O == a.C && a.KH == a.KW && (a.KH == 3 || a.KH == 5 || a.KH == 7) &&
           (int64_t)a.N * a.C * a.HO * a.WO < ((int64_t)1 << 31) && (int64_t)a.H * a.W < ((int64_t)1 << 31);
}

int launch_direct_conv(const DirectConvArgs &a_in, void *stream) {
    DirectConvArgs a = a_in;
    a.ef = make_epi_fast(a.epi);
    if (depthwise_fast_ok(a)) {
        const int64_t total = (int64_t)a.N * a.C * a.HO * a.WO;
        const dim3 grid((unsigned)((total + 255) / 256));
        if (a.KH == 3) hipLaunchKernelGGL(depthwise_kernel<3>, grid, dim3(256), 0, (hipStream_t)stream, a);
        else if (a.KH == 5) hipLaunchKernelGGL(depthwise_kernel<5>, grid, dim3(256), 0, (hipStream_t)stream, a);
        else hipLaunchKernelGGL(depthwise_kernel<7>, grid, dim3(256), 0, (hipStream_t)stream, a);
        return (int)hipGetLastError();
    }
    if (a.pro_relu) return (int)hipErrorInvalidValue;      // only the depthwise kernel applies the relu
    const int npix = a.HO * a.WO;
    const int Og = a.O / a.G;
    const int block = npix >= 256 ? 256 : (npix > 64 ? 128 : 64);
    hipStream_t s = (hipStream_t)stream;
    if (a.transposed) {
        if (a.G != 1 || a.O > 65535 || a.N > 65535) return (int)hipErrorInvalidValue;
        if (few_convt_ok(a)) {
            if (a.O == 1) launch_few_convt<1>(a, s);
            else if (a.O == 2) launch_few_convt<2>(a, s);
            else if (a.O == 3) launch_few_convt<3>(a, s);
            else launch_few_convt<4>(a, s);
            return (int)hipGetLastError();
        }
        hipLaunchKernelGGL(direct_convt_kernel, dim3((npix + block - 1) / block, a.O, a.N), dim3(block), 0, s, a);
        return (int)hipGetLastError();
    }
    if (grouped3_ok(a)) {
        if (Og % 8 == 0) launch_grouped3<8>(a, s);
        else launch_grouped3<4>(a, s);
        return (int)hipGetLastError();
    }
    if (Og % 4 == 0) {
        const dim3 grid((npix + block - 1) / block, a.O / 4, a.N);
        hipLaunchKernelGGL(direct_conv_kernel<4>, grid, dim3(block), 0, s, a);
    } else {
        const dim3 grid((npix + block - 1) / block, a.O, a.N);
        hipLaunchKernelGGL(direct_conv_kernel<1>, grid, dim3(block), 0, s, a);
    }
    return (int)hipGetLastError();
}

// ------------------------------------------------------------------------ pooling
template <bool AVG>
__global__ __launch_bounds__(256) void window_pool_kernel(PoolArgs a) {
    window_pool_body<AVG>(a, blockIdx.x * 256u + threadIdx.x);
}

// Several independent thread-per-output problems in one launch: the depthwise convolutions and window
// pools that the branches of a cell apply to the same few tensors.  Workgroup -> problem by a
// wave-uniform look-up, then exactly the code the problem runs alone (same results bit for bit).
__global__ __launch_bounds__(256) void plane_multi_kernel(PlaneMultiArgs m) {
    const int bx = blockIdx.x;
    int k = 0;
#pragma unroll
    for (int i = 0; i + 1 < kMaxPlaneRegion; ++i) k += bx >= m.block_end[i] ? 1 : 0;
    const uint32_t i = (uint32_t)(bx - (k ? m.block_end[k - 1] : 0)) * 256u + threadIdx.x;
    switch (m.kind[k]) {
    case 3: depthwise_body<3>(m.p[k].dw, i); break;
    case 5: depthwise_body<5>(m.p[k].dw, i); break;
    case 7: depthwise_body<7>(m.p[k].dw, i); break;
    case 10: window_pool_body<false>(m.p[k].pool, i); break;
    default: window_pool_body<true>(m.p[k].pool, i); break;
    }
}

bool plane_region_pool_ok(const PoolArgs &a) {
    return (a.mode == 0 || a.mode == 2) && a.D >= 1 && a.KD >= 1 && a.sd >= 1 && a.DO >= 1 &&
           (int64_t)a.NC * a.DO * a.HO * a.WO < ((int64_t)1 << 31) && (int64_t)a.D * a.H * a.W < ((int64_t)1 << 31);
}

int launch_plane_region(const PlaneMultiArgs &m_in, void *stream) {
    PlaneMultiArgs m = m_in;
    if (m.n < 2 || m.n > kMaxPlaneRegion) return (int)hipErrorInvalidValue;
    int64_t end = 0;
    for (int k = 0; k < m.n; ++k) {
        int64_t total;
        if (m.kind[k] == 3 || m.kind[k] == 5 || m.kind[k] == 7) {
            DirectConvArgs &a = m.p[k].dw;
            if (!depthwise_fast_ok(a) || a.KH != m.kind[k]) return (int)hipErrorInvalidValue;
            a.ef = make_epi_fast(a.epi);
            total = (int64_t)a.N * a.C * a.HO * a.WO;
        } else if (m.kind[k] == 10 || m.kind[k] == 11) {
            const PoolArgs &a = m.p[k].pool;
            if (!plane_region_pool_ok(a) || a.mode != (m.kind[k] == 10 ? 0 : 2)) return (int)hipErrorInvalidValue;
            total = (int64_t)a.NC * a.DO * a.HO * a.WO;
        } else {
            return (int)hipErrorInvalidValue;
        }
        end += (total + 255) / 256;
        if (end >= ((int64_t)1 << 31)) return (int)hipErrorInvalidValue;
        m.block_end[k] = (int32_t)end;
    }
    for (int k = m.n; k < kMaxPlaneRegion; ++k) m.block_end[k] = (int32_t)end;
    hipLaunchKernelGGL(plane_multi_kernel, dim3((unsigned)end), dim3(256), 0, (hipStream_t)stream, m);
    return (int)hipGetLastError();
}

// one wave per (n, c) plane
__global__ __launch_bounds__(256) void global_avg_pool_kernel(PoolArgs a) {
    const int lane = threadIdx.x & (kWave - 1);
    const int nc = blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
    if (nc >= a.NC) return;
    const int hw = a.H * a.W;
    const float *xp = a.x + (int64_t)nc * hw;
    float sum = lane < hw ? xp[lane] : 0.f;
    if (hw > kWave) {
        // eight loads in flight (one at a time a 32x32 image is sixteen round trips long: 6.6 us inside a network, 3.2 back to back)
        float part[8] = {sum, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        for (int i = lane + kWave; i < hw; i += 8 * kWave) {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int o = i + k * kWave;
                const float v = xp[min(o, hw - 1)];
                part[k] += o < hw ? v : 0.f;
            }
        }
        sum = ((part[0] + part[1]) + (part[2] + part[3])) + ((part[4] + part[5]) + (part[6] + part[7]));
    }
    sum = wave_sum(sum);
    if (lane == 0) a.y[nc] = sum / (float)hw;
}

int launch_pool(const PoolArgs &a, void *stream) {
    hipStream_t s = (hipStream_t)stream;
    if (a.D < 1 || a.KD < 1 || a.sd < 1 || a.DO < 1) return (int)hipErrorInvalidValue;
    if ((int64_t)a.NC * a.DO * a.HO * a.WO >= ((int64_t)1 << 31) || (int64_t)a.D * a.H * a.W >= ((int64_t)1 << 31))
        return (int)hipErrorInvalidValue;                      // the window kernels index with 32 bits
    if (a.mode == 0 || a.mode == 2) {
        const int64_t total = (int64_t)a.NC * a.DO * a.HO * a.WO;
        const dim3 grid((unsigned)((total + 255) / 256));
        if (a.mode == 0) hipLaunchKernelGGL(window_pool_kernel<false>, grid, dim3(256), 0, s, a);
        else hipLaunchKernelGGL(window_pool_kernel<true>, grid, dim3(256), 0, s, a);
    } else {
        hipLaunchKernelGGL(global_avg_pool_kernel, dim3((a.NC + 3) / 4), dim3(256), 0, s, a);
    }
    return (int)hipGetLastError();
}

// --------------------------------------------------------------------- layout copy
__global__ __launch_bounds__(256) void layout_kernel(LayoutArgs a) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t o = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; o < a.numel; o += stride) {
        int64_t rem = o, src = 0;
        for (int d = a.ndim - 1; d >= 0; --d) {
            const int64_t q = rem / a.out_dims[d];
            src += (rem - q * a.out_dims[d]) * a.in_strides[d];
            rem = q;
        }
        a.y[o] = a.x[src];
    }
}

int launch_layout(const LayoutArgs &a, void *stream) {
    const int grid = (int)std::min<int64_t>((a.numel + 255) / 256, 256 * 16);
    hipLaunchKernelGGL(layout_kernel, dim3(grid), dim3(256), 0, (hipStream_t)stream, a);
    return (int)hipGetLastError();
}

// ------------------------------------------------------------------------- concat
// Output element o = (r, col): the operand whose column range holds col supplies it.
template <int VEC>
__global__ __launch_bounds__(256) void concat_kernel(ConcatArgs a) {
    const int64_t n = a.outer * a.row / VEC;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const int64_t o = i * VEC;
        const int64_t r = o / a.row;
        int64_t col = o - r * a.row;
        int s = 0;
        while (s < a.n - 1 && col >= a.chunk[s]) col -= a.chunk[s++];
        const float *src = a.src[s] + r * a.chunk[s] + col;
        if constexpr (VEC == 4) *reinterpret_cast<float4 *>(a.y + o) = *reinterpret_cast<const float4 *>(src);
        else a.y[o] = *src;
    }
}

int launch_concat(const ConcatArgs &a, void *stream) {
    bool vec = aligned16(a.y);
    for (int s = 0; s < a.n; ++s) vec = vec && a.chunk[s] % 4 == 0 && aligned16(a.src[s]);
    const int64_t items = a.outer * a.row / (vec ? 4 : 1);
    const int grid = (int)std::min<int64_t>((items + 255) / 256, 256 * 16);
    if (vec) hipLaunchKernelGGL(concat_kernel<4>, dim3(grid), dim3(256), 0, (hipStream_t)stream, a);
    else hipLaunchKernelGGL(concat_kernel<1>, dim3(grid), dim3(256), 0, (hipStream_t)stream, a);
    return (int)hipGetLastError();
}

// ------------------------------------------------------- measurer scratch operands
__global__ __launch_bounds__(256) void fill_kernel(float *p, int64_t n, uint64_t seed) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        uint64_t z = seed + 0x9E3779B97F4A7C15ull * (uint64_t)(i + 1);    // splitmix64 finaliser
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        z ^= z >> 31;
        p[i] = (float)((z >> 40) & 0xFFFFFF) * (2.0f / 16777216.0f) - 1.0f;
    }
}

int launch_fill(float *p, int64_t n, uint64_t seed, void *stream) {
    const int grid = (int)std::min<int64_t>((n + 255) / 256, 256 * 16);
    hipLaunchKernelGGL(fill_kernel, dim3(grid > 0 ? grid : 1), dim3(256), 0, (hipStream_t)stream, p, n, seed);
    return (int)hipGetLastError();
}

// Row ids for a gather: uniform over [0, rows) from the same counter hash, so that a measured
// gather touches rows spread over the whole table, as a real one does.
__global__ __launch_bounds__(256) void fill_ids_kernel(int32_t *p, int64_t n, int32_t rows, uint64_t seed) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        uint64_t z = seed + 0x9E3779B97F4A7C15ull * (uint64_t)(i + 1);
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        z ^= z >> 31;
        p[i] = (int32_t)(((z >> 32) * (uint64_t)(rows > 0 ? rows : 1)) >> 32);
    }
}

int launch_fill_ids(int32_t *p, int64_t n, int32_t rows, uint64_t seed, void *stream) {
    const int grid = (int)std::min<int64_t>((n + 255) / 256, 256 * 16);
    hipLaunchKernelGGL(fill_ids_kernel, dim3(grid > 0 ? grid : 1), dim3(256), 0, (hipStream_t)stream, p, n, rows, seed);
    return (int)hipGetLastError();
}

__global__ void empty_kernel() {}

int launch_empty(void *stream) {
    hipLaunchKernelGGL(empty_kernel, dim3(1), dim3(64), 0, (hipStream_t)stream);
    return (int)hipGetLastError();
}

}  // namespace clg
