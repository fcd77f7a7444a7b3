// First layers (few input channels, a filter of up to eight columns, even column stride) on the bf16
// matrix cores with exactly split operands (gemm_b3.h tells how and why).
//
// Three channels do not fill the 16 values of k of an MFMA, and gathering one value per filter tap
// bound the register-fed kernel: 7x7 stride 2, 3 -> 64 channels at 224x224 and batch 32 took 206 us, for
// 7.6 GFLOP and 122 MB.  Here k runs along an input row: for a fixed (channel, depth tap, filter row)
// the eight values x[2 ow - pad .. + 7] are eight consecutive bf16 in LDS, which a lane reads with one
// 16-byte load at a 4-byte aligned address; columns past the filter's width meet zero weights (an infinity or NaN among
// them makes the result a NaN, and results that are not finite are computed again as a fp32 chain of the filter's own columns).
// An MFMA takes two such rows (one per lane half).  A workgroup copies the input patch of its 128 (256) output
// pixels once, split into the three planes; the patch is 2.5 times its output in values, so the split costs
// little, and the kernel is bound by its stores (64 channels of output per 3 of input).
#include <algorithm>

#include "gemm_b3.h"

namespace clg {

namespace {

// Steps of weights in registers: a step is 0.16 us of MFMAs, a weight comes from the L2 in 0.4 us or more.  (With two
// sets the 224x224 layer took 12.9 us at batch 1.)
constexpr int kRing = 3;

typedef uint32_t u32x4a __attribute__((ext_vector_type(4), aligned(4)));

// WM 32-row tiles x (4 / WM) column tiles of 64 pixels.  UM: pairs of patch values per thread and stage.
template <int WM, int UM>
__global__ __launch_bounds__(256, 2) void b3_first_kernel(B3Args p) {
    constexpr int TN = 2;
    extern __shared__ uint32_t b3_patch[];                                 // [2 buffers][3 planes][cps * prow rows][pxw / 2 words]
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1), half = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int wm = wave % WM, wn = wave / WM;

    const int tile = b3_xcd_remap(blockIdx.x, gridDim.x);
    const int nt = (int)b3_div((uint32_t)tile, p.d_tile), mg = tile - nt * p.tile_div;
    const int mt = min(mg * WM + wm, p.mtiles - 1);
    const bool m_live = mg * WM + wm < p.mtiles;
    const int i0 = mt * 32;
    const int im = (int)b3_div((uint32_t)nt, p.d_strip), tin = nt - im * p.tiles_strip;
    const int ty = (int)b3_div((uint32_t)tin, p.d_ho), tx = tin - ty * p.tiles_x;
    int n = im, od = 0;
    if (p.DO > 1) {
        n = (int)b3_div((uint32_t)im, p.d_do);
        od = im - n * p.DO;
    }
    const int oy0 = ty * p.TH, ox0 = tx * p.TW;
    const int id0 = od * p.sd - p.pd, ih0 = oy0 * p.sh - p.ph, iw0 = ox0 * p.sw - p.pwd;

    const int w_bytes = p.stages * p.steps * (3 * kWave * 16);
    const auto wsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(reinterpret_cast<const char *>(p.w)) + (int64_t)mt * w_bytes, (short)0, w_bytes, 0x00020000);
    uint32_t wo = (uint32_t)lane * 16;
    u32x4 ar[kRing][3];
    auto load_w = [&](int set) {
#pragma unroll
        for (int k = 0; k < 3; ++k) ar[set][k] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(wsrc, (int)wo, k * (kWave * 16), 0));
        wo += 3 * kWave * 16;
    };
#pragma unroll
    for (int r = 0; r + 1 < kRing; ++r) load_w(r);

    // ---- patch: item = pair of neighbouring columns of a row (channel of the stage or depth tap, input row)
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p.x), (short)0, p.x_bytes, 0x00020000);
    const int rows = p.cps * p.prow, words = p.pxw / 2, PL = rows * words;
    uint32_t off0[UM], off1[UM];
#pragma unroll
    for (int u = 0; u < UM; ++u) {
        const int item = tid + u * 256;
        const int r = (int)b3_div((uint32_t)item, p.d_pw), xw = item - r * words;
        const int cp = (int)b3_div((uint32_t)r, p.d_rpi), ih = ih0 + r - cp * p.prow, iw = iw0 + 2 * xw;
        const int id = id0 + cp;                                           // KD > 1: the stage's planes are depth taps
        const bool in = item < PL && ih >= 0 && ih < p.H && (p.KD == 1 || (id >= 0 && id < p.D));
        const int32_t o = (n * p.img_stride + (p.KD == 1 ? cp * p.cs + id0 * p.HW : id * p.HW) + ih * p.W + iw) * 4;
        off0[u] = in && iw >= 0 && iw < p.W ? (uint32_t)o : kB3Out;
        off1[u] = in && iw + 1 >= 0 && iw + 1 < p.W ? (uint32_t)(o + 4) : kB3Out;
    }
    float xv[UM][2];
    auto load = [&](int st) {                                              // (several stages: one channel each)
        const int so = min(st, p.stages - 1) * p.cs * 4;
#pragma unroll
        for (int u = 0; u < UM; ++u) {
            xv[u][0] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)off0[u], so, 0));
            xv[u][1] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)off1[u], so, 0));
        }
    };
    auto store = [&](int buf) {
        uint32_t *dst = b3_patch + buf * 3 * PL;
#pragma unroll
        for (int u = 0; u < UM; ++u) {
            const int item = tid + u * 256;
            uint32_t h, m, l;
            b3_split2(xv[u][0], xv[u][1], h, m, l);
            if (item < PL) {
                dst[item] = h;
                dst[PL + item] = m;
                dst[2 * PL + item] = l;
            }
        }
    };
    load(0);

    // ---- this lane's pixels
    int sbase[TN];
    uint32_t ob[TN];
#pragma unroll
    for (int t = 0; t < TN; ++t) {
        const int jl = (wn * TN + t) * 32 + l32;
        const int y = (int)b3_div((uint32_t)jl, p.d_tw), x = jl - y * p.TW;
        const int yc = min(y, p.TH - 1);                                   // pixels past the tile read its last row
        sbase[t] = yc * p.sh * words + x * (p.sw / 2);
        const uint32_t o = (uint32_t)(n * p.ons + od * p.npix + (oy0 + y) * p.WO + ox0 + x + 4 * half * p.ocs) * 4;
        ob[t] = m_live && y < p.TH && oy0 + y < p.HO && ox0 + x < p.WO ? o : kB3Out;
    }
    f32x16v acc[TN], acs[TN];
#pragma unroll
    for (int t = 0; t < TN; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][r] = acs[t][r] = 0.f;

    for (int st = 0; st < p.stages; ++st) {
        const int buf = st & 1;
        store(buf);
        if (st + 1 < p.stages) load(st + 1);
        lds_barrier();
        const uint32_t *P0 = b3_patch + buf * 3 * PL;
        // filter rows 2 q and 2 q + 1 of the stage, as (plane, row); past the last one: the last one again, with zero weights
        int kh0 = 0, r0 = 0, kh1 = 1, r1 = 1;
        if (p.KHe == 1) {
            kh1 = 0;
            r1 = p.prow;
        }
        const int last = (p.cps - 1) * p.prow + p.KHe - 1;
        // (Columns past the filter and rows past the last one meet zero weights and are multiplied as they are.  An infinity or NaN among them makes the result a
        // NaN, and such results are computed again below; clearing them took two dozen instructions for twelve MFMAs.)
        auto step = [&](auto sc) {
            constexpr int s = sc.value;
            const int ro = min(half ? r1 : r0, last) * words;
            bf16x8 b[TN][3], a[3];
#pragma unroll
            for (int t = 0; t < TN; ++t)
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    b[t][k] = __builtin_bit_cast(bf16x8, (u32x4)*reinterpret_cast<const u32x4a *>(P0 + k * PL + sbase[t] + ro));
            load_w((s + kRing - 1) % kRing);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < 3; ++k) a[k] = __builtin_bit_cast(bf16x8, ar[s][k]);
            constexpr int PA[6] = {0, 2, 0, 1, 1, 0}, PB[6] = {0, 0, 2, 1, 0, 1};
#pragma unroll
            for (int m = 0; m < 6; ++m)
#pragma unroll
                for (int t = 0; t < TN; ++t) {
                    f32x16v &c = m == 0 ? acc[t] : acs[t];
                    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[PA[m]], b[t][PB[m]], c, 0, 0, 0);
                }
            // two filter rows on; behind a plane's last row comes the next plane
            kh0 += 2; r0 += 2;
            while (kh0 >= p.KHe) { kh0 -= p.KHe; r0 += p.prow - p.KHe; }
            kh1 += 2; r1 += 2;
            while (kh1 >= p.KHe) { kh1 -= p.KHe; r1 += p.prow - p.KHe; }
        };
        for (int q = 0; q < p.steps; q += kRing) b3_for<kRing>(step);        // (a multiple of kRing steps)
    }

    // ---- tail and stores (as in b3_kernel)
    float out[TN * 16], bv[TN * 16], av[TN * 16];
    const auto ydst = __builtin_amdgcn_make_buffer_rsrc(p.y, (short)0, (int)(p.c_numel * 4), 0x00020000);
    const auto rsum = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p.ef.add), (short)0, (int)(p.c_numel * 4), 0x00020000);
    const auto rbias = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p.ef.bias), (short)0, p.Cout * 4, 0x00020000);
    const int left = p.Cout - i0 - 4 * half;
#pragma unroll
    for (int n = 0; n < TN * 16; ++n) {
        out[n] = acc[n / 16][n % 16] + acs[n / 16][n % 16];
        bv[n] = av[n] = 0.f;
    }
    const uint32_t bad = b3_doubtful<TN * 16>(out);
    if (p.ef.flags & EF_BIAS) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float v = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rbias, (i0 + 4 * half) * 4, (8 * (r / 4) + r % 4) * 4, 0));
#pragma unroll
            for (int t = 0; t < TN; ++t) bv[t * 16 + r] = v;
        }
    }
    if (p.ef.flags & EF_ADD) {
#pragma unroll
        for (int n = 0; n < TN * 16; ++n) {
            const int rr = 8 * (n % 16 / 4) + n % 4;
            av[n] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsum, (int)(rr < left ? ob[n / 16] : kB3Out), (i0 + rr) * p.ocs * 4, 0));
        }
    }
    fused_tail<TN * 16>(p.ef, out, bv, av);
#pragma unroll
    for (int n = 0; n < TN * 16; ++n) {
        const int rr = 8 * (n % 16 / 4) + n % 4;
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(out[n]), ydst, (int)(rr < left ? ob[n / 16] : kB3Out), (i0 + rr) * p.ocs * 4, 0);
    }

    // ---- doubtful results once more as a fp32 chain (as in b3_kernel)
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(bad != 0) == 0, 1)) return;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll 1
    for (int r = 0; r < TN * 16; ++r) {
        const int rr = 8 * (r % 16 / 4) + r % 4, i = i0 + 4 * half + rr;
        const int jl = (wn * TN + r / 16) * 32 + l32, y = (int)b3_div((uint32_t)jl, p.d_tw), oh = oy0 + y, ow = ox0 + jl - y * p.TW;
        if (!(bad >> r & 1) || !m_live || rr >= left || y >= p.TH || oh >= p.HO || ow >= p.WO) continue;
        float v = 0.f;
        const u32x4 *row = reinterpret_cast<const u32x4 *>(p.w) + (int64_t)mt * p.stages * p.steps * 3 * kWave + (4 * half + rr);
        for (int st = 0; st < p.stages; ++st)
            for (int f = 0; f < p.cps * p.KH && v == v; ++f) {             // filter row of the stage
                const int cp = f / p.KH, ih = oh * p.sh - p.ph + f - cp * p.KH;
                const int c = p.KD == 1 ? cp : st, id = p.KD == 1 ? id0 : id0 + cp;
                const u32x4 *entry = row + ((int64_t)st * p.steps + f / 2) * (3 * kWave) + f % 2 * 32;
                for (int kw = 0; kw < p.KW; ++kw) {
                    const int iw = ow * p.sw - p.pwd + kw;
                    const bool in = id >= 0 && id < p.D && ih >= 0 && ih < p.H && iw >= 0 && iw < p.W;
                    v = fmaf(in ? p.x[(int64_t)n * p.img_stride + (int64_t)c * p.cs + id * p.HW + ih * p.W + iw] : 0.f, b3_weight(entry, kw), v);
                }
            }
        const uint32_t o = (uint32_t)(n * p.ons + od * p.npix + oh * p.WO + ow + i * p.ocs);
        float val[1] = {v}, b1[1] = {p.ef.flags & EF_BIAS ? p.ef.bias[i] : 0.f}, a1[1] = {p.ef.flags & EF_ADD ? p.ef.add[o] : 0.f};
        fused_tail<1>(p.ef, val, b1, a1);
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(val[0]), ydst, (int)(o * 4), 0, 0);
    }
}

// One thread per (row tile, stage, step, lane): filter row 2 * step + lane / 32 of the stage, columns 0..7.
__global__ __launch_bounds__(256) void b3_first_pack_kernel(const float *w, u32x4 *dst, B3Args p) {
    const int64_t d = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t s = d >> 6;
    if (s >= p.pack_steps) return;
    const int lane = (int)(d & 63);
    const int q = (int)(s % p.steps), st = (int)((s / p.steps) % p.stages), mt = (int)(s / p.steps / p.stages);
    const int row = 2 * q + lane / 32, i = mt * 32 + lane % 32;
    const int cp = row / p.KH, kh = row - cp * p.KH;
    const int c = p.KD == 1 ? cp : st, kd = p.KD == 1 ? 0 : cp;
    u32x4 pl[3];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        float v[2];
#pragma unroll
        for (int f = 0; f < 2; ++f) {
            const int kw = 2 * e + f;
            v[f] = mt < p.mtiles && i < p.Cout && cp < p.cps && kw < p.KW
                       ? w[((((int64_t)i * p.Cin + c) * p.KD + kd) * p.KH + kh) * p.KW + kw] : 0.f;
        }
        uint32_t h, m, l;
        b3_split2_full(v[0], v[1], h, m, l);
        pl[0][e] = h;
        pl[1][e] = m;
        pl[2][e] = l;
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) dst[(s * 3 + k) * kWave + lane] = pl[k];
}

template <int WM>
int launch_first_wm(const B3Args &a, hipStream_t s) {
    const int pairs = a.cps * a.prow * (a.pxw / 2), um = (pairs + 255) / 256;
    const size_t lds = (size_t)(a.stages > 1 ? 2 : 1) * 3 * pairs * 4;
    const dim3 grid((unsigned)(a.mgroups * a.ntiles));
    if (um <= 6) hipLaunchKernelGGL((b3_first_kernel<WM, 6>), grid, dim3(256), lds, s, a);
    else if (um <= 12) {
        if (lds > 64 * 1024) {
            static LdsLimit limit;
            const hipError_t e = limit.raise((const void *)b3_first_kernel<WM, 12>);
            if (e != hipSuccess) return (int)e;
        }
        hipLaunchKernelGGL((b3_first_kernel<WM, 12>), grid, dim3(256), lds, s, a);
    } else return (int)hipErrorInvalidValue;
    return (int)hipGetLastError();
}

}  // namespace

bool first_resolve(const GemmArgs &g, B3Args *out) {
    if (g.mode != GM_CONV || g.rf_groups > 1 || g.Cin > 4 || g.KW < 2 || g.KW > 8 || g.sw % 2 || g.KH > 8) return false;
    const bool depth = g.D > 1 || g.KD > 1;
    B3Args a{};
    a.epi = g.epi;
    a.c_numel = g.c_numel;
    a.tile = B3_FIRST;
    a.taps = g.KH * g.KW;
    a.splitk = 1;
    a.groups = a.phases = 1;
    a.Cin = g.Cin; a.Cout = g.Cout; a.KH = a.KHe = g.KH; a.KW = a.KWe = g.KW;
    a.H = g.H; a.W = g.W; a.HW = g.H * g.W; a.HO = g.HO; a.WO = a.WOe = g.WO;
    a.sh = g.sh; a.sw = g.sw; a.ph = g.ph; a.pwd = g.pw;
    a.D = depth ? g.D : 1; a.KD = depth ? g.KD : 1; a.DO = depth ? g.DO : 1;
    a.sd = depth ? g.sd : 1; a.pd = depth ? g.pd : 0;
    if (a.KD == 1 && a.pd != 0) return false;
    a.cs = a.D * a.HW;
    a.img_stride = g.Cin * a.cs;
    if ((int64_t)g.Nimg * g.Cin * a.cs >= ((int64_t)1 << 29) || g.c_numel >= ((int64_t)1 << 29)) return false;
    a.x_bytes = (int32_t)((int64_t)g.Nimg * g.Cin * a.cs * 4);
    a.Nimg = g.Nimg * a.DO;
    a.npix = g.HO * g.WO;
    a.ocs = a.DO * a.npix;
    a.ons = g.Cout * a.ocs;
    a.tiles_m = a.mtiles = (a.Cout + 31) / 32;
    // a stage: all channels, or all depth taps of one channel
    a.cps = a.KD == 1 ? g.Cin : a.KD;
    a.stages = a.KD == 1 ? 1 : g.Cin;
    a.steps = ((a.cps * a.KH + 1) / 2 + kRing - 1) / kRing * kRing;
    const int wm = a.mtiles >= 2 ? 2 : 1, bn = 64 * (4 / wm);
    a.mgroups = (a.mtiles + wm - 1) / wm;
    double best = -1;
    for (int tw = 4; tw <= 32; ++tw) {
        const int th = bn / tw, tx = (a.WO + tw - 1) / tw, ty = (a.HO + th - 1) / th;
        const int prow = (th - 1) * a.sh + a.KH, pxw = ((tw - 1) * a.sw + 8 + 1) / 2 * 2;
        const int pairs = a.cps * prow * (pxw / 2);
        if (pairs > 12 * 256 || (size_t)(a.stages > 1 ? 2 : 1) * 3 * pairs * 4 > 150 * 1024) continue;
        const double cost = (double)tx * ty * (bn * (double)a.steps + 2.0 * pairs);
        if (best >= 0 && cost >= best) continue;
        best = cost;
        a.TW = tw; a.TH = th; a.tiles_x = tx; a.tiles_y = ty; a.prow = prow; a.pxw = pxw;
    }
    if (best < 0) return false;
    a.tiles_strip = a.tiles_x * a.tiles_y;
    const int64_t nt = (int64_t)a.tiles_strip * a.Nimg;
    if (nt * a.mgroups >= ((int64_t)1 << 30)) return false;
    a.ntiles = (int)nt;
    a.jmajor = 1;
    a.tile_div = a.mgroups;
    const int pairs = a.cps * a.prow * (a.pxw / 2);
    if (!b3_set_div(&a.d_tile, a.tile_div, nt * a.mgroups) || !b3_set_div(&a.d_strip, a.tiles_strip, nt) || !b3_set_div(&a.d_ho, a.tiles_x, a.tiles_strip) ||
        !b3_set_div(&a.d_do, a.DO, a.Nimg) || !b3_set_div(&a.d_pw, a.pxw / 2, pairs + 12 * 256) || !b3_set_div(&a.d_rpi, a.prow, pairs + 12 * 256) ||
        !b3_set_div(&a.d_tw, a.TW, bn))
        return false;
    a.pack_steps = (int64_t)a.mtiles * a.stages * a.steps + kRing - 1;      // (and kRing - 1 steps of zeros; the kernel does not read behind its stream)
    *out = a;
    return true;
}

int launch_b3_first_pack(const B3Args &a, const float *w, void *dst, hipStream_t s) {
    const int64_t threads = a.pack_steps * kWave;
    hipLaunchKernelGGL(b3_first_pack_kernel, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s, w, (u32x4 *)dst, a);
    return (int)hipGetLastError();
}

int launch_b3_first(const B3Args &a, hipStream_t s) { return a.mtiles >= 2 ? launch_first_wm<2>(a, s) : launch_first_wm<1>(a, s); }

}  // namespace clg
