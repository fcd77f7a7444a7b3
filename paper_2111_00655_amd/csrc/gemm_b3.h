// Contractions on the bf16 matrix cores with fp32 operands and fp32 results
// ("b3": every operand as the exact sum of three bf16 values).
//
// gfx950's fp32 MFMA runs at 157 TFLOP/s, its bf16 MFMA at 2.5 PFLOP/s.  An fp32
// number x has 24 significant bits, a bf16 has 8, and
//     h = bf16(x), m = bf16(x - h), l = bf16(x - h - m)      (round to nearest)
// holds x exactly (both differences are exact in fp32).  A product is then
//     a b = ah bh + ah bm + am bh + am bm + ah bl + al bh    (+ am bl + al bm + al bl)
// where every product of two bf16 values is exact in the fp32 accumulator's
// format and the three terms left out are 2^-24 |a b| together at most (2^-27.4 rms,
// random in sign): less than what one rounding of a fp32 accumulation loses.
// The leading products have an accumulator of their own, which is rounded once per 16 values of k instead of once per 2 or 4: against
// float64 the results have 0.31 to 0.91 of the error of the fp32 MFMA kernel in their place (K = 8 to 3072, inputs with and without
// a relu; 3x3 convolution, K = 576: 8e-8 of the result's norm against 2.5e-7).  A sum that is a single product
// is the one case in which they are further off: 2.6e-8 against 2.5e-8 in the mean, 8.9e-8 against 6.0e-8 at worst.
// Six bf16 MFMAs of 32x32x16 take 192 cycles of a matrix core, eight fp32 MFMAs of 32x32x2 take 512: 417 instead
// of 157 TFLOP/s.
//
// At the ends of the range.  An infinity has NaN in its small planes, and where a block of rows spans several groups it
// meets the zero weights of its neighbours; a finite input within 2^-9 of the largest float rounds to an infinity (a weight
// does not: b3_split2_full); an operand below 2^-110 loses its last bits (it is off by less than 2^-126).  So a
// result that is not finite, or below 2^-90 without being zero, is computed again as a fp32 chain of the operands themselves, by the lane
// that owns it (`again` below): nothing in the loop pays for it, and a chain ends at its first NaN.  What
// stays: a weight below 2^-110 is held to 2^-134.
//
// Structure.  A wave owns 32 output rows (channels) and TN tiles of 32 output columns
// (pixels); a workgroup has WM waves along the rows, WN along the columns and WK that
// share a tile and split K.
//  * Weights are constants: they are split and packed once per plan in the order in which a
//    wave consumes them (32 rows x 16 values of k = three 1 KB planes, 16 bytes per lane), and
//    are read straight into registers, R - 1 steps ahead.
//  * The input is staged through LDS once per 16 * SC channels, double-buffered: a lane loads eight
//    channels of one position (coalesced along the positions), splits them (5.5 vector
//    instructions per value) and writes three 16-byte pieces.  A wave that shares its rows and columns with no other one stages for itself, without
//    barriers, and a 1x1 filter's unit then is a fragment as it is (DIRECT).  The positions ("slots") are the
//    input patch that the tile's output pixels touch, so a 3x3 filter loads and splits a value once
//    instead of nine times; a tap is a constant offset into the patch, and padding is a slot
//    that stays zero.
//  * What a tile covers: a strip of TW output columns is walked row by row, image after
//    image (or depth slice after depth slice), and a tile is BN consecutive pixels of
//    that walk; small images share a tile, large ones are cut into strips so that the patch
//    stays compact.
//  * First layers have too few channels to fill the 16 values of k of an MFMA: they have a kernel of
//    their own (gemm_b3_first.hip), which takes eight neighbouring pixels of an input row as k.
//  * 3-D: a tile's walk passes depth slice after depth slice; the depth taps of a channel block are
//    stages of their own, one input plane each (DEPTH).
//  * Transposed convolution: the stride^2 sub-pixel phases are stride-1 convolutions over the
//    same input patch; a phase is a further block of output rows with its own tap offset.
#pragma once

#include <type_traits>
#include <utility>

#include <hip/hip_runtime.h>

#include "device_common.h"
#include "lds_limit.h"

namespace clg {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2v __attribute__((ext_vector_type(2)));
typedef float f32x16v __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <int WM_, int WN_, int WK_, int TN_, int CW1_ = 2>
struct B3Cfg {
    static constexpr int WM = WM_, WN = WN_, WK = WK_, TN = TN_, CW1 = CW1_;
    static constexpr int NW = WM * WN * WK, NT = NW * kWave;
    static constexpr int BM = 32 * WM, BN = 32 * TN * WN;
    static constexpr int RED = WK > 1 ? NW * TN * 16 * kWave * 4 : 0;      // bytes in which the K-waves meet
    static constexpr bool PRIV = WM == 1 && WN == 1;                       // a wave stages what it alone reads: no barrier in the loop
};
using B3L = B3Cfg<4, 2, 1, 2, 4>;    // 128 x 128, eight waves
using B3LM = B3Cfg<2, 2, 1, 2>;      // 64 x 128
using B3M = B3Cfg<2, 1, 2, 2>;       // 64 x 64, two K-waves
using B3M8 = B3Cfg<2, 1, 4, 2, 1>;   // 64 x 64, four K-waves
using B3M12 = B3Cfg<3, 1, 4, 2, 3>;  // 96 x 64, four K-waves (dense layers)
using B3S = B3Cfg<1, 1, 4, 2>;       // 32 x 64, four K-waves
using B3SS = B3Cfg<1, 1, 4, 1>;      // 32 x 32, four K-waves
using B3G = B3Cfg<1, 4, 1, 2>;       // 32 x 256: few output rows (grouped convolutions)
using B3G2 = B3Cfg<1, 4, 1, 1>;      // 32 x 128

// A wave of S and SS tiles is alone with its rows and columns and stages for itself.  For 1x1 filters its staging unit (a lane: eight channels of one position)
// already is the fragment that it multiplies, so nothing goes through LDS (DIRECT); otherwise it does, in order and without barriers.
template <class C, int TAPS, bool DENSE>
constexpr bool b3_direct() { return C::PRIV && TAPS == 1 && !DENSE; }
// 16-channel blocks per K-wave and stage
template <class C, int TAPS, bool DENSE>
constexpr int b3_cw() { return TAPS != 1 || b3_direct<C, TAPS, DENSE>() ? 1 : C::CW1; }
// Register sets of the weight stream (a set is loaded R - 1 steps ahead), of the input (loaded D stages ahead of its split) and of
// input fragments (BB = 2: read a step ahead).  Deeper rings gave nothing (128x128 tiles, R = 8 and D = 2, 46 -> 51 us) or cost waves
// (32x32 tiles, R = 8 and D = 4, 9.4 -> 10.9 us): what a compute unit waits for is its own instruction stream and the L1, not a single load.
template <class C, int TAPS>
constexpr int b3_ring() { return TAPS == 9 ? 3 : (TAPS == 4 || C::PRIV || C::BM == 128 ? 4 : 2); }
template <class C, int TAPS, bool DENSE>
constexpr int b3_deep() { return b3_direct<C, TAPS, DENSE>() ? 2 : 1; }
template <class C, int TAPS>
constexpr int b3_ahead() {
    if (C::PRIV) return TAPS != 1 && C::TN > 1 ? 1 : 2;
    return C::BM == 128 && TAPS != 9 ? 2 : 1;
}
// Stages per turn of the loop: every ring is back where it was.
constexpr int b3_turn(int q, int r, int d, int bb) {
    int u = 1;
    while (u * q % r || u % d || u * q % bb) ++u;
    return u;
}
// staging units (16 channels x 32 slots) per wave and stage of 1x1 filters and dense layers
template <class C, bool DENSE>
constexpr int b3_units1() { return C::WK * b3_cw<C, 1, DENSE>() * C::TN * C::WN / C::NW; }

// Division by multiply-high, n / d for d >= 2: m = floor(2^32 / d) + 1, one = 0; d = 1: m = 0, one = ~0.  Exact for numerators
// up to `most` if most * d < 2^32, which b3_set_div checks.
inline bool b3_set_div(B3Div *m, int64_t d, int64_t most) {
    if (d < 1 || most * d >= ((int64_t)1 << 32)) return false;
    m->m = d == 1 ? 0u : (uint32_t)((((uint64_t)1 << 32) / (uint64_t)d) + 1);
    m->one = d == 1 ? ~0u : 0u;
    return true;
}
__device__ __forceinline__ uint32_t b3_div(uint32_t n, const B3Div &d) { return __umulhi(n, d.m) + (n & d.one); }

// One pair of values -> a 32-bit word of each plane.
__device__ __forceinline__ void b3_split2(float a, float b, uint32_t &h, uint32_t &m, uint32_t &l) {
    h = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2v{a, b}, bf16x2));
    a -= __uint_as_float(h << 16);
    b -= __uint_as_float(h & 0xffff0000u);
    m = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2v{a, b}, bf16x2));
    a -= __uint_as_float(m << 16);
    b -= __uint_as_float(m & 0xffff0000u);
    l = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2v{a, b}, bf16x2));
}

// One plane of a pair: the word of it, and what it leaves out in place of the pair.
__device__ __forceinline__ void b3_take(float &a, float &b, uint32_t &w) {
    w = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2v{a, b}, bf16x2));
    a -= __uint_as_float(w << 16);
    b -= __uint_as_float(w & 0xffff0000u);
}
// The staging split in pieces that a wave puts between its products: a plane of a pair each, and the four pairs of a unit take turns
// (the steps of one pair depend on each other).  The ninth is the last plane of all four.
constexpr int kB3Pieces = 9;

// One pair of constant operands, which are split once, into all planes: a finite value that would round to an infinity has the largest finite
// bf16 as its leading plane (what is left then has 16 bits, as elsewhere).
__device__ __forceinline__ void b3_split2_full(float a, float b, uint32_t &h, uint32_t &m, uint32_t &l) {
    constexpr float most = 0x1.fep127f;
    const float ah = __builtin_isfinite(a) ? fminf(fmaxf(a, -most), most) : a, bh = __builtin_isfinite(b) ? fminf(fmaxf(b, -most), most) : b;
    h = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2v{ah, bh}, bf16x2));
    a -= __uint_as_float(h << 16);
    b -= __uint_as_float(h & 0xffff0000u);
    m = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2v{a, b}, bf16x2));
    a -= __uint_as_float(m << 16);
    b -= __uint_as_float(m & 0xffff0000u);
    l = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2v{a, b}, bf16x2));
}

// A weight from its planes: eight values per lane entry, planes kWave entries apart.
__device__ __forceinline__ float b3_weight(const u32x4 *entry, int e) {
    const uint16_t *q = reinterpret_cast<const uint16_t *>(entry) + e;
    const float h = __uint_as_float((uint32_t)q[0] << 16), m = __uint_as_float((uint32_t)q[8 * kWave] << 16), l = __uint_as_float((uint32_t)q[16 * kWave] << 16);
    return __builtin_isfinite(h) ? h + m + l : h;
}

// Bit n: out[n] is computed again, because it is not finite or so small, without being zero, that operands below 2^-110 may
// have made it (2^-90: such an operand is off by less than 2^-126, so 4096 of them against weights of one are off by
// less than 2^-24 of a larger sum).  One and a half instructions per value where no value of the wave is (zeros are sorted out behind the branch).
template <int N>
__device__ __forceinline__ uint32_t b3_doubtful(const float (&out)[N]) {
    static_assert(N <= 32, "a bit per value");
    constexpr uint32_t low = (uint32_t)(127 - 90) << 24, inf = 0xffu << 24;            // (magnitudes: the bits without the sign, shifted up)
    uint32_t most = 0;
#pragma unroll
    for (int n = 0; n < N; ++n) most = max(most, (__float_as_uint(out[n]) << 1) - low);
    uint32_t bad = 0;
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(most >= inf - low) != 0, 0)) {
#pragma unroll
        for (int n = 0; n < N; ++n) {
            const uint32_t v = __float_as_uint(out[n]) << 1;
            bad |= v - 1 < low - 1 || v >= inf ? 1u << n : 0u;
        }
    }
    return bad;
}

// (the same mapping as the other tiled kernels': an XCD gets a contiguous range of tiles)
__device__ __forceinline__ int b3_xcd_remap(int id, int n) {
    const int q = n / 8, r = n % 8;
    const int xcd = id % 8, idx = id / 8;
    return xcd * q + (xcd < r ? xcd : r) + idx;
}

// f(0), f(1), ..., f(N - 1) with the index as a compile-time constant
template <class F, int... I>
__device__ __forceinline__ void b3_each(F &&f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, class F>
__device__ __forceinline__ void b3_for(F &&f) { b3_each(f, std::make_integer_sequence<int, N>{}); }

// Loads through a buffer descriptor: a lane whose offset is kOut (beyond the buffer) gets zero.
constexpr uint32_t kB3Out = 0x80000000u;

template <class C, int TAPS, bool DEPTH, bool DENSE, int UM>
__device__ __forceinline__ void b3_body(const B3Args &p) {
    constexpr int CW = b3_cw<C, TAPS, DENSE>(), SC = C::WK * CW, Q = CW * TAPS;
    constexpr int R = b3_ring<C, TAPS>(), D = b3_deep<C, TAPS, DENSE>(), BB = b3_ahead<C, TAPS>(), U = b3_turn(Q, R, D, BB);
    constexpr int TN = C::TN, WK = C::WK;
    constexpr bool PRIV = C::PRIV, DIRECT = b3_direct<C, TAPS, DENSE>();
    static_assert(DIRECT || BB == 1 || Q > 1, "staging ends a step before the stage does");
    extern __shared__ u32x4 b3_lds[];
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1), half = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int wk = wave % WK, wn = (wave / WK) % C::WN, wm = wave / (WK * C::WN);

    // tile -> (row group, column tile); the faster one is what neighbouring workgroups do not share
    const int tile = b3_xcd_remap(blockIdx.x, gridDim.x);
    const int t_hi = (int)b3_div((uint32_t)tile, p.d_tile), t_lo = tile - t_hi * p.tile_div;
    const int mg = p.jmajor ? t_lo : t_hi, nt = p.jmajor ? t_hi : t_lo;
    const int mt = min(mg * C::WM + wm, p.mtiles - 1);                     // packed row tile (all phases)
    const bool m_live = mg * C::WM + wm < p.mtiles;
    const int phase = p.phases > 1 ? mt / p.tiles_m : 0;
    const int i0 = (mt - phase * p.tiles_m) * 32;
    const int ph_a = p.phases > 1 ? phase / p.sw : 0, ph_b = p.phases > 1 ? phase - ph_a * p.sw : 0;
    const int ks = blockIdx.z;
    const int st_begin = ks * p.stages_per, st_end = min(p.stages, st_begin + p.stages_per);

    const int strip = DENSE ? 0 : (int)b3_div((uint32_t)nt, p.d_strip);
    const int j0 = (DENSE ? nt : nt - strip * p.tiles_strip) * C::BN;
    // slots per 8-channel row of a plane (16-byte units), and one plane
    const int S = TAPS == 1 ? (DENSE ? C::BN + 2 : C::BN) : p.slot_stride;
    const int PL = 2 * SC * S;
    int v0 = 0;
    if constexpr (!DENSE) {
        const uint32_t g = b3_div((uint32_t)j0, p.d_tw), im = b3_div(g, p.d_ho);
        v0 = (int)im * p.rpi + ((int)g - (int)im * p.HO) * p.ly;
    }

    // ---- weights: this wave's stream, three planes of 64 lanes x 16 bytes per step, through a buffer descriptor that ends where the stream does: what a
    // ring reads ahead of the last step is zero and costs no traffic (with four steps per wave it would be a good part of it).  As loads from a
    // scalar pointer the same kernels took 1024 -> 512 at 14x14, batch 32, 50.8 instead of 43.0 us, dense 768 -> 3072 on 389 rows 20.6 instead of 19.8.
    constexpr int STEP = 3 * kWave * 16;
    const int64_t w_first = (((int64_t)mt * WK + wk) * p.stages + st_begin) * (Q * STEP);
    const auto wsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(reinterpret_cast<const char *>(p.w)) + w_first, (short)0,
                                                        (st_end - st_begin) * (Q * STEP), 0x00020000);
    uint32_t wo = (uint32_t)lane * 16;
    u32x4 ar[R][3];
    auto load_w = [&](int set) {
#pragma unroll
        for (int k = 0; k < 3; ++k) ar[set][k] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(wsrc, (int)wo, k * (kWave * 16), 0));
        wo += STEP;
    };
#pragma unroll
    for (int r = 0; r + 1 < R; ++r) load_w(r);

    // ---- staging units of this wave: (16-channel block of the stage, 32 slots); a lane takes eight channels (its half).
    // A wave short of units repeats the last one (the same values to the same place); PRIV: the units of the wave's own blocks.
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p.x), (short)0, p.x_bytes, 0x00020000);
    uint32_t off[UM];                                                      // byte offset, or kB3Out: the slot is padding
    int ldsw[UM], c16l[UM];
    int idu[DEPTH ? UM : 1];
#pragma unroll
    for (int u = 0; u < UM; ++u) {
        const int unit = TAPS == 1 ? wave + u * C::NW : min(wave + u * C::NW, p.units - 1);
        if constexpr (DENSE) {
            // 16 rows x 32 values of k: four lanes per row read 128 contiguous bytes
            const int c32 = PRIV ? wk * (CW / 2) + u / (C::BN / 16) : unit / (C::BN / 16), grp = (PRIV ? u : unit) % (C::BN / 16);
            const int row = grp * 16 + (lane >> 2), part = lane & 3;
            c16l[u] = c32 * 32 + part * 8;                                 // first k of the lane within the stage
            off[u] = (uint32_t)min(j0 + row, p.Nrows - 1) * (uint32_t)p.ldx;
            ldsw[u] = (c32 * 4 + part) * S + row;
        } else {
            const int c16 = PRIV ? wk * CW : (TAPS == 1 ? unit / (C::BN / 32) : (int)b3_div((uint32_t)unit, p.d_g32));
            const int grp = PRIV ? (TAPS == 1 ? u : min(u, p.g32 - 1)) : (TAPS == 1 ? unit % (C::BN / 32) : unit - c16 * p.g32);
            const int slot = grp * 32 + l32;
            int im, ih, iw;
            bool in;
            if constexpr (TAPS == 1) {                                     // a slot is an output pixel
                const uint32_t g = b3_div((uint32_t)(j0 + slot), p.d_tw);
                im = (int)b3_div(g, p.d_ho);
                ih = ((int)g - im * p.HO) * p.ys;
                iw = (strip * p.TW + j0 + slot - (int)g * p.TW) * p.xs;
                in = im < p.Nimg && iw < p.W;
            } else {
                const int r = (int)b3_div((uint32_t)slot, p.d_pw), x = slot - r * p.pw_slots;
                const int v = v0 + r;
                im = (int)b3_div((uint32_t)v, p.d_rpi);
                ih = (v - im * p.rpi) * p.ys - p.ph;
                iw = (strip * p.TW * p.lx + x) * p.xs - p.pwd;
                in = im < p.Nimg && ih >= 0 && ih < p.H && iw >= 0 && iw < p.W;
            }
            int n = im, od = 0;
            if (p.DO > 1) {
                n = (int)b3_div((uint32_t)im, p.d_do);
                od = im - n * p.DO;
            }
            const int id0 = od * p.sd - p.pd;
            const int32_t o = (n * p.img_stride + id0 * p.HW + ih * p.W + iw) * 4;
            off[u] = in ? (uint32_t)(o + half * 32 * p.cs) : kB3Out;
            if constexpr (DEPTH) idu[u] = id0;
            c16l[u] = c16;
            ldsw[u] = (c16 * 2 + half) * S + slot;
        }
    }
    const int cbase = (!DENSE && p.groups > 1) ? (int)b3_div((uint32_t)i0, p.d_cpgo) * p.cpg_in : 0;

    // blocks (and depth taps) in which this lane's eight channels exist; the others are zero, as their weights are
    // (nor is anything read of a stage behind this workgroup's last one)
    const int blk_end = DENSE ? 0 : min(((p.Cf - half * 8 + 15) >> 4) * (DEPTH ? p.KD : 1), st_end * SC);
    const int k_end = DENSE ? min(p.K, st_end * SC * 16) : 0;
    float xs[D][UM][8];
    auto load = [&](int set, int u, int st) {
        float (&xv)[UM][8] = xs[set];
        if constexpr (DENSE) {
            const int k = st * SC * 16 + c16l[u];
            const uint32_t o = k < k_end ? (off[u] + (uint32_t)k) * 4 : kB3Out;
            const u32x4 a = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)o, 0, 0));
            const u32x4 b = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)o, 16, 0));
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                xv[u][i] = __uint_as_float(a[i]);
                xv[u][4 + i] = __uint_as_float(b[i]);
            }
        } else if constexpr (DEPTH) {
            // block: (16 channels, depth tap); a plane before or behind the volume is zero
            const int blk = min(st * SC + c16l[u], p.nC - 1), c16 = (int)b3_div((uint32_t)blk, p.d_kd), kd = blk - c16 * p.KD;
            // (the offset is masked, not selected, so that the scalar work in front of it stays out of a branch.  A slot of padding stays beyond the
            // buffer; off may lie in front of the volume, the sum is in it where the plane is)
            const uint32_t so = (uint32_t)(c16 * 16 * p.cs + kd * p.HW) * 4;
            const bool in = st * SC + c16l[u] < blk_end && (uint32_t)(idu[u] + kd) < (uint32_t)p.D;
            const uint32_t o = (off[u] + so) | (in ? 0u : kB3Out);
#pragma unroll
            for (int i = 0; i < 8; ++i)
                xv[u][i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)o, i * p.cs * 4, 0));
        } else {
            const int c = cbase + min(st * SC + c16l[u], p.nC - 1) * 16;
            const uint32_t so = (uint32_t)(c * p.cs) * 4;                  // (kB3Out + so is outside as well: the buffer has less than 2 GB)
            const uint32_t o = (off[u] + so) | (st * SC + c16l[u] < blk_end ? 0u : kB3Out);
#pragma unroll
            for (int i = 0; i < 8; ++i)
                xv[u][i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)o, i * p.cs * 4, 0));
        }
    };
    bf16x8 b[BB][TN][3];
    uint32_t pl_w[3][4];
    // piece i of the staging work of unit u, input set `set`; the last one writes the unit to LDS buffer `buf` (DIRECT: it is the fragment
    // of column tile u in fragment set `buf`) and loads its next values
    auto piece = [&](int set, int u, int i, int buf, int st_next) {
        float (&xv)[8] = xs[set][u];
        if (i < 8) {
            b3_take(xv[2 * (i & 3)], xv[2 * (i & 3) + 1], pl_w[i >> 2][i & 3]);
        } else {
#pragma unroll
            for (int n = 0; n < 4; ++n) pl_w[2][n] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2v{xv[2 * n], xv[2 * n + 1]}, bf16x2));
            u32x4 pl[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) pl[k] = u32x4{pl_w[k][0], pl_w[k][1], pl_w[k][2], pl_w[k][3]};
            if constexpr (DIRECT) {
#pragma unroll
                for (int k = 0; k < 3; ++k) b[buf][u][k] = __builtin_bit_cast(bf16x8, pl[k]);
            } else {
                u32x4 *dst = b3_lds + buf * 3 * PL + ldsw[u];
#pragma unroll
                for (int k = 0; k < 3; ++k) dst[k * PL] = pl[k];
            }
            load(set, u, st_next);
        }
    };
#pragma unroll
    for (int d = 0; d < D; ++d)
#pragma unroll
        for (int u = 0; u < UM; ++u) load(d, u, st_begin + d);

    // ---- this lane's column of every tile: first slot
    int sbase[TN];
#pragma unroll
    for (int t = 0; t < TN; ++t) {
        const int jl = (wn * TN + t) * 32 + l32;
        if constexpr (TAPS == 1) {
            sbase[t] = jl + half * S;
        } else {
            const uint32_t jj = (uint32_t)min(j0 + jl, p.Ntot - 1);
            const uint32_t g = b3_div(jj, p.d_tw), im = b3_div(g, p.d_ho);
            const int oh = (int)g - (int)im * p.HO;
            sbase[t] = ((int)im * p.rpi + oh * p.ly - v0) * p.pw_slots + ((int)jj - (int)g * p.TW) * p.lx + half * S;
        }
        sbase[t] += wk * CW * 2 * S;
        if (TAPS == 4) {                                                   // where the phase's taps start in the common patch
            const int dh = p.phe_max - (p.KHe - 1 - (ph_a + p.ph_t) / p.sh), dw = p.pwe_max - (p.KWe - 1 - (ph_b + p.pw_t) / p.sw);
            sbase[t] += dh * p.pw_slots + dw;
        }
    }
#pragma unroll
    for (int n = 0; n < kB3Pieces * UM; ++n) piece(0, n / kB3Pieces, n % kB3Pieces, 0, st_begin + D);

    // Two accumulators per tile: the products of the leading planes, and the five small ones (2^-8 of them and
    // less).  The large sum is then rounded once per 16 values of k.
    f32x16v acc[TN], acs[TN];
#pragma unroll
    for (int t = 0; t < TN; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][r] = acs[t][r] = 0.f;

    constexpr int KWt = TAPS == 9 ? 3 : (TAPS == 4 ? 2 : 1);
    auto read_b = [&](int set, int q, int buf) {
        const int tap = q % TAPS;
        const int kh = tap / KWt, kw = tap % KWt;
        const int so = buf * 3 * PL + (q / TAPS) * 2 * S + (TAPS == 1 ? 0 : kh * p.pw_slots + kw);
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int k = 0; k < 3; ++k) b[set][t][k] = reinterpret_cast<const bf16x8 *>(b3_lds)[k * PL + so + sbase[t]];
    };
    if constexpr (!PRIV) lds_barrier();
    if constexpr (!DIRECT && BB > 1) read_b(0, 0, 0);
    for (int st0 = st_begin; st0 < st_end; st0 += U) {                     // (a turn may end behind the last stage: weights and inputs are zero there)
        b3_for<U>([&](auto uc) {
            constexpr int u = uc.value;
            const int st = st0 + u, buf = (st - st_begin) & 1;
            b3_for<Q>([&](auto qc) {
                constexpr int q = qc.value, g = u * Q + q, cur = g % BB, nxt = (g + 1) % BB;
                // Input fragments, and a later step's weights, leave before this step's products.  With a second set of fragments the next step's
                // leave now, the next stage's first ones behind the barrier that ends its staging, one step before this stage
                // ends.  That set pays where its registers cost no resident wave: 128x128 tiles (1024 -> 512 at 14x14, batch 32, 47 -> 44 us) and the PRIV ones;
                // not on 64-row tiles, which lose the third wave of a SIMD (64 -> 256 at 56x56, batch 32, 44 -> 53 us).
                if constexpr (!DIRECT) {
                    if constexpr (BB == 1) {
                        read_b(0, q, buf);
                    } else if constexpr (q + 1 < Q) {
                        read_b(nxt, q + 1, buf);
                    } else {
                        if constexpr (!PRIV) lds_barrier();
                        read_b(nxt, 0, buf ^ 1);
                    }
                }
                load_w((g + R - 1) % R);
                __builtin_amdgcn_sched_barrier(0);
                bf16x8 a[3];
#pragma unroll
                for (int k = 0; k < 3; ++k) a[k] = __builtin_bit_cast(bf16x8, ar[g % R][k]);
                b3_for<6 * TN>([&](auto mc) {
                    constexpr int m = mc.value / TN, t = mc.value % TN;
                    constexpr int PA[6] = {0, 2, 0, 1, 1, 0}, PB[6] = {0, 0, 2, 1, 0, 1};
                    if constexpr (m == 0) acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[PA[m]], b[cur][t][PB[m]], acc[t], 0, 0, 0);
                    else acs[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[PA[m]], b[cur][t][PB[m]], acs[t], 0, 0, 0);
                    // staging work for the next stage, spread over the products of this one (BB = 2: of all steps but the last)
                    constexpr int SLOTS = 6 * TN * (BB > 1 && !DIRECT ? Q - 1 : Q), PIECES = kB3Pieces * UM, slot = q * 6 * TN + mc.value;
                    if constexpr (slot < SLOTS) {
                        constexpr int n0 = slot * PIECES / SLOTS, n1 = (slot + 1) * PIECES / SLOTS;
                        b3_for<n1 - n0>([&](auto nc) {
                            constexpr int n = n0 + nc.value;
                            piece((u + 1) % D, n / kB3Pieces, n % kB3Pieces, DIRECT ? nxt : buf ^ 1, st + 1 + D);
                        });
                    }
                    __builtin_amdgcn_sched_barrier(0);
                });
            });
            if constexpr (!PRIV && BB == 1) lds_barrier();
        });
    }

    // ---- K-waves meet in LDS; every wave finishes its share of the tile's accumulator registers
    constexpr int NR = TN * 16 / WK;                                       // values per lane to finish
    float out[NR];
    if constexpr (WK > 1) {
        float *red = reinterpret_cast<float *>(b3_lds);
        constexpr int PER = TN * 16 * kWave;
        if constexpr (PRIV ? !DIRECT : BB > 1) __syncthreads();        // (some wave's fragments may still be on their way out of the same LDS)
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) red[wave * PER + (t * 16 + r) * kWave + lane] = acc[t][r] + acs[t][r];
        __syncthreads();
        const int w0 = wave - wk;
#pragma unroll
        for (int n = 0; n < NR; ++n) {
            float v = 0.f;
#pragma unroll
            for (int w = 0; w < WK; ++w) v += red[(w0 + w) * PER + (wk * NR + n) * kWave + lane];
            out[n] = v;
        }
    } else {
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) out[t * 16 + r] = acc[t][r] + acs[t][r];
    }
    // Every operand of the fused tail is loaded before the first result is stored, and stores go through a buffer
    // descriptor: what lies outside the output gets an offset that is dropped, so there is no branch per value.
    constexpr int ND = NR >= 16 ? NR / 16 : 1, NE = NR >= 16 ? 16 : NR;    // column tiles, registers of each
    static_assert(NE % 4 == 0, "a lane finishes groups of four rows");
    const int r0 = NR >= 16 ? 0 : (wk * NR) % 16;                          // (tile row of register r: 8 (r / 4) + 4 half + r % 4)
    const bool tail = p.splitk == 1;
    const int flags = tail ? p.ef.flags : 0;
    const auto ydst = __builtin_amdgcn_make_buffer_rsrc(tail ? p.y : p.partial + (int64_t)ks * p.c_numel, (short)0, (int)(p.c_numel * 4), 0x00020000);
    const auto rsum = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p.ef.add), (short)0, (int)(p.c_numel * 4), 0x00020000);
    const auto rbias = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p.ef.bias), (short)0, p.Cout * 4, 0x00020000);
    uint32_t ob[ND];
#pragma unroll
    for (int d = 0; d < ND; ++d) {
        const int t = wk * NR / 16 + d;
        const int j = j0 + (wn * TN + t) * 32 + l32;
        if constexpr (DENSE) {
            ob[d] = m_live && j < p.Nrows ? (uint32_t)(j * p.ldy + 4 * half) * 4 : kB3Out;
        } else {
            const uint32_t g = b3_div((uint32_t)j, p.d_tw), im = b3_div(g, p.d_ho);
            const int oh = (int)g - (int)im * p.HO, ow = strip * p.TW + j - (int)g * p.TW;
            int n = (int)im, od = 0;
            if (p.DO > 1) {
                n = (int)b3_div(im, p.d_do);
                od = (int)im - n * p.DO;
            }
            const uint32_t o = (uint32_t)(n * p.ons + od * p.npix + (oh * p.os + ph_a) * p.WO + ow * p.os + ph_b + 4 * half * p.ocs) * 4;
            ob[d] = m_live && j < p.Ntot && ow < p.WOe ? o : kB3Out;
        }
    }
    const int left = p.Cout - i0 - 4 * half;                               // rows of the tile this lane half may store, from its first one
    const uint32_t bad = b3_doubtful<NR>(out);
    float bv[NR], av[NR];
#pragma unroll
    for (int n = 0; n < NR; ++n) bv[n] = av[n] = 0.f;
    if (flags & EF_BIAS) {
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            const float v = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rbias, (i0 + 4 * half) * 4, (8 * ((r0 + e) / 4) + (r0 + e) % 4) * 4, 0));
#pragma unroll
            for (int d = 0; d < ND; ++d) bv[d * NE + e] = v;
        }
    }
    const int cbase_y = DENSE ? (p.cs_len ? (i0 / p.cs_len) * (int)p.cs_stride + i0 % p.cs_len : i0) : 0;
    // Doubtful results once more: the fp32 chain over this workgroup's part of K, its tail and its store (behind the first one)
    auto again = [&] {
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(bad != 0) == 0, 1)) return;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll 1
        for (int n = 0; n < NR; ++n) {
            const int d = n / NE, e = n % NE, rr = 8 * ((r0 + e) / 4) + (r0 + e) % 4, i = i0 + 4 * half + rr;
            const int j = j0 + (wn * TN + wk * NR / 16 + d) * 32 + l32;
            if (!(bad >> n & 1) || !m_live || rr >= left || j >= (DENSE ? p.Nrows : p.Ntot)) continue;
            float v = 0.f;
            const u32x4 *row = reinterpret_cast<const u32x4 *>(p.w) + (int64_t)mt * WK * p.stages * (Q * 3 * kWave) + (4 * half + rr);
            // entry of block b (of 16 values of k) and tap q; half 0 holds the block's first eight
            auto entry = [&](int b, int q) {
                const int st = b / SC, r = b - st * SC, w = r / CW;
                return row + (((int64_t)w * p.stages + st) * Q + (r - w * CW) * TAPS + q) * (3 * kWave);
            };
            const int b_end = min(st_end * SC, p.nC);
            uint32_t o;
            if constexpr (DENSE) {
                const float *x = p.x + (int64_t)j * p.ldx;
                for (int k = st_begin * SC * 16; k < min(b_end * 16, p.K) && v == v; ++k)
                    v = fmaf(x[k], b3_weight(entry(k / 16, 0) + k / 8 % 2 * 32, k % 8), v);
                o = (uint32_t)(j * p.ldy + 4 * half + cbase_y + rr);
            } else {
                const uint32_t g = b3_div((uint32_t)j, p.d_tw), im = b3_div(g, p.d_ho);
                const int oh = (int)g - (int)im * p.HO, ow = strip * p.TW + j - (int)g * p.TW;
                if (ow >= p.WOe) continue;
                const int nn = p.DO > 1 ? (int)b3_div(im, p.d_do) : (int)im, od = (int)im - nn * p.DO;
                int dh = 0, dw = 0;
                if (TAPS == 4) {
                    dh = p.phe_max - (p.KHe - 1 - (ph_a + p.ph_t) / p.sh);
                    dw = p.pwe_max - (p.KWe - 1 - (ph_b + p.pw_t) / p.sw);
                }
                for (int b = st_begin * SC; b < b_end; ++b) {
                    const int c16 = DEPTH ? b / p.KD : b, id = od * p.sd - p.pd + (DEPTH ? b - c16 * p.KD : 0);
                    for (int c = 0; c < 16 && c16 * 16 + c < p.Cf && v == v; ++c) {
                        const int ch = cbase + c16 * 16 + c;
                        if (p.groups > 1 && ch / p.cpg_in != i / p.cpg_out) continue;      // (a block of rows spans several narrow groups)
                        for (int q = 0; q < TAPS; ++q) {
                            const int ih = (oh * p.ly + dh + q / KWt) * p.ys - p.ph, iw = (ow * p.lx + dw + q % KWt) * p.xs - p.pwd;
                            const bool in = id >= 0 && id < p.D && ih >= 0 && ih < p.H && iw >= 0 && iw < p.W;
                            const float x = in ? p.x[(int64_t)nn * p.img_stride + (int64_t)ch * p.cs + id * p.HW + ih * p.W + iw] : 0.f;
                            v = fmaf(x, b3_weight(entry(b, q) + c / 8 * 32, c % 8), v);
                        }
                    }
                }
                o = (uint32_t)(nn * p.ons + od * p.npix + (oh * p.os + ph_a) * p.WO + ow * p.os + ph_b + i * p.ocs);
            }
            float val[1] = {v}, b1[1] = {flags & EF_BIAS ? p.ef.bias[i] : 0.f}, a1[1] = {flags & EF_ADD ? p.ef.add[o] : 0.f};
            fused_tail<1>(EpiFast{flags, p.ef.scale, nullptr, nullptr}, val, b1, a1);
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(val[0]), ydst, (int)(o * 4), 0, 0);
        }
    };
    if constexpr (DENSE) {
        if (p.Cout % 4 == 0) {                                             // four rows of the tile = 16 contiguous bytes
            if (flags & EF_ADD) {
#pragma unroll
                for (int d = 0; d < ND; ++d)
#pragma unroll
                    for (int e = 0; e < NE; e += 4) {
                        const int rr = 8 * ((r0 + e) / 4);
                        const u32x4 v = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsum, (int)(rr < left ? ob[d] : kB3Out), (cbase_y + rr) * 4, 0));
#pragma unroll
                        for (int f = 0; f < 4; ++f) av[d * NE + e + f] = __uint_as_float(v[f]);
                    }
            }
            fused_tail<NR>(EpiFast{flags, p.ef.scale, nullptr, nullptr}, out, bv, av);
#pragma unroll
            for (int d = 0; d < ND; ++d)
#pragma unroll
                for (int e = 0; e < NE; e += 4) {
                    const int rr = 8 * ((r0 + e) / 4);
                    u32x4 v;
#pragma unroll
                    for (int f = 0; f < 4; ++f) v[f] = __float_as_uint(out[d * NE + e + f]);
                    // (the offset all in the lane register: with a scalar offset the four data registers were overwritten by the
                    // next vector instruction while the store still read them - the compiler inserts a wait only without one)
                    __builtin_amdgcn_raw_buffer_store_b128(v, ydst, (int)((rr < left ? ob[d] : kB3Out) + (uint32_t)(cbase_y + rr) * 4u), 0, 0);
                }
            again();
            return;
        }
    }
    const int rstep = DENSE ? 1 : p.ocs;
    if (flags & EF_ADD) {
#pragma unroll
        for (int d = 0; d < ND; ++d)
#pragma unroll
            for (int e = 0; e < NE; ++e) {
                const int rr = 8 * ((r0 + e) / 4) + (r0 + e) % 4;
                av[d * NE + e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsum, (int)(rr < left ? ob[d] : kB3Out),
                                                                                      (DENSE ? cbase_y + rr : (i0 + rr) * rstep) * 4, 0));
            }
    }
    fused_tail<NR>(EpiFast{flags, p.ef.scale, nullptr, nullptr}, out, bv, av);
#pragma unroll
    for (int d = 0; d < ND; ++d)
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            const int rr = 8 * ((r0 + e) / 4) + (r0 + e) % 4;
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(out[d * NE + e]), ydst, (int)(rr < left ? ob[d] : kB3Out),
                                                  (DENSE ? cbase_y + rr : (i0 + rr) * rstep) * 4, 0);
        }
    again();
}

template <class C, int TAPS, bool DEPTH, bool DENSE, int UM>
__global__ __launch_bounds__(C::NT, 2) void b3_kernel(B3Args p) { b3_body<C, TAPS, DEPTH, DENSE, UM>(p); }

// Dense layers of one shape and tail, one per blockIdx.y (a transformer's q, k and v: 84 tiles each at 389 rows, too few alone).
template <class C, int UM>
__global__ __launch_bounds__(C::NT, 2) void b3_dense_multi_kernel(B3Args p, B3Region r) {
    const int k = blockIdx.y;
    p.x = r.x[k];
    p.w = r.w[k];
    p.y = r.y[k];
    p.ef.bias = r.bias[k];
    p.ef.add = r.add[k];
    b3_body<C, 1, false, true, UM>(p);
}

// gemm_b3_first.hip: first layers (few input channels)
bool first_resolve(const GemmArgs &g, B3Args *out);
int launch_b3_first_pack(const B3Args &a, const float *w, void *dst, hipStream_t s);
int launch_b3_first(const B3Args &a, hipStream_t s);

// host: launches one configuration (instantiated per filter class in gemm_b3_point / _nine / _depth / _phase.hip)
template <int TAPS, bool DEPTH, bool DENSE>
int b3_launch_tile(const B3Args &a, hipStream_t s);

template <class C, int TAPS, bool DEPTH, bool DENSE, int UM>
int b3_launch_um(const B3Args &a, hipStream_t s) {
    const int S = TAPS == 1 ? (DENSE ? C::BN + 2 : C::BN) : a.slot_stride;
    const size_t stage = b3_direct<C, TAPS, DENSE>() ? 0 : (size_t)2 * 3 * 2 * C::WK * b3_cw<C, TAPS, DENSE>() * S * 16;
    const size_t lds = stage > (size_t)C::RED ? stage : (size_t)C::RED;
    if constexpr (DENSE && (std::is_same_v<C, B3M> || std::is_same_v<C, B3M8> || std::is_same_v<C, B3M12> || std::is_same_v<C, B3SS>)) {        // the tiles of regions (b3_region_resolve)
        if (a.region) {
            if (lds > 64 * 1024) {
                static LdsLimit limit;
                const hipError_t e = limit.raise((const void *)b3_dense_multi_kernel<C, UM>);
                if (e != hipSuccess) return (int)e;
            }
            hipLaunchKernelGGL((b3_dense_multi_kernel<C, UM>), dim3((unsigned)(a.mgroups * a.ntiles), (unsigned)a.region->n, 1), dim3(C::NT), lds, s, a, *a.region);
            return (int)hipGetLastError();
        }
    }
    if (a.region) return (int)hipErrorInvalidValue;
    if (lds > 64 * 1024) {
        static LdsLimit limit;
        const hipError_t e = limit.raise((const void *)b3_kernel<C, TAPS, DEPTH, DENSE, UM>);
        if (e != hipSuccess) return (int)e;
    }
    hipLaunchKernelGGL((b3_kernel<C, TAPS, DEPTH, DENSE, UM>), dim3((unsigned)(a.mgroups * a.ntiles), 1, (unsigned)a.splitk),
                       dim3(C::NT), lds, s, a);
    return (int)hipGetLastError();
}

template <class C, int TAPS, bool DEPTH, bool DENSE>
int b3_launch_one(const B3Args &a, hipStream_t s) {
    if constexpr (TAPS == 1) {
        return b3_launch_um<C, TAPS, DEPTH, DENSE, b3_units1<C, DENSE>()>(a, s);
    } else {
        const int um = (a.units + C::NW - 1) / C::NW;
        if (um <= 2) return b3_launch_um<C, TAPS, DEPTH, DENSE, 2>(a, s);
        if (um <= 4) return b3_launch_um<C, TAPS, DEPTH, DENSE, 4>(a, s);
        if (um <= 6) return b3_launch_um<C, TAPS, DEPTH, DENSE, 6>(a, s);
        return (int)hipErrorInvalidValue;
    }
}

#define CLG_B3_INSTANTIATE(TAPS, DEPTH, DENSE)                                             \
    template <>                                                                           \
    int b3_launch_tile<TAPS, DEPTH, DENSE>(const B3Args &a, hipStream_t s) {               \
        switch (a.tile) {                                                                 \
        case B3_L: return b3_launch_one<B3L, TAPS, DEPTH, DENSE>(a, s);                    \
        case B3_LM: return b3_launch_one<B3LM, TAPS, DEPTH, DENSE>(a, s);                  \
        case B3_M: return b3_launch_one<B3M, TAPS, DEPTH, DENSE>(a, s);                    \
        case B3_M8:                                                                       \
            if constexpr (!DEPTH) return b3_launch_one<B3M8, TAPS, DEPTH, DENSE>(a, s);    \
            else return (int)hipErrorInvalidValue;                                        \
        case B3_M12:                                                                      \
            if constexpr (DENSE) return b3_launch_one<B3M12, TAPS, DEPTH, DENSE>(a, s);    \
            else return (int)hipErrorInvalidValue;                                        \
        case B3_S: return b3_launch_one<B3S, TAPS, DEPTH, DENSE>(a, s);                    \
        case B3_SS: return b3_launch_one<B3SS, TAPS, DEPTH, DENSE>(a, s);                  \
        case B3_G: return b3_launch_one<B3G, TAPS, DEPTH, DENSE>(a, s);                    \
        case B3_G2: return b3_launch_one<B3G2, TAPS, DEPTH, DENSE>(a, s);                  \
        default: return (int)hipErrorInvalidValue;                                        \
        }                                                                                 \
    }

}  // namespace clg
