// Kernels of several kinds as one launch: the branches of a cell (NasNet-A, paper Sec. 5.1) at one distance from its inputs are depthwise and
// separable convolutions of several filter sizes, window pools and 1x1 convolutions, each a few microseconds of which most are the launch.
// Workgroup -> problem by a wave-uniform look-up, a switch on the problem's kind, then the code that the problem runs alone.  A workgroup has
// eight waves, which a problem of fewer waves per tile shares out: eight tiles of a 1x1 convolution whose channels are one chunk of
// MFMAs, two of a separable convolution of four waves.  (With four waves, and problems of eight left out, a NasNet-A cell at 28x28 was
// six launches instead of four.)
// Bound by the launch and one or two memory round trips: such a launch takes 4 - 7 us alone or with seven others.  NasNet-A at batch 1: 141 launches
// with regions of one kind, 100 - 106 with these, 611 -> 527 us; batch 4, 231x231, 987 -> 923; batch 2, 101x101, 630 -> 522.  Reading a word of every
// line of the argument block ahead of the look-up gave nothing (515, 516 us).
#include <algorithm>

#include "gemm_rf.h"
#include "lds_limit.h"
#include "plane.h"
#include "sepconv.h"

namespace clg {

namespace {

constexpr int kMixWaves = 8;

// `local`: the workgroup's number within its problem
template <int TAPK, int WGK, int GEO>
__device__ __forceinline__ void mix_conv(const GemmCore &p, const int local, float *lds) {
    constexpr int PER = kMixWaves / WGK, NT = WGK * kWave;               // tiles per workgroup, threads per tile
    const int tiles = ((p.Cout + 15) / 16) * ((p.HO * p.WO + 15) / 16), wgs = (tiles + PER - 1) / PER;
    const int img = local / wgs, wg = xcd_remap(local - img * wgs, wgs);
    const int part = __builtin_amdgcn_readfirstlane((int)threadIdx.x / NT), tile = wg * PER + part;
    conv_rf_body<16, TAPK, WGK, GEO, TAPK == 1 ? 2 : 1>(p, min(tile, tiles - 1), img, 0, threadIdx.x % NT, lds + part * (WGK * RfMfma<16>::NACC * kWave), tile < tiles);
}

template <int KS, int NW>
__device__ __forceinline__ void mix_sep(const SepConvArgs &a, const int local, float *lds) {
    constexpr int PER = kMixWaves / NW, NT = NW * kWave;
    const int wgs = (a.n_tiles + PER - 1) / PER, by = local / wgs;
    const int part = __builtin_amdgcn_readfirstlane((int)threadIdx.x / NT);
    const int floats = a.ngroups * kGroup * kPix + NW * 256 + (KS > 0 ? a.C * KS * KS : 0);
    sepconv_body<KS, NW>(a, (local - by * wgs) * PER + part, by, threadIdx.x % NT, lds + part * floats);
}

// WIDE: with the kinds of more than 128 registers (7x7 depthwise convolutions, separable ones of 5x5 and 7x7); a launch without them has
// four resident waves per SIMD instead of two.  All of NasNet-A under one placement, every region in one launch, us: 4 x 231x231 971 with the wide kernel for
// all regions and 921 with this rule; 1 x 224x224 534 and 534, 2 x 101x101 530 and 528, where launches hardly fill a round.  Wide kinds stay members all the same
// (out of such regions 589, 541 and 905, 13 - 5 launches more; where the members of a large one lose by it, the search turns their digits off).
constexpr bool mix_wide(int32_t kind) {
    return kind == MIX_DW7 || kind == MIX_SEP4 + 5 || kind == MIX_SEP4 + 7 || kind == MIX_SEP8 + 5 || kind == MIX_SEP8 + 7;
}

template <bool WIDE>
__global__ __launch_bounds__(kMixWaves *kWave, WIDE ? 2 : 4) void mix_kernel(MixArgs m) {
    extern __shared__ float lds[];
    const int bx = blockIdx.x;
    int k = 0;
#pragma unroll
    for (int i = 0; i + 1 < kMaxMixRegion; ++i) k += bx >= m.block_end[i] ? 1 : 0;
    const int local = bx - (k ? m.block_end[k - 1] : 0);
    const uint32_t at = (uint32_t)local * (kMixWaves * kWave) + threadIdx.x;
    const MixMember &p = m.p[k];
    switch (m.kind[k]) {
    case MIX_DW3: depthwise_body<3>(p.dw, at); break;
    case MIX_DW5: depthwise_body<5>(p.dw, at); break;
    case MIX_DW7: if constexpr (WIDE) depthwise_body<7>(p.dw, at); break;
    case MIX_MAX: window_pool_body<false>(p.pool, at); break;
    case MIX_AVG: window_pool_body<true>(p.pool, at); break;
    case MIX_SEP4: mix_sep<0, 4>(p.sep, local, lds); break;
    case MIX_SEP4 + 3: mix_sep<3, 4>(p.sep, local, lds); break;
    case MIX_SEP4 + 5: if constexpr (WIDE) mix_sep<5, 4>(p.sep, local, lds); break;
    case MIX_SEP4 + 7: if constexpr (WIDE) mix_sep<7, 4>(p.sep, local, lds); break;
    case MIX_SEP8: mix_sep<0, 8>(p.sep, local, lds); break;
    case MIX_SEP8 + 3: mix_sep<3, 8>(p.sep, local, lds); break;
    case MIX_SEP8 + 5: if constexpr (WIDE) mix_sep<5, 8>(p.sep, local, lds); break;
    case MIX_SEP8 + 7: if constexpr (WIDE) mix_sep<7, 8>(p.sep, local, lds); break;
    case MIX_CONV + 1: mix_conv<1, 1, 0>(p.conv, local, lds); break;
    case MIX_CONV + 2: mix_conv<1, 2, 0>(p.conv, local, lds); break;
    case MIX_CONV + 4: mix_conv<1, 4, 0>(p.conv, local, lds); break;
    case MIX_CONV + 8: mix_conv<1, 8, 0>(p.conv, local, lds); break;
    case MIX_RCONV + 1: mix_conv<1, 1, 4>(p.conv, local, lds); break;
    case MIX_RCONV + 2: mix_conv<1, 2, 4>(p.conv, local, lds); break;
    case MIX_RCONV + 4: mix_conv<1, 4, 4>(p.conv, local, lds); break;
    case MIX_RCONV + 8: mix_conv<1, 8, 4>(p.conv, local, lds); break;
    case MIX_ANY + 1: mix_conv<0, 1, 0>(p.conv, local, lds); break;
    case MIX_ANY + 2: mix_conv<0, 2, 0>(p.conv, local, lds); break;
    case MIX_ANY + 4: mix_conv<0, 4, 0>(p.conv, local, lds); break;
    default: mix_conv<0, 8, 0>(p.conv, local, lds); break;
    }
}

template <bool WIDE>
int launch_mix(const MixArgs &m, unsigned groups, size_t lds, hipStream_t s) {
    if (lds > 64 * 1024) {
        static LdsLimit limit;
        const hipError_t e = limit.raise((const void *)mix_kernel<WIDE>);
        if (e != hipSuccess) return (int)e;
    }
    hipLaunchKernelGGL(mix_kernel<WIDE>, dim3(groups), dim3(kMixWaves * kWave), lds, s, m);
    return (int)hipGetLastError();
}

int sep_ks(const SepConvArgs &a) { return !a.has_dw ? 0 : a.KH; }

}  // namespace

int32_t mix_conv_kind(const GemmArgs &a) {
    if (a.mode != GM_CONV || a.rf_ts != 16 || a.splitk != 1 || a.D > 1 || a.DO > 1 || a.rf_fold || a.rf_convt || a.rf_d2s || a.KH != 1 || a.KW != 1) return 0;
    if (a.rf_wgk > kMixWaves) return 0;
    if (a.rf_tapk == 1) return (a.rf_prelu ? MIX_RCONV : MIX_CONV) + a.rf_wgk;
    return a.rf_tapk == 0 && !a.rf_prelu ? MIX_ANY + a.rf_wgk : 0;
}

int32_t mix_sep_kind(const SepConvArgs &a) {
    if (a.has_dw && (a.KH != a.KW || (a.KH != 3 && a.KH != 5 && a.KH != 7))) return 0;
    if (kMixWaves / a.nwaves * sepconv_lds_bytes(a) > 160 * 1024) return 0;
    return a.nwaves == 4 ? MIX_SEP4 + sep_ks(a) : (a.nwaves == 8 ? MIX_SEP8 + sep_ks(a) : 0);
}

// Long problems go first: the last workgroup of a few hundred is dispatched a microsecond behind the first.
int32_t mix_weight(int32_t kind) {
    if (kind >= MIX_SEP4 && kind <= MIX_SEP8 + 7) return 100 + kind % 10;
    if (kind >= MIX_CONV) return 50 + kind % 10;
    return kind < MIX_MAX ? 10 + kind : 0;
}

int launch_mix_region(const MixArgs &m_in, void *stream) {
    MixArgs m = m_in;
    if (m.n < 2 || m.n > kMaxMixRegion) return (int)hipErrorInvalidValue;
    int64_t end = 0;
    size_t lds = 0;
    bool wide = false;
    constexpr int threads = kMixWaves * kWave;
    for (int k = 0; k < m.n; ++k) {
        const int32_t kind = m.kind[k];
        wide = wide || mix_wide(kind);
        MixMember &p = m.p[k];
        if (kind == MIX_DW3 || kind == MIX_DW5 || kind == MIX_DW7) {
            if (!depthwise_fast_ok(p.dw) || p.dw.KH != kind) return (int)hipErrorInvalidValue;
            p.dw.ef = make_epi_fast(p.dw.epi);
            end += ((int64_t)p.dw.N * p.dw.C * p.dw.HO * p.dw.WO + threads - 1) / threads;
        } else if (kind == MIX_MAX || kind == MIX_AVG) {
            if (!plane_region_pool_ok(p.pool) || p.pool.mode != (kind == MIX_MAX ? 0 : 2)) return (int)hipErrorInvalidValue;
            end += ((int64_t)p.pool.NC * p.pool.DO * p.pool.HO * p.pool.WO + threads - 1) / threads;
        } else if (kind >= MIX_SEP4 && kind <= MIX_SEP8 + 7) {
            if (mix_sep_kind(p.sep) != kind || (p.sep.has_dw != 0) != (p.sep.wd != nullptr)) return (int)hipErrorInvalidValue;
            p.sep.ef = make_epi_fast(p.sep.epi);
            const int per = kMixWaves / p.sep.nwaves;
            lds = std::max(lds, per * sepconv_lds_bytes(p.sep));
            end += ((int64_t)p.sep.n_tiles + per - 1) / per * ((p.sep.m_tiles + p.sep.mt_per_wg - 1) / p.sep.mt_per_wg);
        } else if (kind >= MIX_CONV && kind <= MIX_ANY + 8) {
            const GemmCore &c = p.conv;
            if (c.rf_ts != 16 || (c.ef.flags & EF_GENERIC) || c.rf_wgk != kind % 10) return (int)hipErrorInvalidValue;
            const int64_t tiles = (int64_t)((c.Cout + 15) / 16) * (((int64_t)c.HO * c.WO + 15) / 16), per = kMixWaves / c.rf_wgk;
            if (c.rf_wgk > 1) lds = std::max(lds, (size_t)kMixWaves * RfMfma<16>::NACC * kWave * sizeof(float));
            end += (tiles + per - 1) / per * c.Nimg;
        } else {
            return (int)hipErrorInvalidValue;
        }
        if (end >= ((int64_t)1 << 31)) return (int)hipErrorInvalidValue;
        m.block_end[k] = (int32_t)end;
    }
    for (int k = m.n; k < kMaxMixRegion; ++k) m.block_end[k] = (int32_t)end;
    if (lds > 160 * 1024) return (int)hipErrorInvalidValue;
    return wide ? launch_mix<true>(m, (unsigned)end, lds, (hipStream_t)stream) : launch_mix<false>(m, (unsigned)end, lds, (hipStream_t)stream);
}

}  // namespace clg
