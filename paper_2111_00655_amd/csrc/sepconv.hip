// Packing, launch shape and dispatch of the one-kernel separable convolution (sepconv.h).
#include <algorithm>

#include <hip/hip_runtime.h>

#include "sepconv.h"

namespace clg {

namespace {

// Packed 1x1 weights: [m-tile][group][lane][4]; value j of lane l in group g of
// m-tile mt is Wp[mt*16 + l%16][(4g + j)*4 + l/16], zero outside the matrix.
__global__ void sepconv_pack_kernel(const float *w, float *dst, int Cout, int C, int ngroups, int64_t total) {
    const int64_t d = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (d >= total) return;
    const int j = (int)(d & 3), lane = (int)((d >> 2) & 63);
    const int64_t gg = d >> 8;
    const int g = (int)(gg % ngroups), mt = (int)(gg / ngroups);
    const int row = mt * kRows + lane % 16, c = (4 * g + j) * 4 + lane / 16;
    dst[d] = (row < Cout && c < C) ? w[(int64_t)row * C + c] : 0.f;
}

template <int KS, int NW>
__global__ __launch_bounds__(NW * 64) void sepconv_kernel(SepConvArgs a) {
    extern __shared__ float lds[];
    sepconv_body<KS, NW>(a, blockIdx.x, blockIdx.y, threadIdx.x, lds);
}

// Several separable convolutions of one kernel shape (filter size, waves per workgroup) in one launch:
// sibling branches of a cell.  Workgroup -> problem by a wave-uniform look-up, then the problem's own
// (pixel tile, channel-tile block) and exactly the code it runs alone.
template <int KS, int NW>
__global__ __launch_bounds__(NW * 64) void sepconv_multi_kernel(SepMultiArgs m) {
    const int bx = blockIdx.x;
    int k = 0;
#pragma unroll
    for (int i = 0; i + 1 < kMaxSepRegion; ++i) k += bx >= m.block_end[i] ? 1 : 0;
    const int local = bx - (k ? m.block_end[k - 1] : 0);
    const int nt = m.p[k].n_tiles;
    const int by = local / nt;
    extern __shared__ float lds[];
    sepconv_body<KS, NW>(m.p[k], local - by * nt, by, threadIdx.x, lds);
}

}  // namespace

// Launch shape for these sizes.  Waves per workgroup: as many as it takes for phase 1 to be about one
// round of loads per thread.  The waves then share phase 2: each takes one 16-row tile of output
// channels, and when there are more waves than tiles (or long channel ranges) several waves split a
// tile's channel range.
static int pow2_ceil(int v) {
    int p = 1;
    while (p < v) p *= 2;
    return p;
}

void sepconv_resolve(SepConvArgs *a) {
    a->ngroups = (a->C + kGroup - 1) / kGroup;
    a->m_tiles = (a->Cout + kRows - 1) / kRows;
    a->n_tiles = (int32_t)(((int64_t)a->N * a->HO * a->WO + kPix - 1) / kPix);
    const int ks = !a->has_dw ? 0 : ((a->KH == a->KW && (a->KH == 3 || a->KH == 5 || a->KH == 7)) ? a->KH : -1);
    a->nwaves = (ks == 5 || ks == 7) ? 8 : 16;                 // those two would not fit 16 waves' register budget
    for (int nw : {8, 4})                                      // the fewest waves that finish phase 1 in one round
        if (a->ngroups * kGroup <= nw * 4 * sep_round_channels(ks, nw)) a->nwaves = nw;
    // waves per tile: so many that a wave's channel groups are all in registers before phase 1
    const int pre = ks == 0 ? 8 : 4;
    const int kparts = std::min(a->nwaves, pow2_ceil((a->ngroups + pre - 1) / pre));
    a->mt_per_wg = std::min(a->nwaves / kparts, pow2_ceil(a->m_tiles));
}

size_t sepconv_pack_bytes(const SepConvArgs &a) {
    return (size_t)a.m_tiles * a.ngroups * 64 * 4 * sizeof(float);
}

size_t sepconv_lds_bytes(const SepConvArgs &a) {
    return ((size_t)a.ngroups * kGroup * kPix + (size_t)a.nwaves * 256 + (a.has_dw ? (size_t)a.C * a.KH * a.KW : 0)) * sizeof(float);
}

int launch_sepconv_pack(const SepConvArgs &a, const float *w, float *dst, void *stream) {
    const int64_t total = (int64_t)a.m_tiles * a.ngroups * 256;
    hipLaunchKernelGGL(sepconv_pack_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                       w, dst, a.Cout, a.C, a.ngroups, total);
    return (int)hipGetLastError();
}

static int sep_ks(const SepConvArgs &a) {
    return !a.has_dw ? 0 : ((a.KH == a.KW && (a.KH == 3 || a.KH == 5 || a.KH == 7)) ? a.KH : -1);
}

int sepconv_region_key(const SepConvArgs &a) { return (sep_ks(a) + 1) * 100 + a.nwaves; }

int launch_sepconv_region(const SepConvArgs *members, int n, void *stream) {
    if (n < 2 || n > kMaxSepRegion) return (int)hipErrorInvalidValue;
    SepMultiArgs m{};
    m.n = n;
    size_t lds = 0;
    int64_t end = 0;
    const int ks = sep_ks(members[0]), nw = members[0].nwaves;
    for (int k = 0; k < n; ++k) {
        SepConvArgs &a = m.p[k];
        a = members[k];
        a.ef = make_epi_fast(a.epi);
        if (sep_ks(a) != ks || a.nwaves != nw || (a.has_dw != 0) != (a.wd != nullptr)) return (int)hipErrorInvalidValue;
        lds = std::max(lds, sepconv_lds_bytes(a));
        end += (int64_t)a.n_tiles * ((a.m_tiles + a.mt_per_wg - 1) / a.mt_per_wg);
        if (end >= ((int64_t)1 << 31)) return (int)hipErrorInvalidValue;
        m.block_end[k] = (int32_t)end;
    }
    for (int k = n; k < kMaxSepRegion; ++k) m.block_end[k] = (int32_t)end;
    if (lds > 160 * 1024) return (int)hipErrorInvalidValue;
    void (*kern)(SepMultiArgs) = nullptr;
#define CLG_SEP_PICK(KS_, NW_) if (ks == KS_ && nw == NW_) kern = sepconv_multi_kernel<KS_, NW_>;
    CLG_SEP_PICK(-1, 4) CLG_SEP_PICK(-1, 8) CLG_SEP_PICK(-1, 16)
    CLG_SEP_PICK(0, 4) CLG_SEP_PICK(0, 8) CLG_SEP_PICK(0, 16)
    CLG_SEP_PICK(3, 4) CLG_SEP_PICK(3, 8) CLG_SEP_PICK(3, 16)
    CLG_SEP_PICK(5, 4) CLG_SEP_PICK(5, 8) CLG_SEP_PICK(7, 4) CLG_SEP_PICK(7, 8)
#undef CLG_SEP_PICK
    if (!kern) return (int)hipErrorInvalidValue;
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return (int)e;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)end), dim3(nw * 64), lds, (hipStream_t)stream, m);
    return (int)hipGetLastError();
}

int launch_sepconv(const SepConvArgs &a_in, void *stream) {
    SepConvArgs a = a_in;
    a.ef = make_epi_fast(a.epi);
    const dim3 grid((unsigned)a.n_tiles, (unsigned)((a.m_tiles + a.mt_per_wg - 1) / a.mt_per_wg));
    const size_t lds = sepconv_lds_bytes(a);
    if (lds > 160 * 1024) return (int)hipErrorInvalidValue;
    const int ks = !a.wd ? 0 : ((a.KH == a.KW && (a.KH == 3 || a.KH == 5 || a.KH == 7)) ? a.KH : -1);
    void (*kern)(SepConvArgs) = nullptr;
#define CLG_SEP_PICK(KS_, NW_) if (ks == KS_ && a.nwaves == NW_) kern = sepconv_kernel<KS_, NW_>;
    CLG_SEP_PICK(-1, 4) CLG_SEP_PICK(-1, 8) CLG_SEP_PICK(-1, 16)
    CLG_SEP_PICK(0, 4) CLG_SEP_PICK(0, 8) CLG_SEP_PICK(0, 16)
    CLG_SEP_PICK(3, 4) CLG_SEP_PICK(3, 8) CLG_SEP_PICK(3, 16)
    CLG_SEP_PICK(5, 4) CLG_SEP_PICK(5, 8) CLG_SEP_PICK(7, 4) CLG_SEP_PICK(7, 8)
#undef CLG_SEP_PICK
    if (!kern || (a.has_dw != 0) != (a.wd != nullptr))
        return (int)hipErrorInvalidValue;
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return (int)e;
    }
    hipLaunchKernelGGL(kern, grid, dim3(a.nwaves * 64), lds, (hipStream_t)stream, a);
    return (int)hipGetLastError();
}

}  // namespace clg
