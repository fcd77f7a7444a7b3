// Scaled-dot-product attention as ONE kernel (gfx950):
//   batch_matmul(q, k^T) -> [mul_scalar] -> softmax -> batch_matmul(p, v) [-> transpose -> reshape]
// i.e. out[h] = softmax(scale * q[h] k[h]^T) v[h] per head h, the heads optionally merged on store
// ([H, S, d] -> [S, H*d]).  Run operator by operator this is three launches plus the score tensor's
// round trip through memory; at batch 1 and sequence 128 (BERT-base, paper Sec. 5.1) each of them
// is a few microseconds of mostly launch.
//
// A workgroup of eight waves owns 16 (32) query rows of one head.  Scores: the block is cut into 16 x 16 tiles
// (v_mfma_f32_16x16x4_f32, contraction over d); q and k are both read 16 bytes per lane along d: lane
// (slot s, row r) takes elements 16g + 4s .. + 3 of its row for the four MFMAs of group g - the order of
// the contraction index does not matter as long as both operands use the same one.  The scaled scores go
// to LDS; the waves share out the rows of the softmax (max, exp, sum); the probabilities stay in
// LDS and are the A operand of the second product (read 16 bytes per lane, the same index order).
// Nothing but q, k, v and the result touches memory.
//
// What bounds it is the L1: some 5 us of matrix work at most, and k and v pass through a compute unit's L1 once per workgroup.  So a wave keeps the
// same keys in both products, loads all its rows of k at once, and those of v, 16 bytes per lane as well (the columns of d are dealt out so that
// a lane's four neighbouring ones belong to four column tiles), between the products of the scores, which wait for k only.  The lanes of an MFMA's
// operand hold 16 bytes of 16 rows each, and a load in that pattern takes the L1 27 ns instead of the 7 of a contiguous one: q (once per
// workgroup) and k are loaded in the order of memory and change lanes through LDS.  Every wave has a partial result of all columns; they meet in LDS.
// Twelve heads of 64, us: 128 keys 4.3, 256 keys 6.1, 389 keys 13.1, 512 keys 14.7; with k loaded as the MFMA wants it, every wave loading the query rows so
// as well, and v before the first product, 5.1, 7.5, 16.1 and 17.9 (of that, 16 bytes instead of 4 per LDS access of the softmax made 0.6 at 389 and 512 keys).
// k passes through LDS in slices of 32 columns, in the place of the partial results: with whole rows in a place of their own a compute unit held one workgroup
// of 128-wide heads instead of two to four.  384 heads, us, k as the MFMA wants it, whole rows and slices: heads of 128, 16 keys 6.0, 8.3 and 6.0, 64 keys 22.4, 30.8 and 22.0, 128 keys 67, 76
// and 65, 256 keys 215, 222 and 180; heads of 64, 64 keys 14.6, 12.4 and 12.5, 200 keys 70, 72 and 63, 300 keys 177, 149 and 118; heads of 32, 512 keys 163, 201 and 161.  Seven keys
// are 0.1 - 0.2 us slower for the barrier that query rows in LDS need.
// A head's tiles on one XCD: no change.  Sixteen waves with two column tiles of v per wave: slower from 128 to 389 keys.
#include <algorithm>
#include <type_traits>

#include <hip/hip_runtime.h>

#include "device_common.h"
#include "kernels.h"
#include "lds_limit.h"

namespace clg {

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

// Value of another lane of the same row of 16 lanes through the data-parallel-primitive path of the
// vector ALU (no LDS round trip as a general shuffle has): CTRL 0xB1 = lane ^ 1, 0x4E = lane ^ 2
// (quad permutations), 0x141 = mirror within 8 lanes, 0x140 = mirror within 16 lanes.  Applied in
// this order with max or + they leave the reduction over the 16 lanes in every one of them.
template <int CTRL>
__device__ __forceinline__ float dpp_peer(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float row16_max(float v) {
    v = fmaxf(v, dpp_peer<0xB1>(v));
    v = fmaxf(v, dpp_peer<0x4E>(v));
    v = fmaxf(v, dpp_peer<0x141>(v));
    return fmaxf(v, dpp_peer<0x140>(v));
}
__device__ __forceinline__ float row16_sum(float v) {
    v += dpp_peer<0xB1>(v);
    v += dpp_peer<0x4E>(v);
    v += dpp_peer<0x141>(v);
    return v + dpp_peer<0x140>(v);
}

constexpr int kRows = 16;          // query rows of a tile
constexpr int kMaxKeys = 512;
constexpr int kWaves = 8;
constexpr int kCUs = 256;          // compute units of an MI355X

// D16 = head size / 16; MAXT = key tiles per wave (kWaves * MAXT tiles cover the keys); RT = row tiles; CS = column
// splits of the second product; SL = columns of k that a wave passes through LDS at a time.
// R: Ahead (workgroups behind the heads read ahead) or NoAhead.
template <int D16, int MAXT, int RT, int CS, int SL, class R>
__global__ __launch_bounds__(kWaves * kWave) void attention_kernel(AttentionArgs a, R ra) {
    constexpr int ROWS = kRows * RT, d = D16 * 16, ldr = d + 4;
    constexpr int KS = kWaves / CS, VT = D16 / CS;           // key splits of the second product, column tiles of a wave
    constexpr int VG = MAXT * CS;                            // key tiles of a wave in it
    constexpr int VEC = VT < 4 ? VT : 4, NV = VT / VEC;      // columns of d per load of v, loads per row
    static_assert(kWaves % CS == 0 && D16 % CS == 0, "the waves share out the column tiles");
    static_assert(CS == 1 || MAXT == 1, "a wave loads v's tile u with the scores of its key tile u");
    constexpr int LPR = kWave * kWaves / ROWS;               // lanes per row of the softmax
    constexpr int PPL = kWaves * MAXT * 4 / LPR;             // 16-byte parts of a row per lane
    static_assert(PPL * LPR == kWaves * MAXT * 4, "a lane takes whole parts");
    typedef float vecv __attribute__((ext_vector_type(VEC)));
    typedef float vecu __attribute__((ext_vector_type(VEC), aligned(4)));      // (v may lie at any address of a float)
    extern __shared__ float lds[];                           // [ROWS][ldp]: scores, then probabilities, behind them lds_q and lds_k; then [KS][ROWS][ldr]: partial results
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, s = lane >> 4;
    const int h = blockIdx.y, q0 = blockIdx.x * ROWS;
    if constexpr (std::is_same_v<R, Ahead>) {
        asm volatile("" ::"s"(a.q), "s"(a.k), "s"(a.v), "s"(a.y), "s"(a.Sq), "s"(a.Sk));      // (loaded with a.B, not behind the branch on it)
        if (h >= a.B)
            return read_ahead(ra, (blockIdx.x + gridDim.x * (h - a.B)) * (kWaves * kWave) + tid, gridDim.x * (gridDim.y - a.B) * (kWaves * kWave));
    }
    const int nct = (a.Sk + 15) / 16;                        // key tiles
    const int ldp = nct * 16 + 4;
    const float *Q = a.q + (int64_t)h * a.Sq * d;
    const float *K = a.k + (int64_t)h * a.Sk * d;
    const float *V = a.v + (int64_t)h * a.Sk * d;

    // ---- all loads: key tiles wave, wave + kWaves, ... of this wave (past the end: the last key row, not used)
    // (in the order of memory, whole lines: 64 lanes of one load that read 16 bytes of 16 rows each take 64 cycles of the L1, neighbouring ones 17.  The
    // lanes that multiply them get q and k through LDS, k through the wave's own part of it, slice after slice.)
    floatx4 qa[RT][D16], ko[MAXT][D16];
    constexpr int GS = SL / 16, lks = SL + 4;
    constexpr int LC = 32, PPL_K = LC / 4, RPL = kWave / PPL_K;          // columns, 16-byte parts and rows of one load of k
    constexpr bool Q_LATE = D16 >= 4 && RT == 1;             // query rows read from LDS again for every key tile: fewer registers
    static_assert(d % LC == 0 && LC % SL == 0 && SL % 16 == 0, "whole slices per load");
    float *const lds_q = lds + ROWS * ldp;                   // [ROWS][ldr]
    float *const lds_k = lds_q + ROWS * ldr + 16 * wave * lks;           // [16][lks]
    constexpr int PPR = 4 * D16;                             // 16-byte parts of a row of q
    floatx4 q_own = {0.f, 0.f, 0.f, 0.f};
    static_assert(ROWS * PPR <= kWaves * kWave, "16 bytes per lane");
    const int q_row = tid / PPR, q_part = tid % PPR, k_row = lane / PPL_K, k_part = lane % PPL_K;
    if (q_row < ROWS) q_own = reinterpret_cast<const floatx4 *>(Q + (int64_t)min(q0 + q_row, a.Sq - 1) * d)[q_part];
#pragma unroll
    for (int u = 0; u < MAXT; ++u)
        if (!(D16 == 8 && MAXT == 1) || wave < nct)          // (heads of 128, 16 keys: loads of the other waves took 0.2 of 4.6 us)
#pragma unroll
        for (int i = 0; i < D16; ++i)
            ko[u][i] = reinterpret_cast<const floatx4 *>(K + (int64_t)min((wave + kWaves * u) * 16 + i % (LC / 16) * RPL + k_row, a.Sk - 1) * d)[i / (LC / 16) * PPL_K + k_part];
    // (heads of 128 leave no registers for v before the scores are done)
    constexpr bool EARLY_V = D16 <= 4;
    const int ks = wave / CS, c0 = wave % CS * VT * 16;      // key tiles ks, ks + KS, ... and first column in the second product
    vecv vb[VG][4][NV];                                      // row 4s + q of the tile, columns c0 + 16 VEC c + VEC r ..
    auto load_v = [&](int u, int q) {
#pragma unroll
        for (int c = 0; c < NV; ++c)
            vb[u][q][c] = *reinterpret_cast<const vecu *>(V + (int64_t)min((ks + KS * u) * 16 + 4 * s + q, a.Sk - 1) * d + c0 + 16 * VEC * c + VEC * r);
    };
    auto load_all_v = [&] {
#pragma unroll
        for (int u = 0; u < VG; ++u)
#pragma unroll
            for (int q = 0; q < 4; ++q) load_v(u, q);
    };
    constexpr bool LATE_V = EARLY_V && MAXT > 1;             // v's loads between the products of the scores
    if constexpr (EARLY_V && !LATE_V) load_all_v();
    __builtin_amdgcn_sched_barrier(0);                       // every load leaves before anything waits
    if (q_row < ROWS) *reinterpret_cast<floatx4 *>(lds_q + q_row * ldr + 4 * q_part) = q_own;
    lds_barrier();
    auto load_q = [&](int g) {
#pragma unroll
        for (int t = 0; t < RT; ++t) qa[t][g] = *reinterpret_cast<const floatx4 *>(lds_q + (16 * t + r) * ldr + 16 * g + 4 * s);
    };
    if constexpr (!Q_LATE) {
#pragma unroll
        for (int g = 0; g < D16; ++g) load_q(g);
    }
    // ---- scores; accumulator g of a lane: row 4s + g, column r of the tile
#pragma unroll
    for (int u = 0; u < MAXT; ++u) {
        const int kt = wave + kWaves * u;
        if (kt < nct) {                                      // uniform over the wave
            floatx4 acc[RT][2];                              // even and odd groups of d apart: shorter chains
#pragma unroll
            for (int t = 0; t < RT; ++t) acc[t][0] = acc[t][1] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int g0 = 0; g0 < D16; g0 += GS) {
                floatx4 kb[GS];
                constexpr int LPB = LC / 16;                 // loads per block of LC columns
#pragma unroll
                for (int i = 0; i < LPB; ++i)
                    if (LC == SL || k_part / (SL / 4) == g0 / GS % (LC / SL))
                        *reinterpret_cast<floatx4 *>(lds_k + (i * RPL + k_row) * lks + 4 * (k_part % (SL / 4))) = ko[u][g0 / LPB * LPB + i];
#pragma unroll
                for (int g = 0; g < GS; ++g) kb[g] = *reinterpret_cast<const floatx4 *>(lds_k + r * lks + 16 * g + 4 * s);
                if constexpr (Q_LATE) {
#pragma unroll
                    for (int g = 0; g < GS; ++g) load_q(g0 + g);
                }
                constexpr int E = GS < 2 ? 1 : 2;            // groups side by side
#pragma unroll
                for (int g = 0; g < GS; g += E)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        if constexpr (LATE_V) {
                            if (g0 + g == 0) {
                                load_v(u, q);
                                __builtin_amdgcn_sched_barrier(0);
                            }
                        }
#pragma unroll
                        for (int e = 0; e < E; ++e)
#pragma unroll
                            for (int t = 0; t < RT; ++t)
                                acc[t][(g0 + e) % 2] = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[t][g0 + g + e][q], kb[g + e][q], acc[t][(g0 + e) % 2], 0, 0, 0);
                    }
            }
            const int col = kt * 16 + r;
#pragma unroll
            for (int t = 0; t < RT; ++t)
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    lds[(16 * t + 4 * s + g) * ldp + col] = col < a.Sk ? (acc[t][0][g] + acc[t][1][g]) * a.scale : -INFINITY;
        }
    }
    if constexpr (!EARLY_V) load_all_v();
    lds_barrier();                                           // (LDS only: the v operands stay in flight)

    // ---- softmax: LPR lanes per row, a lane takes the parts c, c + LPR, ...
    {
        const int c = tid % LPR, parts = nct * 4;            // 16-byte parts of a row
        float4 *row = reinterpret_cast<float4 *>(lds + tid / LPR * ldp);
        float4 v[PPL];
        float mx = -INFINITY;
#pragma unroll
        for (int i = 0; i < PPL; ++i) {
            v[i] = c + LPR * i < parts ? row[c + LPR * i] : make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
            mx = fmaxf(mx, fmaxf(fmaxf(v[i].x, v[i].y), fmaxf(v[i].z, v[i].w)));
        }
        mx = row16_max(mx);
#pragma unroll
        for (int o = 16; o < LPR; o *= 2) mx = fmaxf(mx, __shfl_xor(mx, o));
        float sum = 0.f;
#pragma unroll
        for (int i = 0; i < PPL; ++i) {                      // exp(-inf) = 0 for the padded columns
            v[i] = make_float4(__expf(v[i].x - mx), __expf(v[i].y - mx), __expf(v[i].z - mx), __expf(v[i].w - mx));
            sum += c + LPR * i < parts ? (v[i].x + v[i].y) + (v[i].z + v[i].w) : 0.f;
        }
        sum = row16_sum(sum);
#pragma unroll
        for (int o = 16; o < LPR; o *= 2) sum += __shfl_xor(sum, o);
        const float inv = 1.0f / sum;
#pragma unroll
        for (int i = 0; i < PPL; ++i)
            if (c + LPR * i < parts) row[c + LPR * i] = make_float4(v[i].x * inv, v[i].y * inv, v[i].z * inv, v[i].w * inv);
    }
    lds_barrier();

    // ---- P[ROWS x keys of this wave] V[keys x d]; A operand from LDS (row r), 16 bytes per lane
    floatx4 o[RT][VT];
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int n = 0; n < VT; ++n) o[t][n] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < VG; ++u) {
        const int kt = ks + KS * u;
        if (kt < nct) {
            float4 pa[RT];
#pragma unroll
            for (int t = 0; t < RT; ++t) pa[t] = *reinterpret_cast<const float4 *>(lds + (16 * t + r) * ldp + 16 * kt + 4 * s);
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int t = 0; t < RT; ++t)
#pragma unroll
                    for (int n = 0; n < VT; ++n)
                        o[t][n] = __builtin_amdgcn_mfma_f32_16x16x4f32((&pa[t].x)[q], vb[u][q][n / VEC][n % VEC], o[t][n], 0, 0, 0);
        }
    }
    lds_barrier();                                           // the probabilities have been read: their place holds the partial results now
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int c = 0; c < NV; ++c) {
                vecv w;
#pragma unroll
                for (int e = 0; e < VEC; ++e) w[e] = o[t][c * VEC + e][g];
                *reinterpret_cast<vecv *>(lds + (ks * ROWS + 16 * t + 4 * s + g) * ldr + c0 + 16 * VEC * c + VEC * r) = w;
            }
    lds_barrier();
#pragma unroll
    for (int e = tid; e < ROWS * d; e += kWaves * kWave) {
        const int row = e / d, col = e % d, qi = q0 + row;
        float v = 0.f;
#pragma unroll
        for (int k = 0; k < KS; ++k) v += lds[(k * ROWS + row) * ldr + col];
        if (qi < a.Sq) a.y[a.merge ? ((int64_t)qi * a.B + h) * d + col : ((int64_t)h * a.Sq + qi) * d + col] = v;
    }
}

template <int D16, int MAXT, int RT, int CS, int SL>
size_t lds_bytes(int Sk) {
    constexpr int ROWS = kRows * RT, ldr = D16 * 16 + 4;
    const int ldp = (Sk + 15) / 16 * 16 + 4;
    return (size_t)std::max(ROWS * (ldp + ldr) + 16 * kWaves * (SL + 4), kWaves / CS * ROWS * ldr) * sizeof(float);
}

template <int D16, int MAXT, int RT, int CS, int SL, class R>
int launch_as(const AttentionArgs &a, const R &r, dim3 grid, hipStream_t s) {
    const size_t lds = lds_bytes<D16, MAXT, RT, CS, SL>(a.Sk);
    if (lds > 64 * 1024) {
        static LdsLimit limit;
        const hipError_t e = limit.raise((const void *)attention_kernel<D16, MAXT, RT, CS, SL, R>);
        if (e != hipSuccess) return (int)e;
    }
    hipLaunchKernelGGL((attention_kernel<D16, MAXT, RT, CS, SL, R>), grid, dim3(kWaves * kWave), lds, s, a, r);
    return (int)hipGetLastError();
}

template <int D16, int MAXT, int RT, int CS, int SL = 32>
int launch_one(const AttentionArgs &a, const AttentionGrid &g, const Ahead *ahead, hipStream_t s) {
    const dim3 grid((unsigned)g.tiles, (unsigned)a.B);
    if (ahead && ahead->n && g.spare) return launch_as<D16, MAXT, RT, CS, SL>(a, *ahead, dim3(grid.x, grid.y + (unsigned)(g.spare / g.tiles)), s);
    return launch_as<D16, MAXT, RT, CS, SL>(a, NoAhead{}, grid, s);
}

// Up to 128 keys a wave takes one column tile of the result (a short second product: adding eight partial results would be
// the longer part); beyond, all columns of its own keys.
template <int D16>
int launch_heads(const AttentionArgs &a, const Ahead *r, hipStream_t s) {
    const int tiles = (a.Sk + 15) / 16;
    const AttentionGrid g = attention_grid(a);
    if (tiles <= kWaves) return launch_one<D16, 1, 1, D16>(a, g, r, s);
    if (tiles <= 2 * kWaves) return launch_one<D16, 2, 1, 1>(a, g, r, s);
    // Registers hold two of these workgroups per compute unit, LDS from 449 keys on only with narrower slices of k, which otherwise take 2 % longer (512 keys, slices
    // of 32 and 16 columns, us: 192 heads 102 and 83, 24 heads 17.8 and 15.8, 16 heads 9.5 and 9.7).
    if constexpr (D16 == 2)
        if (g.rows == 2 * kRows && (int64_t)g.tiles * a.B > kCUs && lds_bytes<2, 4, 2, 1, 32>(a.Sk) > 80 * 1024) return launch_one<2, 4, 2, 1, 16>(a, g, r, s);
    if constexpr (D16 <= 4)
        if (g.rows == 2 * kRows) return tiles <= 3 * kWaves ? launch_one<D16, 3, 2, 1>(a, g, r, s) : launch_one<D16, 4, 2, 1>(a, g, r, s);
    return tiles <= 3 * kWaves ? launch_one<D16, 3, 1, 1>(a, g, r, s) : launch_one<D16, 4, 1, 1>(a, g, r, s);
}

}  // namespace

bool attention_shape_ok(const AttentionArgs &a) {
    return a.B >= 1 && a.B <= 65535 && a.Sq >= 1 && a.Sk >= 1 && a.Sk <= kMaxKeys &&
           (a.d == 32 || a.d == 64 || a.d == 128) && (int64_t)a.Sq * a.d < ((int64_t)1 << 31);
}

// Two row tiles share each load of k and v, where single ones would be more than one workgroup per compute unit from 385 keys on, more
// than two below (twelve heads, one and two row tiles, us: 389 keys, heads of 64, 14.1 and 13.7, heads of 32 9.0 and 8.8; 512 keys 16.1 and 15.4, 10.3 and 9.9; 384
// heads of 64, 300 keys, 126 and 118).  The line is drawn at twelve heads, where both are one round: from 385 keys on a compute unit holds two workgroups with one row tile
// but one with two, and many heads take longer with two (24 heads, 389 keys, heads of 64 20.1 and 26.1, of 32 12.1 and 14.0; 96 heads 57 and 65, 32 and 31; 384 heads
// 206 and 241, 112 and 112).  Heads of 128 have no registers for a second row tile.
// Reading ahead: at most 64 workgroups, last, in whole rows of the grid, and only on compute units that have none of the others (one in
// the way of those made all of BERT-base on 512 rows 7 % slower).
AttentionGrid attention_grid(const AttentionArgs &a) {
    const int keys = (a.Sk + 15) / 16;                       // key tiles
    const int64_t groups = (int64_t)((a.Sq + kRows - 1) / kRows) * a.B;
    const bool two = a.d <= 64 && keys > 2 * kWaves && groups > (keys <= 3 * kWaves ? 2 : 1) * kCUs;
    AttentionGrid g;
    g.rows = two ? 2 * kRows : kRows;
    g.tiles = (a.Sq + g.rows - 1) / g.rows;
    const int64_t own = (int64_t)g.tiles * a.B;
    g.spare = own < kCUs ? (int32_t)std::min<int64_t>(kCUs - own, 64) / g.tiles * g.tiles : 0;
    return g;
}

int launch_attention(const AttentionArgs &a, const Ahead *ahead, void *stream) {
    if (!attention_shape_ok(a)) return (int)hipErrorInvalidValue;
    for (const void *p : {(const void *)a.q, (const void *)a.k})
        if (((uintptr_t)p & 15) != 0) return (int)hipErrorInvalidValue;        // rows are read 16 bytes at a time
    hipStream_t s = (hipStream_t)stream;
    return a.d == 32 ? launch_heads<2>(a, ahead, s) : (a.d == 64 ? launch_heads<4>(a, ahead, s) : launch_heads<8>(a, ahead, s));
}

}  // namespace clg
