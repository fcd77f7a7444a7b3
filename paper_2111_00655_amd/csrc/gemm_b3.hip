// Planning, weight packing and dispatch of the split-operand contraction kernels (gemm_b3.h).
#include <algorithm>

#include "gemm_b3.h"

namespace clg {

template <> int b3_launch_tile<1, false, false>(const B3Args &a, hipStream_t s);
template <> int b3_launch_tile<1, false, true>(const B3Args &a, hipStream_t s);
template <> int b3_launch_tile<9, false, false>(const B3Args &a, hipStream_t s);
template <> int b3_launch_tile<9, true, false>(const B3Args &a, hipStream_t s);
template <> int b3_launch_tile<4, false, false>(const B3Args &a, hipStream_t s);

namespace {

struct TileShape { int wm, wn, wk, tn, cw1; };
template <class C>
constexpr TileShape shape_of() { return {C::WM, C::WN, C::WK, C::TN, C::CW1}; }
TileShape tile_shape(int t) {
    switch (t) {
    case B3_L: return shape_of<B3L>();
    case B3_LM: return shape_of<B3LM>();
    case B3_M: return shape_of<B3M>();
    case B3_M8: return shape_of<B3M8>();
    case B3_M12: return shape_of<B3M12>();
    case B3_S: return shape_of<B3S>();
    case B3_SS: return shape_of<B3SS>();
    case B3_G: return shape_of<B3G>();
    default: return shape_of<B3G2>();
    }
}
// 16-channel blocks per K-wave and stage (as b3_cw)
int tile_cw(int t, int taps, bool dense) {
    const TileShape s = tile_shape(t);
    return taps != 1 || (s.wm == 1 && s.wn == 1 && !dense) ? 1 : s.cw1;
}

int ceil_div(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

// Everything of the launch that depends on the tile; false: the tile does not take the problem.  split_cus: split K across
// workgroups where the tiles leave most of that many compute units idle.
bool place(B3Args *a, int tile, int split_cus = 0) {
    const TileShape ts = tile_shape(tile);
    const int nw = ts.wm * ts.wn * ts.wk, bn = 32 * ts.tn * ts.wn;
    const int cw = tile_cw(tile, a->taps, a->dense), sc = ts.wk * cw, um = a->taps == 1 ? sc * ts.tn * ts.wn / nw : 6;
    a->tile = tile;
    a->mgroups = ceil_div(a->mtiles, ts.wm);
    if (a->groups > 1 && ts.wm != 1) return false;           // the row tiles of a workgroup share the staged channels
    a->stages = ceil_div(a->nC, sc);
    a->stages_per = a->stages;
    a->splitk = 1;
    bool ok = b3_set_div(&a->d_g32, 1, 1);
    if (a->dense) {
        a->units = sc / 2 * (bn / 16);
        a->g32 = 1;
        a->slot_stride = bn + 2;                             // four k-parts of a row are written together: two slots of shift keep them in different banks
        a->slots = bn;
        a->ntiles = a->tiles_strip = ceil_div(a->Nrows, bn);
    } else {
        // strips: as few as possible, but narrow enough that the patch of a tile stays compact
        double best = -1;
        for (int ns = 1; ns <= a->WOe; ++ns) {
            const int tw = ceil_div(a->WOe, ns);
            if (ns > 1 && (tw < 4 || tw == ceil_div(a->WOe, ns - 1))) {
                if (tw < 4) break;
                continue;
            }
            // output rows a run of bn pixels touches; a step to the next image skips the rest of its patch rows
            const int halo_h = a->KHe + a->phe_max;          // patch rows of one output row (phe_max: extra rows of the other phases)
            const int halo_w = a->KWe + a->pwe_max;
            const int rows = bn % tw == 0 ? bn / tw : ceil_div(bn - 1, tw) + 1;
            const int cross = a->Nimg > 1 ? std::min(ceil_div(rows - 1, a->HO), a->Nimg - 1) : 0;
            const int vrows = (rows - 1) * a->ly + cross * std::max(0, halo_h - a->ly) + halo_h;
            const int pw = (tw - 1) * a->lx + halo_w;
            const int slots = a->taps == 1 ? bn : vrows * pw, g32 = ceil_div(slots, 32), s = g32 * 32;
            if (sc * g32 > um * nw || (int64_t)2 * 3 * 2 * sc * s * 16 > 150 * 1024) continue;
            const int nst = ceil_div(a->WOe, tw);
            const int64_t run = (int64_t)a->Nimg * a->HO * tw;
            const double tiles = (double)nst * ceil_div(run, bn);
            const double cost = tiles * (slots + 4.0 * bn);
            if (best >= 0 && cost >= best) continue;
            best = cost;
            a->TW = tw;
            a->Ntot = (int)run;
            a->tiles_strip = ceil_div(run, bn);
            a->ntiles = nst * a->tiles_strip;
            a->rpi = (a->HO - 1) * a->ly + halo_h;
            a->pw_slots = pw;
            a->slots = slots;
            a->slot_stride = s;
            a->g32 = g32;
            a->units = sc * g32;
        }
        if (best < 0) return false;
        ok = ok && b3_set_div(&a->d_tw, a->TW, (int64_t)a->Ntot + bn) && b3_set_div(&a->d_strip, a->tiles_strip, a->ntiles) && b3_set_div(&a->d_ho, a->HO, (int64_t)a->Ntot / a->TW + bn) &&
             b3_set_div(&a->d_pw, a->pw_slots, a->slots + 64) && b3_set_div(&a->d_rpi, a->rpi, (int64_t)a->Nimg * a->rpi + a->slots) &&
             b3_set_div(&a->d_do, a->DO, a->Nimg + 64) && b3_set_div(&a->d_kd, a->KD, a->nC) && b3_set_div(&a->d_cpgo, a->groups > 1 ? a->cpg_out : 1, a->Cout + 32);
    }
    ok = ok && b3_set_div(&a->d_g32, a->g32, a->units + 64);
    a->tile_div = a->jmajor ? a->mgroups : a->ntiles;
    const int64_t wgs = (int64_t)a->mgroups * a->ntiles;
    ok = ok && wgs < ((int64_t)1 << 31) && b3_set_div(&a->d_tile, a->tile_div, wgs);
    // Too few tiles for half of the compute units (deep layers, short sequences): K is split across workgroups and a
    // second kernel adds the partial tiles and applies the fused tail.  The 64 x 64 tile gives two workgroups to a compute
    // unit (four waves leave half of each SIMD's time to memory latency), the others one.  A split keeps two stages
    // or more: a single one has nothing to load behind its products.  Dense 3072 -> 768 on 389 rows 25.5 -> 19.0 us
    // (32 x 32 tiles before), 3x3 512 -> 512 on five 7x7 images 21.6 -> 15.1, 3x3x3 256 -> 256 on 2x7x7 20.9 -> 11.9; below some
    // 10 us the best unsplit tile wins, and is a candidate of its own.
    if (split_cus && wgs * 2 <= split_cus && !a->cs_len) {
        const int64_t want = (tile == B3_M ? 2 : 1) * split_cus / wgs;
        const int ks = (int)std::min({want, (int64_t)a->stages / 2, (int64_t)16});
        if (ks > 1) {
            a->stages_per = ceil_div(a->stages, ks);
            a->splitk = ceil_div(a->stages, a->stages_per);
        }
    }
    // A wave's weights of its stages lie behind one buffer descriptor (11 million input channels of a 4x4 transposed filter are the first
    // that do not fit).
    ok = ok && (int64_t)a->stages_per * cw * a->taps * (3 * kWave * 16) < ((int64_t)1 << 31);
    a->pack_steps = (int64_t)a->mtiles * ts.wk * a->stages * cw * a->taps + 4;      // (and four steps of zeros; no kernel reads behind its stream)
    return ok;
}

}  // namespace

bool b3_resolve(const GemmArgs &g, int tile, int epi_flags, int n_cus, bool split, B3Args *out) {
    if (epi_flags & EF_GENERIC) return false;
    if (tile == B3_FIRST) return first_resolve(g, out);
    B3Args a{};
    a.epi = g.epi;
    a.c_numel = g.c_numel;
    if (g.c_numel >= ((int64_t)1 << 29)) return false;                   // 31-bit byte offsets
    a.phases = 1;
    a.groups = 1;
    a.taps = 1;
    a.DO = a.D = a.KD = 1;
    if (g.mode == GM_NT) {
        if (g.batch != 1 || g.K % 16 || (int64_t)g.M * g.lda >= ((int64_t)1 << 29) || (g.cs_len && g.cs_len % 32)) return false;
        a.dense = 1;
        a.x_bytes = (int32_t)(((int64_t)(g.M - 1) * g.lda + g.K) * 4);
        a.Cout = g.N;
        a.Nrows = g.M;
        a.K = g.K;
        a.ldx = g.lda;
        a.ldy = g.ldc;
        a.ldb = g.ldb;
        a.cs_len = g.cs_len;
        a.cs_stride = g.cs_stride;
        a.nC = ceil_div(g.K, 16);
        a.Cf = g.K;
        a.jmajor = g.M > g.N ? 1 : 0;
    } else if (g.mode == GM_CONV || g.mode == GM_CONVT) {
        const bool depth = g.D > 1 || g.KD > 1;
        a.convt = g.mode == GM_CONVT;
        a.Cin = g.Cin; a.KH = g.KH; a.KW = g.KW;
        a.H = g.H; a.W = g.W; a.HW = g.H * g.W;
        a.D = depth ? g.D : 1;
        a.KD = depth ? g.KD : 1;
        a.DO = depth ? g.DO : 1;
        a.sd = depth ? g.sd : 1;
        a.pd = depth ? g.pd : 0;
        a.Nimg = g.Nimg * a.DO;
        a.cs = a.D * a.HW;
        if ((int64_t)g.Nimg * g.Cin * a.cs >= ((int64_t)1 << 29)) return false;      // 31-bit byte offsets
        a.x_bytes = (int32_t)((int64_t)g.Nimg * g.Cin * a.cs * 4);
        a.img_stride = g.Cin * a.cs;
        a.groups = g.rf_groups > 1 ? g.rf_groups : 1;
        a.Cout = g.Cout;
        a.sh = g.sh; a.sw = g.sw;
        a.KHe = g.KH; a.KWe = g.KW;
        a.ph = g.ph; a.pwd = g.pw;
        a.HO = g.HO; a.WOe = a.WO = g.WO;
        a.os = 1;
        int she = g.sh, swe = g.sw;
        int cin = g.Cin;
        if (a.convt) {
            // phases as stride-1 convolutions over one common patch
            if (depth || a.groups > 1 || g.sh != g.sw || g.KH % g.sh || g.KW % g.sw || g.HO % g.sh || g.WO % g.sw) return false;
            a.phases = g.sh * g.sw;
            a.KHe = g.KH / g.sh;
            a.KWe = g.KW / g.sw;
            a.ph_t = g.ph;
            a.pw_t = g.pw;
            int lo_h = 1 << 30, lo_w = 1 << 30;
            a.phe_max = a.pwe_max = -(1 << 30);
            for (int q = 0; q < g.sh; ++q) {
                const int e = a.KHe - 1 - (q + g.ph) / g.sh, f = a.KWe - 1 - (q + g.pw) / g.sw;
                lo_h = std::min(lo_h, e); lo_w = std::min(lo_w, f);
                a.phe_max = std::max(a.phe_max, e); a.pwe_max = std::max(a.pwe_max, f);
            }
            if (lo_h < 0 || lo_w < 0) return false;
            a.ph = a.phe_max;
            a.pwd = a.pwe_max;
            a.HO = g.HO / g.sh;
            a.WOe = g.WO / g.sw;
            a.os = g.sh;
            she = swe = 1;
            if (!(a.KHe == 2 && a.KWe == 2) || cin % 16) return false;
            a.taps = 4;
        } else {
            if (a.groups > 1) {
                if (depth || g.Cin % a.groups || g.Cout % a.groups) return false;
                a.cpg_in = g.Cin / a.groups;
                a.cpg_out = g.Cout / a.groups;
                if (32 % a.cpg_out && a.cpg_out % 32) return false;
                if (a.cpg_out < 32 && g.Cout % 32) return false;
                cin = (a.cpg_out < 32 ? 32 / a.cpg_out : 1) * a.cpg_in;
                if (cin % 16) return false;
            }
            const bool one = g.KH == 1 && g.KW == 1, three = g.KH == 3 && g.KW == 3;
            if (one && (g.ph || g.pw)) return false;
            if (a.KD == 1 ? a.pd != 0 : !three) return false;
            if (a.groups == 1 && cin % 16 && (cin < 64 || cin % 8)) return false;      // mostly padding (first layers: first_resolve); a lane's eight channels exist or do not
            a.taps = one ? 1 : 9;
            if (!one && !three) return false;
        }
        a.Cf = cin;
        a.nC = ceil_div(cin, 16) * a.KD;
        // A slot of padding (kB3Out) stays beyond the buffer whatever channel block and depth tap are added to it: their offset has 31 bits too.
        if (depth && (int64_t)(ceil_div(cin, 16) - 1) * 16 * a.cs + (int64_t)(a.KD - 1) * a.HW >= ((int64_t)1 << 29)) return false;
        // slot geometry: with one filter row (column) only the rows (columns) that are read get slots
        a.ys = a.KHe == 1 ? she : 1;
        a.ly = a.KHe == 1 ? 1 : she;
        const bool one_col = a.KWe == 1;
        a.xs = one_col ? swe : 1;
        a.lx = one_col ? 1 : swe;
        a.npix = g.HO * g.WO;
        a.ocs = a.DO * a.npix;
        a.ons = g.Cout * a.ocs;
        a.jmajor = (int64_t)g.Nimg * g.Cin * a.cs > (int64_t)g.Cout * cin * g.KH * g.KW * a.KD ? 1 : 0;
        if (!a.convt) a.phe_max = a.pwe_max = 0;
        if ((int64_t)a.Nimg * a.HO * a.WOe > ((int64_t)1 << 28)) return false;
    } else {
        return false;
    }
    a.tiles_m = ceil_div(a.Cout, 32);
    a.mtiles = a.tiles_m * a.phases;
    if (tile == B3_M && split && a.taps == 1) {
        // No more 64 x 64 tiles than compute units: eight waves each, since four leave a SIMD one wave, which hides nothing (us, four and eight waves,
        // five images: 256 -> 64 at 50x50, 196 tiles, 9.2 and 7.9; 256 -> 1024 at 13x13, 224 tiles, 9.9 and 8.3; 2048 -> 512 at 7x7, 32 tiles and K split, 14.1 and
        // 11.3; dense 768 -> 3072 on 200 rows, 192 tiles, 14.0 and 11.9).  Where units get several workgroups the smaller one
        // is better (64 -> 256 at 50x50, 784 tiles, 13.7 and 21; dense 768 -> 3072 on 389 rows, 336 tiles, 20.4 and 22.3).
        B3Args b = a;
        if (place(&b, B3_M8, n_cus) && (int64_t)b.mgroups * b.ntiles <= n_cus) {
            *out = b;
            return true;
        }
        // Dense layers with more than that, but no more 96 x 64 tiles than compute units: every unit has one tile and one round, of 12 waves, where
        // some would have two of the small ones and others one (us, 64 x 64 tiles, 96 x 64 ones of six and of 12 waves: 768 -> 3072 on 389 rows, 336 and
        // 224 tiles, 19.9, 18.0 and 16.0, on 353 rows 19.4, 17.0 and 15.5; 768 -> 4096 on 300 rows 19.8, 18.0 and 16.0; 1024 -> 3072 on 384 rows 24.0, 22.9
        // and 20.2; 768 -> 2048 on 700 rows 20.4, 18.6 and 17.5).  1x1 filters, whose loads are short of registers: 256 -> 1024 on six 14x14 12.1, 12.9.
        B3Args c = a;
        if (a.dense && place(&c, B3_M12) && (int64_t)c.mgroups * c.ntiles <= n_cus) {
            *out = c;
            return true;
        }
    }
    // So it is with 3x3 and 2x2 taps where a tile's K is long, from 256 channels on, and not split (us, four and eight waves: 3x3 512 -> 512 on 32 7x7
    // 46.2 and 41.9, on 24 45.8 and 41.5, 256 -> 256 on 16 14x14 24.3 and 22.3, on 20 25.9 and 24.4; 4x4 transposed, stride 2, 512 -> 256 on 64 4x4 37.5 and
    // 35.9, 256 -> 128 on 32 8x8 18.1 and 17.2.  128 -> 128 on eight 28x28 17.1 and 17.3; split, 512 -> 512 on five 7x7 14.5 and 18.9).
    if (tile == B3_M && split && a.taps != 1 && a.KD == 1 && a.nC >= 16) {
        B3Args b = a;
        if (place(&b, B3_M8)) {
            const int64_t tiles = (int64_t)b.mgroups * b.ntiles;
            if (tiles <= n_cus && tiles * 2 > n_cus) {
                *out = b;
                return true;
            }
        }
    }
    if (tile != B3_NONE) {
        if (!place(&a, tile, split ? n_cus : 0)) return false;
    } else {
        // the largest tile that gives every compute unit a workgroup; row tiles no taller than the problem
        const int wide[] = {B3_L, B3_LM, B3_M, B3_S, B3_SS}, narrow[] = {B3_G, B3_G2, B3_S, B3_SS};
        const bool few_rows = a.mtiles == 1 || a.groups > 1;
        bool found = false;
        for (int n = 0; n < (few_rows ? 4 : 5); ++n) {
            B3Args b = a;
            const int t = few_rows ? narrow[n] : wide[n];
            if (t == B3_L && a.mtiles < 4) continue;
            if (!place(&b, t)) continue;
            *out = b;
            found = true;
            if ((int64_t)b.mgroups * b.ntiles >= n_cus) break;
        }
        return found;
    }
    *out = a;
    return true;
}

bool b3_region_resolve(const GemmArgs *m, int n, int n_cus, B3Args *out) {
    if (n < 2 || n > kMaxB3Region) return false;
    const GemmArgs &a = m[0];
    for (int k = 1; k < n; ++k) {
        const GemmArgs &b = m[k];
        if (b.mode != a.mode || b.M != a.M || b.N != a.N || b.K != a.K || b.lda != a.lda || b.ldb != a.ldb || b.ldc != a.ldc || b.batch != a.batch ||
            b.c_numel != a.c_numel || b.cs_len != a.cs_len || b.cs_stride != a.cs_stride || b.epi.n != a.epi.n)
            return false;
        for (int s = 0; s < a.epi.n; ++s)
            if (b.epi.s[s].op != a.epi.s[s].op || b.epi.s[s].scalar != a.epi.s[s].scalar) return false;
    }
    // Where the members have fewer 32 x 32 tiles than for 3/4 of the compute units, the register-fed region is as fast or faster (one
    // launch of siblings and a relu, us, split-operand against register-fed: two layers 256 -> 256 on 384 rows, 192 tiles, 7.4 and 7.1;
    // three on 200 rows, 168 tiles, 7.2 and 6.9, four on 256, 256 tiles, 7.4 and 7.5; two 512 -> 512 on 160 rows, 160
    // tiles, 8.6 and 8.5, on 200, 224 tiles, 8.7 and 9.3; three 768 -> 768 on 200 rows 12.5 and 14.9, four 1024 -> 1024 on 512 32 and 56).
    if ((int64_t)n * ((a.M + 31) / 32) * ((a.N + 31) / 32) * 4 <= (int64_t)3 * n_cus) return false;
    // 64 x 64 tiles once the members have them for 9/16 of the compute units, four-wave 32 x 32 ones before.  Two layers of BERT-base,
    // us with q, k, v on the fp32 register-fed region, on 64 x 64 and on 32 x 32 tiles: 128 rows 99.0, 106.8, 98.3; 200 rows
    // 132.2, 133.8, 130.8; 256 rows 139.2, 138.0, 140.7; 320 rows 152.1, 144.7, 149.4; 389 rows 202.4, 190.2, 195.6.
    // With no more 64 x 64 tiles, or else 96 x 64 ones, than compute units, the members get those of eight or twelve waves, as a layer alone does
    // (b3_resolve).  All of BERT-base, us, its q, k and v on four waves per tile and on these: 256 rows 816 and 793, 320 rows 911 and 888, 389 rows
    // 1105 and 1086 (252 tiles of 64 x 64), 512 rows 1267 and 1222 (288 of them, 192 of 96 x 64).  With 64 x 64 tiles from 5/16 of the units on: 160
    // rows 657 -> 677, 200 rows 792 -> 785.
    const int tile = (int64_t)n * a.M * a.N >= (int64_t)64 * 64 * (n_cus * 9 / 16) ? B3_M : B3_SS;
    if (a.mode != GM_NT) return false;
    if (tile == B3_M) {
        for (int t : {B3_M8, B3_M12})
            if (b3_resolve(a, t, epi_fast_flags(a.epi), n_cus, false, out) && out->dense && (int64_t)n * out->mgroups * out->ntiles <= n_cus) return true;
    }
    return b3_resolve(a, tile, epi_fast_flags(a.epi), n_cus, false, out) && out->dense;
}

int launch_b3_region(const B3Args *members, int n, void *stream) {
    if (n < 2 || n > kMaxB3Region) return (int)hipErrorInvalidValue;
    B3Args a = members[0];
    B3Region r{};
    r.n = n;
    for (int k = 0; k < n; ++k) {
        const EpiFast ef = make_epi_fast(members[k].epi);
        if (ef.flags & EF_GENERIC) return (int)hipErrorInvalidValue;
        r.x[k] = members[k].x;
        r.w[k] = members[k].w;
        r.y[k] = members[k].y;
        r.bias[k] = ef.bias;
        r.add[k] = ef.add;
        a.ef = ef;
    }
    a.region = &r;
    return b3_launch_tile<1, false, true>(a, (hipStream_t)stream);
}

size_t b3_pack_bytes(const B3Args &a) { return (size_t)a.pack_steps * 3 * kWave * 16; }

size_t b3_scratch_bytes(const B3Args &a) { return a.splitk > 1 ? (size_t)a.splitk * (size_t)a.c_numel * sizeof(float) : 0; }

namespace {

// Adds split-K partial tiles in slice order and applies the fused tail, V consecutive values per thread (four where they
// share a channel, or have four neighbouring ones).  A slice is at most 2 MB and in some XCD's L2, so the bound is the latency of the
// loads: F slices' leave together, from workgroups of one wave, which reach four times as many compute units as 256 threads do (all
// of a 512 -> 512 layer on 4x4 is 32 KB).  Layer and reduction, us, with 256 threads and four slices, one wave and eight, one wave and
// 16: 3x3x3 512 -> 512 on 1x4x4 (16 slices) 15.0, 14.2, 13.8; 256 -> 256 on 2x7x7 (12) 12.6, 12.3, 11.9; 128 -> 128 on 4x14x14 (6) 13.9,
// 13.5, 13.6; 3x3 512 -> 512 on five 7x7 (8) 15.5, 15.1, 15.4; 1x1 2048 -> 512 on those (8) 11.4, 11.1, 11.2.
constexpr int kReduceThreads = kWave;
template <int V, int F>
__global__ __launch_bounds__(kReduceThreads) void b3_reduce_kernel(const float *partial, float *y, uint32_t numel, int splitk, EpiFast ef,
                                                                   uint32_t inner, uint32_t channels) {
    const uint32_t i = (blockIdx.x * (uint32_t)kReduceThreads + threadIdx.x) * V;
    if (i >= numel) return;
    typedef float vec __attribute__((ext_vector_type(V)));
    auto at = [](const float *p, uint32_t o) { return *reinterpret_cast<const vec *>(p + o); };
    vec bv = 0.f, av = 0.f, sum = 0.f;
    const auto parts = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(partial), (short)0, (int)(splitk * numel * 4), 0x00020000);
    for (int k = 0; k < splitk; k += F) {
        vec v[F];
#pragma unroll
        for (int e = 0; e < F; ++e) {               // (behind the last slice: beyond the buffer, zero)
            const int o = (int)(((uint32_t)(k + e) * numel + i) * 4u);
            if constexpr (V == 4) v[e] = __builtin_bit_cast(vec, __builtin_amdgcn_raw_buffer_load_b128(parts, o, 0, 0));
            else v[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(parts, o, 0, 0));
        }
        if (k == 0) {
            if (ef.flags & EF_BIAS) {
                if (inner == 1) bv = at(ef.bias, i % channels);
                else bv = ef.bias[i / inner % channels];
            }
            if (ef.flags & EF_ADD) av = at(ef.add, i);
        }
#pragma unroll
        for (int e = 0; e < F; ++e) sum += v[e];
    }
    float v[V], b[V], a[V];
#pragma unroll
    for (int e = 0; e < V; ++e) {
        v[e] = sum[e];
        b[e] = bv[e];
        a[e] = av[e];
    }
    fused_tail<V>(ef, v, b, a);
    vec out;
#pragma unroll
    for (int e = 0; e < V; ++e) out[e] = v[e];
    *reinterpret_cast<vec *>(y + i) = out;
}

int launch_b3_reduce(const B3Args &a, hipStream_t s) {
    const uint32_t n = (uint32_t)a.c_numel, inner = (uint32_t)std::max(a.epi.bias_inner, 1), c = (uint32_t)std::max(a.epi.bias_c, 1);
    const bool bias = a.ef.flags & EF_BIAS;
    bool four = n % 4 == 0 && (!bias || (inner == 1 ? c % 4 == 0 : inner % 4 == 0));
    for (const void *p : {(const void *)a.partial, (const void *)a.y, (const void *)a.ef.add, (const void *)(inner == 1 ? a.ef.bias : nullptr)})
        four = four && ((uintptr_t)p & 15) == 0;
    const uint32_t per = (uint32_t)kReduceThreads * (four ? 4 : 1);
    const auto kernel = a.splitk > 8 ? (four ? b3_reduce_kernel<4, 16> : b3_reduce_kernel<1, 16>) : (four ? b3_reduce_kernel<4, 8> : b3_reduce_kernel<1, 8>);
    hipLaunchKernelGGL(kernel, dim3((n + per - 1) / per), dim3(kReduceThreads), 0, s, a.partial, a.y, n, a.splitk, a.ef, inner, c);
    return (int)hipGetLastError();
}

// One thread per (step, lane): eight weights of row lane % 32, k = 16 * block + 8 * (lane / 32) + 0..7, in three planes.
__global__ __launch_bounds__(256) void b3_pack_kernel(const float *w, u32x4 *dst, B3Args p, int wk_n, int cw) {
    const int64_t d = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t step = d >> 6;
    if (step >= p.pack_steps) return;
    const int lane = (int)(d & 63);
    const int64_t per_wave = (int64_t)p.stages * cw * p.taps;
    const int64_t wave = step / per_wave;                    // (row tile, K-wave)
    const int n = (int)(step - wave * per_wave);
    const int tap = n % p.taps, blk = n / p.taps;            // block: stage * cw + c
    const int wk = (int)(wave % wk_n);
    const int64_t mt = wave / wk_n;
    const int phase = (int)(mt / p.tiles_m);
    const int i = (int)(mt - (int64_t)phase * p.tiles_m) * 32 + lane % 32;
    const int b = (blk / cw) * wk_n * cw + wk * cw + blk % cw;         // block of 16 channels (and depth tap)
    const int c16 = b / p.KD, kd = b - c16 * p.KD;
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int c = c16 * 16 + (lane / 32) * 8 + e;
        float x = 0.f;
        if (mt < p.mtiles && i < p.Cout && c < p.Cf) {
            if (p.dense) {
                x = w[(int64_t)i * p.ldb + c];
            } else if (p.convt) {
                // w is [Cin][Cout][KH][KW]; tap u of the phase is kernel tap r + s * (KH/s - 1 - u)
                const int a_h = phase / p.sw, a_w = phase - a_h * p.sw;
                const int uh = tap / p.KWe, uw = tap - uh * p.KWe;
                const int kh = (a_h + p.ph_t) % p.sh + p.sh * (p.KHe - 1 - uh), kw = (a_w + p.pw_t) % p.sw + p.sw * (p.KWe - 1 - uw);
                x = w[(((int64_t)c * p.Cout + i) * p.KH + kh) * p.KW + kw];
            } else if (p.groups > 1) {
                const int ch = ((i / 32 * 32) / p.cpg_out) * p.cpg_in + c, grp = i / p.cpg_out;
                if (ch / p.cpg_in == grp) x = w[((int64_t)i * p.cpg_in + (ch - grp * p.cpg_in)) * p.taps + tap];
            } else {
                x = w[(((int64_t)i * p.Cin + c) * p.KD + kd) * p.taps + tap];
            }
        }
        v[e] = x;
    }
    u32x4 pl[3];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        uint32_t h, m, l;
        b3_split2_full(v[2 * e], v[2 * e + 1], h, m, l);
        pl[0][e] = h;
        pl[1][e] = m;
        pl[2][e] = l;
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) dst[(step * 3 + k) * kWave + lane] = pl[k];
}

}  // namespace

int launch_b3_pack(const B3Args &a, const float *w, void *dst, void *stream) {
    if (a.tile == B3_FIRST) return launch_b3_first_pack(a, w, dst, (hipStream_t)stream);
    const int64_t threads = a.pack_steps * kWave;
    hipLaunchKernelGGL(b3_pack_kernel, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, (hipStream_t)stream, w, (u32x4 *)dst, a,
                       tile_shape(a.tile).wk, tile_cw(a.tile, a.taps, a.dense));
    return (int)hipGetLastError();
}

int launch_b3(const B3Args &a_in, void *stream, bool reduce) {
    B3Args a = a_in;
    hipStream_t s = (hipStream_t)stream;
    a.ef = make_epi_fast(a.epi);
    if (a.ef.flags & EF_GENERIC) return (int)hipErrorInvalidValue;
    int e;
    if (a.tile == B3_FIRST) return launch_b3_first(a, s);
    if (a.dense) e = b3_launch_tile<1, false, true>(a, s);
    else if (a.taps == 1) e = b3_launch_tile<1, false, false>(a, s);
    else if (a.taps == 9) e = a.KD > 1 ? b3_launch_tile<9, true, false>(a, s) : b3_launch_tile<9, false, false>(a, s);
    else if (a.taps == 4) e = b3_launch_tile<4, false, false>(a, s);
    else e = (int)hipErrorInvalidValue;
    if (e || a.splitk <= 1 || !reduce) return e;
    return launch_b3_reduce(a, s);
}

}  // namespace clg
