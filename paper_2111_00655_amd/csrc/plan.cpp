// Placement -> kernel sequence (paper Sec. 4.1: a placement is a set of
// disjoint matches covering G; Sec. 5.1: tensors are handed between backends
// by pointer, without copies), and its execution on a HIP stream.
#include <algorithm>
#include <map>

#include <hip/hip_runtime_api.h>

#include "core.h"

namespace clg {

namespace {

constexpr int64_t kAlign = 256;
int64_t round_up(int64_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

// First-fit allocator over one linear workspace; tracks the peak.
struct Arena {
    struct Block { int64_t off, size; };
    std::vector<Block> live;     // sorted by offset
    int64_t peak = 0;
    int64_t alloc(int64_t bytes) {
        const int64_t size = round_up(std::max<int64_t>(bytes, 1));
        int64_t off = 0;
        size_t pos = 0;
        for (; pos < live.size(); ++pos) {
            if (live[pos].off - off >= size) break;
            off = live[pos].off + live[pos].size;
        }
        live.insert(live.begin() + (long)pos, Block{off, size});
        peak = std::max(peak, off + size);
        return off;
    }
    void release(int64_t off) {
        for (size_t i = 0; i < live.size(); ++i)
            if (live[i].off == off) {
                live.erase(live.begin() + (long)i);
                return;
            }
    }
};

std::vector<int32_t> operands_of(const KernelCall &c) {
    std::vector<int32_t> v;
    for (int32_t x : {c.a_node, c.b_node, c.c_node})
        if (x >= 0) v.push_back(x);
    for (int32_t x : c.epi_nodes)
        if (x >= 0) v.push_back(x);
    return v;
}

// ---- regions (the graph-level backend, paper Sec. 4.3) -------------------------------------------
// Which several-problems-per-launch kernel could run the call beside siblings of the same class
// (0: none): 1 dense with packed weights, 2 register-fed 1x1 convolution, 3 thread-per-output kernels
// (depthwise convolution with its unrolled-tap kernel, window pools), 100 and up separable convolutions.
enum RegionClass { RC_NONE = 0, RC_DENSE = 1, RC_CONV1X1 = 2, RC_PLANE = 3, RC_SEPCONV = 100 };
int region_class(const KernelCall &c) {
    if (c.kind == CALL_SEPCONV) return RC_SEPCONV + sepconv_region_key(c.sep);      // one class per kernel instantiation
    if (c.kind == CALL_DIRECT_CONV) return depthwise_fast_ok(c.dconv) ? RC_PLANE : RC_NONE;
    if (c.kind == CALL_POOL) return plane_region_pool_ok(c.pool) ? RC_PLANE : RC_NONE;
    if (c.kind == CALL_B3) return c.b3.dense ? RC_DENSE : RC_NONE;
    if (c.kind != CALL_GEMM || !c.gemm.rf_ts || c.gemm.splitk != 1 || !c.pack_bytes) return RC_NONE;
    const GemmArgs &a = c.gemm;
    if (a.rf_tapk == -1) return a.rf_ragged ? RC_NONE : RC_DENSE;
    return a.rf_tapk == 1 && !a.rf_convt && !a.rf_fold ? RC_CONV1X1 : RC_NONE;
}

// A dense call on the register-fed kernel: itself, or a split-operand one lowered again for 16 x 16 tiles and at most four
// K-waves, which is what the search places most on layers of 128 - 512 rows.
bool register_fed(const Context &ctx, const KernelCall &c, KernelCall *out) {
    *out = c;
    if (c.kind != CALL_B3) return true;
    if (!rf_resolve_dense(&out->gemm, 16, epi_fast_flags(out->gemm.epi), ctx.n_cus, -4, 1)) return false;
    out->kind = CALL_GEMM;
    out->pack_bytes = rf_pack_bytes(out->gemm);
    out->scratch_bytes = 0;
    return true;
}

// Lowers member `c` again for the leader's kernel shape (tile edge, K-waves per workgroup).
bool relower_for(const Context &ctx, const KernelCall &leader, const KernelCall &c, KernelCall *out) {
    if (!register_fed(ctx, c, out)) return false;
    if (out->kind != CALL_GEMM) return true;                 // thread-per-output kernels: every member runs as it is
    GemmArgs &a = out->gemm;
    const int ts = leader.gemm.rf_ts, wgk = leader.gemm.rf_wgk;
    if (a.rf_ts != ts || a.rf_wgk != wgk || a.rf_nb != leader.gemm.rf_nb) {
        const int flags = epi_fast_flags(a.epi);
        const bool dense = a.rf_tapk == -1;
        if (!dense && (a.KD > 1 || a.rf_fold)) return false;
        const bool ok = dense ? rf_resolve_dense(&a, ts, flags, ctx.n_cus, wgk, leader.gemm.rf_nb == 2 ? 2 : 1)
                              : rf_resolve(&a, ts, flags, ctx.n_cus, wgk);
        if (!ok) return false;
        out->pack_bytes = rf_pack_bytes(a);
        out->scratch_bytes = gemm_scratch_bytes(a);
    }
    return out->scratch_bytes == 0 && rf_same_launch_shape(leader.gemm, a);
}

// Dense siblings of one shape and tail with enough rows and tiles run on the split-operand kernel inside a region, whatever
// kernel each would use alone (figures: b3_region_resolve, kB3DenseRows).  Leaves `fused` empty otherwise.
bool dense_region_b3(const Context &ctx, const std::vector<KernelCall> &calls, const std::vector<int32_t> &members, std::vector<KernelCall> *fused) {
    const size_t n = members.size();
    if (n > kMaxB3Region) return false;
    GemmArgs m[kMaxB3Region];
    for (size_t k = 0; k < n; ++k) m[k] = calls[(size_t)members[k]].gemm;
    B3Args b;
    if (m[0].M < kB3DenseRows || !b3_region_resolve(m, (int)n, ctx.n_cus, &b)) return false;
    for (size_t k = 0; k < n; ++k) {
        fused->push_back(calls[(size_t)members[k]]);
        KernelCall &c = fused->back();
        c.kind = CALL_B3;
        c.b3 = b;
        c.b3.epi = m[k].epi;
        c.pack_bytes = b3_pack_bytes(b);
        c.scratch_bytes = 0;
    }
    return true;
}

// A 1x1 convolution, separable or depthwise convolution or window pool as member of a mixed region: the kind under which it runs there (0: it does
// not).  *out: the call, a convolution lowered again for 16 x 16 tiles and at most eight waves per tile.
int32_t mix_kind(const Context &ctx, const KernelCall &c, KernelCall *out) {
    *out = c;
    if (c.kind == CALL_SEPCONV) return mix_sep_kind(c.sep);
    if (c.kind == CALL_DIRECT_CONV) return depthwise_fast_ok(c.dconv) ? c.dconv.KH : 0;
    if (c.kind == CALL_POOL) return plane_region_pool_ok(c.pool) ? (c.pool.mode == 0 ? MIX_MAX : MIX_AVG) : 0;
    if (c.kind != CALL_GEMM || !c.gemm.rf_ts || !c.pack_bytes || c.gemm.mode != GM_CONV || c.gemm.KH != 1 || c.gemm.KW != 1 || c.gemm.D > 1) return 0;
    GemmArgs &a = out->gemm;
    const int flags = epi_fast_flags(a.epi);
    if (!rf_resolve(&a, 16, flags, ctx.n_cus, -8)) return 0;
    out->pack_bytes = rf_pack_bytes(a);
    out->scratch_bytes = 0;
    return mix_conv_kind(a);
}

// Calls in order of their distance from the graph's inputs, if that brings together kernels that a mixed region can hold: a
// region's members read nothing that its first kernel or a later one makes, and in the order of the sinks' depths a separable convolution of one
// kernel (five operators deep) and a pool (one operator) that read the same tensor lie far apart.  Concatenations that can be aliases count nothing.
void order_by_level(const Context &ctx, const Graph &g, std::vector<KernelCall> *calls) {
    const size_t nc = calls->size();
    std::vector<int32_t> level(nc, 0), at(g.nodes.size(), -1), order(nc);
    std::map<int32_t, int32_t> kind_at;                      // level -> kind of the first member there
    auto free_of_charge = [&](size_t i) { return (*calls)[i].kind == CALL_CONCAT && (*calls)[i].cat.outer == 1; };
    bool mixed = false;
    for (size_t i = 0; i < nc; ++i) {
        for (int32_t v : operands_of((*calls)[i])) {
            const int32_t j = at[v];
            if (j >= 0) level[i] = std::max(level[i], level[(size_t)j] + (free_of_charge(i) ? 0 : 1));
        }
        at[(*calls)[i].out_node] = (int32_t)i;
        order[i] = (int32_t)i;
        KernelCall c;
        const int32_t kind = mix_kind(ctx, (*calls)[i], &c);
        if (kind && kind_at.emplace(level[i], kind).first->second != kind) mixed = true;
    }
    if (!mixed) return;
    std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) {
        return level[(size_t)a] != level[(size_t)b] ? level[(size_t)a] < level[(size_t)b] : free_of_charge((size_t)a) < free_of_charge((size_t)b);
    });
    std::vector<KernelCall> moved;
    moved.reserve(nc);
    for (int32_t i : order) moved.push_back(std::move((*calls)[(size_t)i]));
    calls->swap(moved);
}

// Finds the regions of a freshly lowered kernel sequence and moves every member next to its region's
// first one (a member only moves forward past kernels it does not depend on, so the order stays
// topological).  Greedy and deterministic: scanning in order, a kernel of a fusable kind opens a
// region; later kernels of the same family join when everything they read was produced before the
// region's first kernel and the common kernel shape (that of the member with the most flops) takes them.  Where more kernels of
// several kinds are free than of the opener's, they are a mixed region, if `allow_mixed`.
void find_regions(const Context &ctx, const Graph &g, bool allow_mixed, Plan *plan) {
    std::vector<KernelCall> &calls = plan->calls;
    const size_t nc = calls.size();
    if (allow_mixed) order_by_level(ctx, g, &calls);
    std::vector<int32_t> produced_at(g.nodes.size(), -1);
    for (size_t i = 0; i < nc; ++i) produced_at[calls[i].out_node] = (int32_t)i;
    std::vector<int32_t> reg_of(nc, -1);
    struct Found { std::vector<int32_t> members; std::vector<KernelCall> fused; bool mixed = false; };
    std::vector<int32_t> kind(nc, 0);
    std::vector<KernelCall> as_mixed(nc);
    for (size_t i = 0; i < nc && allow_mixed; ++i) kind[i] = mix_kind(ctx, calls[i], &as_mixed[i]);
    std::vector<Found> found;
    for (size_t i = 0; i < nc; ++i) {
        const int cls = region_class(calls[i]);
        if (reg_of[i] >= 0 || (cls == RC_NONE && !kind[i])) continue;
        std::vector<int32_t> cand{(int32_t)i}, mix;
        const size_t cap = cls == RC_PLANE ? (size_t)kMaxPlaneRegion : (cls >= RC_SEPCONV ? (size_t)kMaxSepRegion : (size_t)kMaxRegion);
        if (kind[i]) mix.push_back((int32_t)i);
        for (size_t j = i + 1; j < nc; ++j) {
            const bool like = cls != RC_NONE && region_class(calls[j]) == cls && cand.size() < cap, other = kind[i] && kind[j] && mix.size() < (size_t)kMaxMixRegion;
            if (reg_of[j] >= 0 || (!like && !other)) continue;
            bool free = true;
            for (int32_t v : operands_of(calls[j]))
                if (g.nodes[v].is_op() && produced_at[v] >= (int32_t)i) free = false;
            if (free && like) cand.push_back((int32_t)j);
            if (free && other) mix.push_back((int32_t)j);
        }
        if (mix.size() > cand.size()) {
            Found f;
            f.mixed = true;
            f.members = mix;                               // (in the plan's order; a launch takes them by weight)
            for (int32_t c : mix) {
                f.fused.push_back(as_mixed[(size_t)c]);
                reg_of[(size_t)c] = (int32_t)found.size();
            }
            found.push_back(std::move(f));
            continue;
        }
        if (cand.size() < 2) continue;
        int32_t lead = cand[0];
        for (int32_t c : cand)
            if (calls[c].flops > calls[lead].flops) lead = c;
        Found f;
        if (cls == RC_DENSE) {
            // siblings of one shape: the split-operand kernel, four of them where the opener runs it alone as well; others: the register-fed one
            if (calls[i].kind == CALL_B3 && cand.size() > (size_t)kMaxB3Region) {
                const std::vector<int32_t> four(cand.begin(), cand.begin() + kMaxB3Region);
                if (dense_region_b3(ctx, calls, four, &f.fused)) cand = four;
            } else {
                (void)dense_region_b3(ctx, calls, cand, &f.fused);
            }
            if (!f.fused.empty()) f.members = cand;
        }
        KernelCall leader;
        if (f.members.empty() && register_fed(ctx, calls[lead], &leader))
            for (int32_t c : cand) {
                KernelCall fc;
                if (relower_for(ctx, leader, calls[c], &fc)) {
                    f.members.push_back(c);
                    f.fused.push_back(std::move(fc));
                }
            }
        if (f.members.size() < 2 || f.members[0] != (int32_t)i) continue;     // the opener must be in (else try from the next kernel)
        for (int32_t c : f.members) reg_of[c] = (int32_t)found.size();
        found.push_back(std::move(f));
    }
    plan->regions.clear();
    plan->region_of.assign(nc, -1);
    plan->fuse_mark.assign(nc, 0);
    if (found.empty()) return;
    // new order: a region's members right behind its first one
    std::vector<int32_t> order, new_pos(nc, -1);
    for (size_t i = 0; i < nc; ++i) {
        if (reg_of[i] >= 0 && found[reg_of[i]].members[0] != (int32_t)i) continue;     // emitted with its region
        if (reg_of[i] < 0) {
            new_pos[i] = (int32_t)order.size();
            order.push_back((int32_t)i);
        } else {
            for (int32_t c : found[reg_of[i]].members) {
                new_pos[c] = (int32_t)order.size();
                order.push_back(c);
            }
        }
    }
    std::vector<KernelCall> moved;
    moved.reserve(nc);
    for (int32_t c : order) moved.push_back(std::move(calls[c]));
    calls.swap(moved);
    for (Found &f : found) {
        Region r;
        for (int32_t c : f.members) {
            r.members.push_back(new_pos[c]);
            plan->region_of[new_pos[c]] = (int32_t)plan->regions.size();
        }
        r.fused = std::move(f.fused);
        r.mixed = f.mixed;
        r.order.resize(r.members.size());
        for (size_t k = 0; k < r.order.size(); ++k) r.order[k] = (int32_t)k;
        if (r.mixed) {
            auto weight = [&](int32_t k) {
                KernelCall c;
                return mix_weight(mix_kind(ctx, r.fused[(size_t)k], &c));
            };
            std::stable_sort(r.order.begin(), r.order.end(), [&](int32_t a, int32_t b) { return weight(a) > weight(b); });
        }
        r.packed.assign(r.members.size(), nullptr);
        plan->regions.push_back(std::move(r));
    }
}

// Lowers a register-fed dense layer in front of a layer norm again, with K split four ways in workgroups of four waves, where that shares out long
// rows better: the layer norm adds up the partial results at no launch of its own.  The lines were drawn by whole encoders under one placement, unsplit and split, by the
// number T of 16 x 16 tiles on 256 compute units (us; layers written K -> N):
//  * T <= half the compute units, from K = 2048 on.  3072 -> 768 T = 48 434 and 401, 96 460 and 448; 4096 -> 1024 64 327 and 292, 128 363 and 348; 2048 -> 512 64 321 and 311, 128 349 and 345;
//    3584 -> 896 56 357 and 330; 6144 -> 1536 96 238 and 229; 2816 -> 704 44 432 and 399; 2560 -> 768 96 447 and 447; the one loss 2560 -> 640 120 416 and 422.
//  * From half a round of tiles to one: nothing to gain (3072 -> 768 144, 192 and 240: 476 and 476, 497 and 496, 511 and 513).
//  * Between one round of tiles and one and a quarter, where K's chunks share out evenly over slices and waves (K % 1024 = 0) and the layer norm has four slices in flight
//    (N <= 1024): 3072 -> 768 288 589 and 575, 4096 -> 768 288 643 and 630, 4096 -> 1024 320 475 and 469, 3072 -> 1024 320 433 and 423, 3072 -> 512 288 760 and 719; otherwise 2560 -> 640 320 547 and 562,
//    3584 -> 896 280 498 and 506, 3072 -> 1152 288 351 and 355.  From K = 3072 on: 2048 -> 768 288 490 and 517, 2048 -> 512 320 496 and 496.
//  * Up to one and a half rounds, as long as K is below 4096: 3072 -> 768 384 627 and 620, 3072 -> 1024 384 449 and 441, 3072 -> 896 336 486 and 481, but 4096 -> 1024 384 486 and 490, 4096 -> 768
//    336 655 and 655, 384 675 and 681.  More tiles: 3072 -> 768 432 650 and 657, 480 658 and 674.
// Split 2, 3, 6 and 12 ways, or in workgroups of eight and sixteen waves, 3072 -> 768 is up to 4 % slower than so; 768 -> 768 as well 1 - 2 % slower.
bool split_for_norm(const Context &ctx, const KernelCall &own, KernelCall *c) {
    *c = own;
    GemmArgs a = own.gemm;
    const int64_t tiles = (int64_t)((a.M + 15) / 16) * ((a.N + 15) / 16), n = ctx.n_cus;
    const bool few = a.K >= 2048 && tiles * 2 <= n;
    const bool more = a.K >= 3072 && a.K % 1024 == 0 && a.N <= 1024 && tiles > n && tiles * 4 <= (a.K < 4096 ? 6 : 5) * n;
    if (!few && !more) return false;
    if (!rf_resolve_dense(&a, 16, epi_fast_flags(a.epi), ctx.n_cus, -4, 1, 4) || a.splitk < 2) return false;
    c->gemm = a;
    c->pack_bytes = rf_pack_bytes(a);
    c->scratch_bytes = gemm_scratch_bytes(a);
    c->name = "dense_rf16_w" + std::to_string(a.rf_wgk) + "_k" + std::to_string(a.splitk);
    return true;
}

// Finds the joins of a sequence in its final order.
void find_joins(const Context &ctx, const Graph &g, Plan *plan) {
    const std::vector<KernelCall> &calls = plan->calls;
    const size_t nc = calls.size();
    plan->joins.clear();
    plan->join_of.assign(nc, -1);
    std::vector<int32_t> readers(g.nodes.size(), 0);
    for (const KernelCall &c : calls)
        for (int32_t v : operands_of(c)) ++readers[v];
    auto reads = [](const KernelCall &c, int32_t v) {
        const std::vector<int32_t> in = operands_of(c);
        return std::count(in.begin(), in.end(), v);
    };
    auto add = [&](const Join &j) {
        for (int32_t k = 0; k < j.n; ++k) plan->join_of[j.first + k] = (int32_t)plan->joins.size();
        plan->joins.push_back(j);
    };
    auto alone = [&](size_t i, int32_t kind) { return i < nc && calls[i].kind == kind && plan->region_of[i] < 0 && plan->join_of[i] < 0; };
    for (size_t i = 0; i < nc; ++i) {
        for (size_t d : {i + 1, i}) {                        // the dense layer: behind a pool, or the first
            if (plan->join_of[i] >= 0 || !alone(i, d == i ? CALL_GEMM : CALL_POOL) || !alone(d, CALL_GEMM) || !alone(d + 1, CALL_ROWWISE)) continue;
            const KernelCall &dense = calls[d], &soft = calls[d + 1];
            if (dense.gemm_swap || soft.a_node != dense.out_node || (d != i && (dense.a_node != calls[i].out_node || reads(dense, calls[i].out_node) != 1))) continue;
            Join j{};
            j.kind = JOIN_CLASSIFIER;
            j.first = (int32_t)i;
            j.n = (int32_t)(d + 2 - i);
            if (classifier_resolve(d == i ? nullptr : &calls[i].pool, dense.gemm, soft.row, ctx.n_cus, &j.classifier)) add(j);
        }
        // a dense layer whose result only the layer norm behind it reads, as what is normalised: split already, or to be split for that
        if (!(alone(i, CALL_B3) || alone(i, CALL_GEMM)) || !alone(i + 1, CALL_ROWWISE)) continue;
        const KernelCall &c = calls[i], &n = calls[i + 1];
        const bool b3 = c.kind == CALL_B3;
        const Epilogue &e = b3 ? c.b3.epi : c.gemm.epi;
        const int rows = b3 ? c.b3.Nrows : c.gemm.M, len = b3 ? c.b3.Cout : c.gemm.N, ld = b3 ? c.b3.ldy : c.gemm.ldc, flags = epi_fast_flags(e);
        if (b3 ? !c.b3.dense || c.b3.splitk < 2 : c.gemm.rf_tapk != -1 || !c.gemm.rf_ts || c.gemm.rf_ragged || c.gemm.cs_len || c.gemm_swap) continue;
        if (n.a_node != c.out_node || readers[c.out_node] != 1 || g.is_output[c.out_node]) continue;
        if (n.row.mode != 1 || n.row.rows != rows || n.row.len != len || ld != len || !rowwise_sums_shape_ok(n.row)) continue;
        if (flags & ~(EF_BIAS | EF_ADD) || ((flags & EF_BIAS) && (e.bias_inner > 1 || e.bias_c != len))) continue;
        Join j{};
        j.kind = JOIN_NORM;
        j.lowered = !b3;
        if (!b3 && !split_for_norm(ctx, c, &j.split)) continue;
        j.first = (int32_t)i;
        j.n = 2;
        add(j);
    }
}

}  // namespace

size_t plan_num_launches(const Plan &p) {
    size_t n = 0;
    for (size_t i = 0; i < p.calls.size(); ++i) n += p.elided[i] ? 0 : 1;
    for (const Join &j : p.joins) n -= j.kind == JOIN_CLASSIFIER ? (size_t)j.n - 1 : 0;      // (a split layer's join saves its reduction, which counts as none)
    if (p.max_lanes > 1 || p.handed.empty()) return n;
    for (const Region &r : p.regions) {
        size_t in = 0;
        for (int32_t c : r.members) in += p.handed[c] ? 1 : 0;
        if (in >= 2) n -= in - 1;
    }
    return n;
}

// Which kernels read the packed weights of later ones ahead.  A network whose weights fit the memory-side cache (256 MB) finds them there pass
// after pass; a larger one streams them from HBM (BERT-base: 340 MB), and each of its dense layers then takes 1.3 - 3.5 us longer than with its
// weights in that cache.  Layer norms and attention leave most of the chip idle: workgroups of theirs read (64 bytes apart, nothing is
// kept) what later kernels will stream.
//  * How much: a layer norm 16 MB, which make it 1 us longer; more makes it longer than the dense layers gain (BERT-base, 389 rows: 14 MB more in a
//    layer norm 1102 instead of 1077 us).  Attention 2.4 MB per microsecond that it takes itself, and no more than 61 KB per read-ahead workgroup of its
//    launch (17.7 MB in 8 us: on 36 workgroups, 288 rows, 853 us, with 3.5 MB instead 873; on 19, 304 rows, 948 and 879).  It takes 4 us, and the
//    products of a workgroup at 310 GFLOP per second (heads of 64, measured alone and by this: 128 keys 4.8 and 5.7 us, 256 6.6 and 7.4, 389 13.7 and
//    14.3, 512 15.4 and 17.5).
//  * Where: attention with room for all that lies before the kernel after next that could read ahead takes all of it (389 rows: 1077 us, with
//    a share in the layer norm 1099, without any 1123); otherwise the nearest one before that has room (256 rows: 795, attention first 820, without 864).
//  * From 96 rows on: below, everything takes a few microseconds and reading ahead prolongs what it hides in (us without and with, all of BERT-base: 16 rows 435
//    and 436 - 459, 64 rows 509 and 506 - 528, 128 rows 649 and 623).
//  * The figures are BERT-base's.  Encoders of 28 layers of 8 heads, 16 of 10 and 8 of 16 (heads of 64), at ten lengths of 96 - 512 rows each, were
//    0.994 - 1.065 times as fast as without reading ahead, 1.024 in the mean (16 heads, 50 - 97 MB a layer, the least: 1.01).
static void plan_read_ahead(Plan *plan) {
    constexpr int64_t kMemorySideCache = (int64_t)256 << 20, kWorthIt = 1 << 20;
    constexpr int kRows = 96, kReach = 8;
    const size_t nc = plan->calls.size();
    int64_t total = 0;
    for (const KernelCall &c : plan->calls) total += (int64_t)c.pack_bytes;
    plan->ahead.clear();
    if (total <= kMemorySideCache) return;
    plan->ahead.assign(nc, {});
    std::vector<int64_t> room(nc, 0);
    for (size_t i = 0; i < nc; ++i) {
        const KernelCall &c = plan->calls[i];
        if (c.kind == CALL_ATTENTION && c.att.Sq >= kRows) {
            const AttentionGrid grid = attention_grid(c.att);
            room[i] = (int64_t)(std::min(2.4e6, 61e3 * grid.spare) * (4.0 + 4.0 * grid.rows * c.att.Sk * c.att.d / 310e3));
        }
        if (c.kind == CALL_ROWWISE && c.row.rows >= kRows && rowwise_reads_ahead(c.row)) room[i] = 16000000;
    }
    std::vector<char> placed(nc, 0);
    auto place = [&](size_t i, size_t j) {
        room[i] -= (int64_t)plan->calls[j].pack_bytes;
        plan->ahead[i].push_back((int32_t)j);
        placed[j] = 1;
    };
    for (size_t i = 0; i < nc; ++i) {
        if (plan->calls[i].kind != CALL_ATTENTION || !room[i]) continue;
        int64_t sum = 0;
        std::vector<size_t> all;
        for (size_t j = i + 1, hosts = 0; j < nc && j <= i + kReach && hosts < 2; ++j) {
            if (room[j]) ++hosts;
            if ((int64_t)plan->calls[j].pack_bytes < kWorthIt) continue;
            sum += (int64_t)plan->calls[j].pack_bytes;
            all.push_back(j);
        }
        if (sum <= room[i] && all.size() <= (size_t)kMaxAhead)
            for (size_t j : all) place(i, j);
    }
    for (size_t j = 0; j < nc; ++j) {
        if (placed[j] || (int64_t)plan->calls[j].pack_bytes < kWorthIt) continue;
        for (size_t i = j; i-- > 0 && j - i <= kReach;)
            if (room[i] >= (int64_t)plan->calls[j].pack_bytes && plan->ahead[i].size() < (size_t)kMaxAhead) {
                place(i, j);
                break;
            }
    }
}

// The kernel calls of a placement, in the order of their sinks.
static int32_t lower_placement(Context &ctx, Graph &g, const int32_t *ids, size_t n, Plan *plan) {
    g.finalize();
    if (!g.matched) return fail(CLG_INVALID_ARG, "clg_match_all has not been called on this graph");
    const int n_nodes = (int)g.nodes.size();
    std::vector<int32_t> owner(n_nodes, -1);
    for (size_t i = 0; i < n; ++i) {
        if (ids[i] < 0 || ids[i] >= (int32_t)g.matches.size())
            return fail(CLG_UNKNOWN_ID, "match id %d (the graph has %zu matches)", ids[i], g.matches.size());
        for (int32_t v : g.matches[ids[i]].nodes) {
            if (owner[v] >= 0)
                return fail(CLG_OVERLAP, "matches %d and %d both contain node %d", owner[v], ids[i], v);
            owner[v] = ids[i];
        }
    }
    for (int32_t v : g.op_ids)
        if (owner[v] < 0) return fail(CLG_NOT_A_COVER, "operator node %d (%s) is not covered", v, op_name(g.nodes[v].kind));

    // a group reads other groups only through their sinks, so ordering groups
    // by the position of their sink is a topological order of the quotient graph
    std::vector<int32_t> seq(ids, ids + n);
    std::sort(seq.begin(), seq.end(), [&](int32_t a, int32_t b) {
        return g.rank[g.matches[a].sink] < g.rank[g.matches[b].sink];
    });

    plan->ctx = &ctx;
    plan->graph = &g;
    plan->calls.clear();
    for (int32_t id : seq) {
        KernelCall c;
        const int32_t rc = lower_match(ctx, g, id, &c);
        if (rc != CLG_OK) return rc;
        plan->calls.push_back(std::move(c));
    }
    return CLG_OK;
}

// Regions and joins of the lowered calls, their order, and where each value lives.
static int32_t arrange_plan(const Context &ctx, const Graph &g, bool mixed_regions, bool joins, Plan *plan) {
    const int n_nodes = (int)g.nodes.size();
    find_regions(ctx, g, mixed_regions, plan);
    find_joins(ctx, g, plan);
    if (!joins) {
        plan->joins.clear();
        plan->join_of.assign(plan->calls.size(), -1);
    }

    // every operand must be a leaf or the sink of an earlier group
    const size_t nc = plan->calls.size();
    std::vector<int32_t> produced_at(n_nodes, -1);
    for (size_t i = 0; i < nc; ++i) {
        for (int32_t v : operands_of(plan->calls[i])) {
            if (!g.nodes[v].is_op()) continue;
            if (produced_at[v] < 0)
                return fail(CLG_INVALID_ARG, "kernel %zu reads node %d before any kernel has produced it", i, v);
        }
        produced_at[plan->calls[i].out_node] = (int32_t)i;
    }

    // Concatenation without a copy (Sec. 5.1 hands tensors over by pointer): when the extents before the
    // axis are all 1, every operand is one contiguous piece of the result.  If each operand is produced by a
    // kernel of this plan, has no buffer of its own to go to (not a graph output), is not already part of
    // another concatenation and starts on a 16-byte boundary, its producer writes it straight into its place
    // in the result and the concatenation launches nothing.  Such results nest (root = outermost one).
    plan->value_offset.assign(n_nodes, -1);
    plan->value_output.assign(n_nodes, -1);
    plan->scratch_offset.assign(nc, -1);
    plan->elided.assign(nc, 0);
    std::vector<int32_t> alias_of(n_nodes, -1);
    std::vector<int64_t> alias_delta(n_nodes, 0);
    for (size_t k = 0; k < g.outputs.size(); ++k) plan->value_output[g.outputs[k]] = (int32_t)k;
    for (size_t i = 0; i < nc; ++i) {
        const KernelCall &c = plan->calls[i];
        if (c.kind != CALL_CONCAT || c.cat.outer != 1) continue;
        bool ok = true;
        int64_t off = 0;
        for (int k = 0; k < c.cat.n && ok; ++k) {
            const int32_t v = c.epi_nodes[k];
            ok = g.nodes[v].is_op() && plan->value_output[v] < 0 && alias_of[v] < 0 && off % 16 == 0;
            for (int j = 0; j < k; ++j) ok = ok && c.epi_nodes[j] != v;
            off += 4 * c.cat.chunk[k];
        }
        if (!ok) continue;
        off = 0;
        for (int k = 0; k < c.cat.n; ++k) {
            alias_of[c.epi_nodes[k]] = c.out_node;
            alias_delta[c.epi_nodes[k]] = off;
            off += 4 * c.cat.chunk[k];
        }
        plan->elided[i] = 1;
        plan->calls[i].name += "_alias";
        plan->calls[i].bytes = 0;
    }
    std::vector<int32_t> root(n_nodes);
    std::vector<int64_t> delta(n_nodes, 0);                  // byte offset of a value inside its root's buffer
    for (int v = n_nodes - 1; v >= 0; --v) {                 // a result comes after its operands: roots resolve first
        root[v] = alias_of[v] < 0 ? v : root[alias_of[v]];
        delta[v] = alias_of[v] < 0 ? 0 : delta[alias_of[v]] + alias_delta[v];
    }

    // workspace: one buffer per root value that is not a graph output, reused once the last reader of the
    // root or of any value inside it has run; per-call scratch lives for its call only
    plan->value_delta.assign(n_nodes, 0);
    std::vector<int32_t> release_at(n_nodes, -1);            // root -> call after which its buffer is free
    for (size_t i = 0; i < nc; ++i) {
        const int32_t r = root[plan->calls[i].out_node];
        release_at[r] = std::max(release_at[r], (int32_t)i);
        for (int32_t v : operands_of(plan->calls[i])) release_at[root[v]] = std::max(release_at[root[v]], (int32_t)i);
    }
    std::vector<std::vector<int32_t>> releases(nc);
    for (int v = 0; v < n_nodes; ++v)
        if (root[v] == v && release_at[v] >= 0 && g.nodes[v].is_op() && plan->value_output[v] < 0)
            releases[(size_t)release_at[v]].push_back(v);
    Arena arena;
    auto place_output = [&](size_t i) {
        const int32_t v = plan->calls[i].out_node, r = root[v];
        if (plan->value_output[r] >= 0) {
            if (v != r) {
                plan->value_output[v] = plan->value_output[r];
                plan->value_delta[v] = delta[v];
            }
        } else {
            if (plan->value_offset[r] < 0) plan->value_offset[r] = arena.alloc(4 * g.nodes[r].shape.numel());
            plan->value_offset[v] = plan->value_offset[r] + delta[v];
        }
    };
    // The members of a region may run as one launch: all their results are placed before any of them
    // runs, and what they read is released only after the last of them.  The plan so made holds for
    // every choice of digits (members run one by one use the same buffers in the same order).  So it is with a join,
    // whose last kernel also reads the first one's scratch.
    for (size_t i = 0; i < nc; ++i) {
        const KernelCall &c = plan->calls[i];
        const int32_t ri = plan->region_of[i], ji = plan->join_of[i];
        std::vector<int32_t> only{(int32_t)i};
        if (ji >= 0) {
            only.clear();
            for (int32_t k = 0; k < plan->joins[ji].n; ++k) only.push_back(plan->joins[ji].first + k);
        }
        const std::vector<int32_t> &together = ri >= 0 ? plan->regions[ri].members : only;
        if (together.front() == (int32_t)i)
            for (int32_t m : together) place_output((size_t)m);
        Join *const low = ji >= 0 && plan->joins[ji].lowered ? &plan->joins[ji] : nullptr;
        if (low && low->first == (int32_t)i) low->scratch_offset = arena.alloc((int64_t)low->split.scratch_bytes);
        if (c.scratch_bytes) {
            plan->scratch_offset[i] = arena.alloc((int64_t)c.scratch_bytes);
            if (ji < 0) arena.release(plan->scratch_offset[i]);
        }
        if (together.back() != (int32_t)i) continue;
        if (low) arena.release(low->scratch_offset);
        for (int32_t m : together) {
            if (ji >= 0 && plan->calls[m].scratch_bytes) arena.release(plan->scratch_offset[m]);
            for (int32_t r2 : releases[(size_t)m]) arena.release(plan->value_offset[r2]);
        }
    }
    plan->workspace_bytes = (size_t)arena.peak;
    return CLG_OK;
}

int32_t compile_plan(Context &ctx, Graph &g, const int32_t *ids, size_t n, Plan *plan) {
    int32_t rc = lower_placement(ctx, g, ids, n, plan);
    if (rc != CLG_OK) return rc;
    // Joins keep a little more at a time, and kernels in order of their level a good deal more (NasNet-A, ten 224x224 images: 33.8 MB instead of 30.4): the first
    // arrangement that fits the fixed workspace, so that neither keeps a plan out of it; the first of all where none does.
    const std::vector<KernelCall> lowered = plan->calls;
    constexpr bool kArrangements[][2] = {{true, true}, {true, false}, {false, true}, {false, false}, {true, true}};      // mixed regions, joins
    for (const bool *how : kArrangements) {
        plan->calls = lowered;
        rc = arrange_plan(ctx, g, how[0], how[1], plan);
        if (rc != CLG_OK) return rc;
        if (plan->workspace_bytes <= (size_t)CLG_STATIC_WORKSPACE_BYTES) break;
    }
    schedule_lanes(plan);

    const size_t nc = plan->calls.size();
    // kernels that read their weights in a packed order get a private copy,
    // written once here and owned by the plan
    plan->packed.assign(nc, nullptr);
    if (ctx.device >= 0) {
        bool any = false;
        for (size_t i = 0; i < nc; ++i) {
            const KernelCall &c = plan->calls[i];
            if (!c.pack_bytes) continue;
            const void *w = g.nodes[c.b_node].dev_ptr;
            if (!w) return fail(CLG_INVALID_ARG, "constant node %d has no device pointer", c.b_node);
            if (hipMalloc(&plan->packed[i], c.pack_bytes) != hipSuccess) {
                (void)hipGetLastError();
                plan->packed[i] = nullptr;
                return fail(CLG_OUT_OF_MEMORY, "allocation of %zu bytes for packed weights failed", c.pack_bytes);
            }
            const int32_t rc = pack_weights(c, w, plan->packed[i], nullptr);
            if (rc != CLG_OK) return rc;
            any = true;
        }
        // a region member whose kernel shape differs inside the region reads a second packed copy
        for (Region &r : plan->regions)
            for (size_t k = 0; k < r.members.size(); ++k) {
                const KernelCall &own = plan->calls[(size_t)r.members[k]], &fc = r.fused[k];
                if (fc.kind == own.kind && fc.pack_bytes == own.pack_bytes &&
                    (fc.kind == CALL_B3 ? fc.b3.tile == own.b3.tile : fc.gemm.rf_ts == own.gemm.rf_ts && fc.gemm.rf_wgk == own.gemm.rf_wgk))
                    continue;
                const void *w = g.nodes[fc.b_node].dev_ptr;
                if (hipMalloc(&r.packed[k], fc.pack_bytes) != hipSuccess) {
                    (void)hipGetLastError();
                    r.packed[k] = nullptr;
                    return fail(CLG_OUT_OF_MEMORY, "allocation of %zu bytes for packed weights failed", fc.pack_bytes);
                }
                const int32_t rc = pack_weights(fc, w, r.packed[k], nullptr);
                if (rc != CLG_OK) return rc;
                any = true;
            }
        // (nor does a join's call always read the packed copy that its kernel has alone)
        for (Join &j : plan->joins) {
            const KernelCall &own = plan->calls[(size_t)j.first], &c = j.split;
            if (!j.lowered || (own.gemm.rf_ts == c.gemm.rf_ts && own.gemm.rf_ngtot == c.gemm.rf_ngtot && own.pack_bytes >= c.pack_bytes)) continue;
            if (hipMalloc(&j.packed, c.pack_bytes) != hipSuccess) {
                (void)hipGetLastError();
                j.packed = nullptr;
                return fail(CLG_OUT_OF_MEMORY, "allocation of %zu bytes for packed weights failed", c.pack_bytes);
            }
            const int32_t rc = pack_weights(c, g.nodes[c.b_node].dev_ptr, j.packed, nullptr);
            if (rc != CLG_OK) return rc;
            any = true;
        }
        if (any && hipStreamSynchronize(nullptr) != hipSuccess)
            return fail(CLG_HIP_ERROR, "weight packing failed: %s", hipGetErrorString(hipGetLastError()));
    }
    plan_read_ahead(plan);
    plan->missing_const = -1;
    for (const KernelCall &c : plan->calls)
        for (int32_t v : operands_of(c))
            if (g.nodes[v].kind == NODE_CONST && !g.nodes[v].dev_ptr) plan->missing_const = v;
    return CLG_OK;
}

Plan::~Plan() {
    if (counted && graph) --graph->live_plans;
    for (void *p : packed)
        if (p) (void)hipFree(p);
    for (Region &r : regions)
        for (void *p : r.packed)
            if (p) (void)hipFree(p);
    for (Join &j : joins)
        if (j.packed) (void)hipFree(j.packed);
    for (void *e : events)
        if (e) (void)hipEventDestroy((hipEvent_t)e);
    for (void *e : ev_end)
        if (e) (void)hipEventDestroy((hipEvent_t)e);
    if (ev_begin) (void)hipEventDestroy((hipEvent_t)ev_begin);
    for (void *s : side_streams)
        if (s) (void)hipStreamDestroy((hipStream_t)s);
}

int32_t set_plan_lanes(Plan &p, int32_t lanes) {
    for (void *s : p.side_streams)
        if (s && hipStreamSynchronize((hipStream_t)s) != hipSuccess)
            return fail(CLG_HIP_ERROR, "synchronising a lane failed: %s", hipGetErrorString(hipGetLastError()));
    for (void *e : p.events)
        if (e) (void)hipEventDestroy((hipEvent_t)e);
    for (void *e : p.ev_end)
        if (e) (void)hipEventDestroy((hipEvent_t)e);
    if (p.ev_begin) (void)hipEventDestroy((hipEvent_t)p.ev_begin);
    for (void *s : p.side_streams)
        if (s) (void)hipStreamDestroy((hipStream_t)s);
    p.events.clear();
    p.ev_end.clear();
    p.ev_begin = nullptr;
    p.side_streams.clear();
    p.max_lanes = lanes;
    schedule_lanes(&p);
    return CLG_OK;
}

// Lane schedule.  A placement's quotient graph has independent branches (the
// projection shortcut next to the main path of a residual block; the query, key
// and value projections of an attention layer), and at batch 1 one kernel rarely
// fills the chip, so such branches run on different HIP streams.  Dependencies
// are the data dependencies between kernels plus every reuse of a workspace
// region (the workspace was planned for the sequential order).  Kernels are
// still enqueued in plan order; a kernel stays on the lane of its latest
// dependency when everything queued there is among its (transitive)
// dependencies, and otherwise moves to another lane, waiting on events for what
// it needs from elsewhere.
void schedule_lanes(Plan *plan) {
    const Graph &g = *plan->graph;
    const size_t nc = plan->calls.size();
    plan->lane.assign(nc, 0);
    plan->waits.assign(nc, {});
    plan->signals.assign(nc, 0);
    plan->n_lanes = 1;
    if (plan->max_lanes <= 1 || nc < 3) return;

    struct Region { int64_t lo, hi; };
    auto overlap = [](const std::vector<Region> &a, const std::vector<Region> &b) {
        for (const Region &x : a)
            for (const Region &y : b)
                if (x.lo < y.hi && y.lo < x.hi) return true;
        return false;
    };
    std::vector<std::vector<Region>> rd(nc), wr(nc);
    std::vector<int32_t> produced_at(g.nodes.size(), -1);
    for (size_t i = 0; i < nc; ++i) {
        const KernelCall &c = plan->calls[i];
        for (int32_t v : operands_of(c))
            if (plan->value_offset[v] >= 0)
                rd[i].push_back({plan->value_offset[v], plan->value_offset[v] + round_up(4 * g.nodes[v].shape.numel())});
        if (plan->value_offset[c.out_node] >= 0)
            wr[i].push_back({plan->value_offset[c.out_node],
                             plan->value_offset[c.out_node] + round_up(4 * g.nodes[c.out_node].shape.numel())});
        if (plan->scratch_offset[i] >= 0)
            wr[i].push_back({plan->scratch_offset[i], plan->scratch_offset[i] + round_up((int64_t)c.scratch_bytes)});
        if (plan->join_of[i] >= 0 && plan->joins[(size_t)plan->join_of[i]].lowered) {
            const Join &j = plan->joins[(size_t)plan->join_of[i]];
            wr[i].push_back({j.scratch_offset, j.scratch_offset + round_up((int64_t)j.split.scratch_bytes)});
        }
        produced_at[c.out_node] = (int32_t)i;
    }
    // direct dependencies and their transitive closure (bit sets over calls)
    const size_t words = (nc + 63) / 64;
    std::vector<std::vector<int32_t>> deps(nc);
    std::vector<std::vector<uint64_t>> reach(nc, std::vector<uint64_t>(words, 0));
    for (size_t j = 0; j < nc; ++j) {
        for (int32_t v : operands_of(plan->calls[j])) {
            const int32_t i = g.nodes[v].is_op() ? produced_at[v] : -1;
            if (i >= 0 && (size_t)i < j) deps[j].push_back(i);
        }
        for (size_t i = 0; i < j; ++i)
            if (overlap(wr[j], rd[i]) || overlap(wr[j], wr[i]) || overlap(rd[j], wr[i])) deps[j].push_back((int32_t)i);
        std::sort(deps[j].begin(), deps[j].end());
        deps[j].erase(std::unique(deps[j].begin(), deps[j].end()), deps[j].end());
        for (int32_t i : deps[j]) {
            reach[j][(size_t)i / 64] |= (uint64_t)1 << (i % 64);
            for (size_t w = 0; w < words; ++w) reach[j][w] |= reach[i][w];
        }
    }
    auto depends = [&](size_t j, int32_t i) { return i < 0 || ((reach[j][(size_t)i / 64] >> (i % 64)) & 1) != 0; };

    const int lanes = std::min<int>(plan->max_lanes, 4);
    std::vector<int32_t> last(lanes, -1);            // last call queued on each lane
    for (size_t j = 0; j < nc; ++j) {
        int pick = (!plan->handed.empty() && !plan->handed[j]) ? 0 : -1;   // not handed over: the caller's stream
        if (plan->join_of[j] >= 0) {                       // a join runs on one lane, the caller's stream if any of its kernels has to
            const Join &jn = plan->joins[(size_t)plan->join_of[j]];
            if (jn.first < (int32_t)j) pick = plan->lane[(size_t)jn.first];
            else
                for (int32_t k = 0; k < jn.n && !plan->handed.empty(); ++k)
                    if (!plan->handed[j + (size_t)k]) pick = 0;
        }
        const int home = deps[j].empty() ? 0 : plan->lane[deps[j].back()];
        if (pick < 0 && depends(j, last[home])) pick = home;
        for (int l = 0; l < lanes && pick < 0; ++l)
            if (depends(j, last[l])) pick = l;         // a lane whose queue this call follows anyway (or an idle one)
        if (pick < 0) {                                // every lane holds unrelated work: join the least recently used
            pick = 0;
            for (int l = 1; l < lanes; ++l)
                if (last[l] < last[pick]) pick = l;
        }
        plan->lane[j] = pick;
        last[pick] = (int32_t)j;
        plan->n_lanes = std::max(plan->n_lanes, pick + 1);
        // wait for the latest direct dependency on every other lane (a lane runs in order)
        std::vector<int32_t> latest(lanes, -1);
        for (int32_t i : deps[j])
            if (plan->lane[i] != pick) latest[plan->lane[i]] = std::max(latest[plan->lane[i]], i);
        for (int l = 0; l < lanes; ++l)
            if (latest[l] >= 0) {
                plan->waits[j].push_back(latest[l]);
                plan->signals[latest[l]] = 1;
            }
    }
}

int32_t measure_plan(Plan &p, const void *const *inputs, void *const *outputs, void *workspace, size_t ws_bytes,
                     void *stream, const clg_measure_opts &o, int64_t *ns) {
    if (p.ctx->device < 0) return fail(CLG_HIP_ERROR, "host-only context: no device to execute on");
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) {
        if (e0) (void)hipEventDestroy(e0);
        return fail(CLG_HIP_ERROR, "hipEventCreate failed");
    }
    int32_t rc = CLG_OK;
    double best = -1;
    for (int32_t i = 0; i < o.warmup && rc == CLG_OK; ++i)
        rc = execute_plan(p, inputs, outputs, workspace, ws_bytes, stream, nullptr);
    for (int32_t b = 0; b < o.batches && rc == CLG_OK; ++b) {
        (void)hipEventRecord(e0, (hipStream_t)stream);
        for (int32_t i = 0; i < o.reps && rc == CLG_OK; ++i)
            rc = execute_plan(p, inputs, outputs, workspace, ws_bytes, stream, nullptr);
        (void)hipEventRecord(e1, (hipStream_t)stream);
        if (hipEventSynchronize(e1) != hipSuccess && rc == CLG_OK)
            rc = fail(CLG_HIP_ERROR, "waiting for a timed batch failed: %s", hipGetErrorString(hipGetLastError()));
        float ms = 0.f;
        if (rc == CLG_OK && hipEventElapsedTime(&ms, e0, e1) != hipSuccess) rc = fail(CLG_HIP_ERROR, "hipEventElapsedTime failed");
        const double per = (double)ms * 1.0e6 / o.reps;
        if (best < 0 || per < best) best = per;
    }
    if (rc != CLG_OK) (void)hipStreamSynchronize((hipStream_t)stream);
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc == CLG_OK) *ns = (int64_t)(best + 0.5);
    return rc;
}

int32_t pack_weights(const KernelCall &c, const void *w, void *dst, void *stream) {
    const int err = c.kind == CALL_SEPCONV ? launch_sepconv_pack(c.sep, (const float *)w, (float *)dst, stream)
                    : c.kind == CALL_B3    ? launch_b3_pack(c.b3, (const float *)w, dst, stream)
                                           : launch_rf_pack(c.gemm, (const float *)w, (float *)dst, stream);
    if (err != 0) return fail(CLG_HIP_ERROR, "weight packing launch failed: %s", hipGetErrorString((hipError_t)err));
    return CLG_OK;
}

int32_t bind_gemm(const KernelCall &c, const void *a, const void *b, void *out, const void *const *epi_ptrs,
                  void *scratch, const void *packed, GemmArgs *kp) {
    GemmArgs &k = *kp;
    k = c.gemm;
    k.A = (const float *)a; k.B = (const float *)b; k.C = (float *)out;
    if (c.gemm_swap) {                               // A = weights, B = activations
        k.A = (const float *)b; k.B = (const float *)a;
    }
    if (c.pack_bytes) {
        if (!packed) return fail(CLG_INVALID_ARG, "%s needs packed weights, none were prepared", c.name.c_str());
        if (c.gemm.rf_tapk == -1) k.B = (const float *)packed;      // dense: the weights are the second operand
        else k.A = (const float *)packed;
    }
    k.partial = (float *)scratch;
    for (int s = 0; s < k.epi.n; ++s) k.epi.s[s].ptr = (const float *)epi_ptrs[s];
    return CLG_OK;
}

// One member of a mixed region with its pointers bound.
static int32_t bind_mix(const KernelCall &c, const void *a, const void *b, const void *c3, void *out, const void *const *epi_ptrs, const void *packed,
                        MixMember *m, int32_t *kind) {
    auto bind = [&](Epilogue &e) {
        for (int s = 0; s < e.n; ++s) e.s[s].ptr = (const float *)epi_ptrs[s];
    };
    if (c.pack_bytes && !packed) return fail(CLG_INVALID_ARG, "%s needs packed weights, none were prepared", c.name.c_str());
    if (c.kind == CALL_SEPCONV) {
        m->sep = c.sep;
        m->sep.x = (const float *)a; m->sep.wp = (const float *)packed; m->sep.wd = (const float *)c3; m->sep.y = (float *)out;
        bind(m->sep.epi);
        *kind = mix_sep_kind(c.sep);
    } else if (c.kind == CALL_DIRECT_CONV) {
        m->dw = c.dconv;
        m->dw.x = (const float *)a; m->dw.w = (const float *)b; m->dw.y = (float *)out;
        bind(m->dw.epi);
        *kind = c.dconv.KH;
    } else if (c.kind == CALL_POOL) {
        m->pool = c.pool;
        m->pool.x = (const float *)a; m->pool.y = (float *)out;
        bind(m->pool.epi);
        *kind = c.pool.mode == 0 ? MIX_MAX : MIX_AVG;
    } else {
        GemmArgs k;
        const int32_t rc = bind_gemm(c, a, b, out, epi_ptrs, nullptr, packed, &k);
        if (rc != CLG_OK) return rc;
        k.ef = make_epi_fast(k.epi);
        m->conv = k;
        *kind = mix_conv_kind(k);
    }
    return CLG_OK;
}

int32_t launch_call(const KernelCall &c, const void *a, const void *b, const void *c3, void *out,
                    const void *const *epi_ptrs, void *scratch, const void *packed, void *stream, const Ahead *ahead) {
    auto bind = [&](Epilogue e) {
        for (int s = 0; s < e.n; ++s) e.s[s].ptr = (const float *)epi_ptrs[s];
        return e;
    };
    int err = 0;
    switch (c.kind) {
    case CALL_GEMM: {
        GemmArgs k;
        const int32_t rc = bind_gemm(c, a, b, out, epi_ptrs, scratch, packed, &k);
        if (rc != CLG_OK) return rc;
        err = launch_gemm(k, stream);
        break;
    }
    case CALL_B3: {
        if (!packed) return fail(CLG_INVALID_ARG, "%s needs packed weights, none were prepared", c.name.c_str());
        B3Args k = c.b3;
        k.x = (const float *)a; k.w = packed; k.y = (float *)out; k.partial = (float *)scratch;
        k.epi = bind(c.b3.epi);
        err = launch_b3(k, stream);
        break;
    }
    case CALL_DIRECT_CONV: {
        DirectConvArgs k = c.dconv;
        k.x = (const float *)a; k.w = (const float *)b; k.y = (float *)out;
        k.epi = bind(c.dconv.epi);
        err = launch_direct_conv(k, stream);
        break;
    }
    case CALL_POOL: {
        PoolArgs k = c.pool;
        k.x = (const float *)a; k.y = (float *)out;
        k.epi = bind(c.pool.epi);
        err = launch_pool(k, stream);
        break;
    }
    case CALL_ROWWISE: {
        RowwiseArgs k = c.row;
        k.x = (const float *)a; k.gamma = (const float *)b; k.beta = (const float *)c3; k.y = (float *)out;
        k.pro = bind(c.row.pro);
        for (int t = 0; t < k.n_gather; ++t) {           // an embedding: tables and id lists ride in the step slots
            k.tab[t] = (const float *)epi_ptrs[t];
            k.gid[t] = (const int32_t *)epi_ptrs[3 + t];
        }
        if (k.n_gather) k.x = nullptr;
        err = launch_rowwise(k, ahead, stream);
        break;
    }
    case CALL_ELTWISE: {
        EltwiseArgs k = c.elt;
        k.x = (const float *)a; k.ids = (const int32_t *)b; k.y = (float *)out;
        k.epi = bind(c.elt.epi);
        err = launch_eltwise(k, stream);
        break;
    }
    case CALL_LAYOUT: {
        LayoutArgs k = c.layout;
        k.x = (const float *)a; k.y = (float *)out;
        err = launch_layout(k, stream);
        break;
    }
    case CALL_SEPCONV: {
        if (!packed) return fail(CLG_INVALID_ARG, "%s needs packed weights, none were prepared", c.name.c_str());
        SepConvArgs k = c.sep;
        k.x = (const float *)a; k.wp = (const float *)packed; k.wd = (const float *)c3; k.y = (float *)out;
        k.epi = bind(c.sep.epi);
        err = launch_sepconv(k, stream);
        break;
    }
    case CALL_ATTENTION: {
        AttentionArgs k = c.att;
        k.q = (const float *)a; k.k = (const float *)b; k.v = (const float *)c3; k.y = (float *)out;
        err = launch_attention(k, ahead, stream);
        break;
    }
    case CALL_CONCAT: {
        ConcatArgs k = c.cat;
        for (int s = 0; s < k.n; ++s) k.src[s] = (const float *)epi_ptrs[s];
        k.y = (float *)out;
        err = launch_concat(k, stream);
        break;
    }
    default:
        return fail(CLG_INVALID_ARG, "unknown call kind %d", c.kind);
    }
    if (err != 0)
        return fail(CLG_HIP_ERROR, "launch of %s failed: %s", c.name.c_str(), hipGetErrorString((hipError_t)err));
    return CLG_OK;
}

// Whether two arrays of floats share memory (a null one shares none).
static bool meet(const float *p, int64_t n, const float *q, int64_t m) {
    return p && q && (uintptr_t)p < (uintptr_t)q + 4 * (uintptr_t)m && (uintptr_t)q < (uintptr_t)p + 4 * (uintptr_t)n;
}

// The launches of a join, operands by `ptr_of`; *done = false: the addresses are such that they run one by one (a caller's output buffer may lie over an
// input, or over another output, which kernels that run one after the other take as long as each reads before a later one writes).
template <class F>
static int32_t launch_join(const Plan &p, const Join &j, const F &ptr_of, void *workspace, const Ahead *ahead, void *stream, bool *done) {
    const size_t first = (size_t)j.first, last = first + (size_t)j.n - 1;
    auto in = [&](int32_t v) { return (const float *)ptr_of(v); };
    auto out = [&](size_t i) { return (float *)const_cast<void *>(ptr_of(p.calls[i].out_node)); };
    auto bind = [&](Epilogue e, const KernelCall &c) {
        for (int s = 0; s < e.n; ++s) e.s[s].ptr = in(c.epi_nodes[s]);
        return e;
    };
    void *scratch = p.scratch_offset[first] >= 0 ? (char *)workspace + p.scratch_offset[first] : nullptr;
    int err;
    *done = true;
    if (j.kind == JOIN_CLASSIFIER) {
        const size_t d = last - 1;
        const KernelCall &c = p.calls[d];
        ClassifierArgs a = j.classifier;
        if (c.pack_bytes && !p.packed[d]) return fail(CLG_INVALID_ARG, "%s needs packed weights, none were prepared", c.name.c_str());
        a.x = in(p.calls[first].a_node);
        a.pooled = d > first ? out(first) : nullptr;
        a.w = c.pack_bytes ? (const float *)p.packed[d] : in(c.b_node);
        a.logits = out(d);
        a.prob = out(last);
        a.ef = make_epi_fast(bind(c.gemm.epi, c));
        // (rows are read, weights and bias included, while results of others are written)
        const int64_t rows = a.rows;
        const struct { const float *p; int64_t n; } outs[] = {{a.pooled, rows * a.lda}, {a.logits, rows * a.N}, {a.prob, rows * a.N}},
            ins[] = {{a.x, rows * (a.hw ? (int64_t)a.K * a.hw : a.lda)}, {c.pack_bytes ? nullptr : a.w, (int64_t)a.N * a.ldb}, {a.ef.flags & EF_BIAS ? a.ef.bias : nullptr, a.N}};
        for (const auto &o : outs) {
            for (const auto &i : ins)
                if (meet(o.p, o.n, i.p, i.n)) *done = false;
            for (const auto &o2 : outs)
                if (&o2 != &o && meet(o.p, o.n, o2.p, o2.n)) *done = false;
        }
        if (!*done) return CLG_OK;
        err = launch_classifier(a, stream);
    } else {
        const KernelCall &c = j.lowered ? j.split : p.calls[first], &n = p.calls[last];
        const void *w = j.packed ? j.packed : p.packed[first];
        if (!w) return fail(CLG_INVALID_ARG, "%s needs packed weights, none were prepared", c.name.c_str());
        if (j.lowered) scratch = (char *)workspace + j.scratch_offset;
        const bool b3 = c.kind == CALL_B3;
        const EpiFast ef = make_epi_fast(bind(b3 ? c.b3.epi : c.gemm.epi, c));
        RowwiseArgs r = n.row;
        r.gamma = in(n.b_node); r.beta = in(n.c_node); r.y = out(last);
        r.pro = bind(n.row.pro, n);
        const SplitSum sum{(const float *)scratch, ef.flags & EF_BIAS ? ef.bias : nullptr, ef.flags & EF_ADD ? ef.add : nullptr, b3 ? c.b3.splitk : c.gemm.splitk,
                           (int32_t)(b3 ? c.b3.c_numel : c.gemm.c_numel)};
        // (a wave reads its row of the residual before it writes the same row; bias and other rows are read while it does)
        const int64_t numel = (int64_t)r.rows * r.len;
        if (!rowwise_sums_ok(r, sum) || meet(r.y, numel, sum.bias, r.len) || (r.y != sum.add && meet(r.y, numel, sum.add, numel))) {
            *done = false;
            return CLG_OK;
        }
        if (b3) {
            B3Args k = c.b3;
            k.x = in(c.a_node); k.w = w; k.y = out(first); k.partial = (float *)scratch;
            k.epi = bind(c.b3.epi, c);
            err = launch_b3(k, stream, false);
        } else {
            const void *epi[kMaxEpi];
            for (int s = 0; s < kMaxEpi; ++s) epi[s] = c.epi_nodes[s] >= 0 ? ptr_of(c.epi_nodes[s]) : nullptr;
            GemmArgs k;
            const int32_t rc = bind_gemm(c, in(c.a_node), in(c.b_node), out(first), epi, scratch, w, &k);
            if (rc != CLG_OK) return rc;
            err = launch_gemm(k, stream, false);
        }
        if (!err) err = launch_rowwise_sum(r, sum, ahead, stream);
    }
    if (err != 0) return fail(CLG_HIP_ERROR, "launch of %s and what follows it failed: %s", p.calls[first].name.c_str(), hipGetErrorString((hipError_t)err));
    return CLG_OK;
}

int32_t execute_plan(Plan &p, const void *const *inputs, void *const *outputs, void *workspace,
                     size_t ws_bytes, void *stream, int64_t *kernel_ns) {
    Context &ctx = *p.ctx;
    Graph &g = *p.graph;
    if (ctx.device < 0) return fail(CLG_HIP_ERROR, "host-only context: no device to execute on");
    if (ws_bytes < p.workspace_bytes)
        return fail(CLG_WORKSPACE_TOO_SMALL, "workspace has %zu bytes, the plan needs %zu", ws_bytes, p.workspace_bytes);
    if (p.workspace_bytes && !workspace) return fail(CLG_INVALID_ARG, "workspace is null");
    if (((uintptr_t)workspace & 255) != 0) return fail(CLG_INVALID_ARG, "workspace is not 256-byte aligned");
    if ((g.n_inputs && !inputs) || (!g.outputs.empty() && !outputs)) return fail(CLG_INVALID_ARG, "inputs/outputs is null");
    for (int i = 0; i < g.n_inputs; ++i)
        if (!inputs[i]) return fail(CLG_INVALID_ARG, "input %d is null", i);
    for (size_t i = 0; i < g.outputs.size(); ++i)
        if (!outputs[i]) return fail(CLG_INVALID_ARG, "output %zu is null", i);
    if (p.missing_const >= 0) return fail(CLG_INVALID_ARG, "constant node %d has no device pointer", p.missing_const);

    auto ptr_of = [&](int32_t v) -> const void * {
        if (v < 0) return nullptr;
        const Node &nd = g.nodes[v];
        if (nd.kind == NODE_CONST) return nd.dev_ptr;
        if (nd.kind == NODE_INPUT) return inputs[nd.input_index];
        if (p.value_output[v] >= 0) return (const char *)outputs[p.value_output[v]] + p.value_delta[v];
        return (const char *)workspace + p.value_offset[v];
    };
    std::vector<hipEvent_t> ev;
    if (kernel_ns) {
        ev.resize(2 * p.calls.size());
        for (auto &e : ev)
            if (hipEventCreate(&e) != hipSuccess) return fail(CLG_HIP_ERROR, "hipEventCreate failed");
    }
    // lanes: per-kernel timing runs everything on the caller's stream
    const bool lanes = !kernel_ns && p.n_lanes > 1;
    hipError_t he = hipSuccess;
    if (lanes) {
        if (p.side_streams.empty()) {                  // first execution: the plan's own streams and events
            p.side_streams.assign((size_t)p.n_lanes - 1, nullptr);
            p.ev_end.assign((size_t)p.n_lanes - 1, nullptr);
            p.events.assign(p.calls.size(), nullptr);
            for (auto &s : p.side_streams)
                if (he == hipSuccess) he = hipStreamCreateWithFlags((hipStream_t *)&s, hipStreamNonBlocking);
            for (auto &e : p.ev_end)
                if (he == hipSuccess) he = hipEventCreateWithFlags((hipEvent_t *)&e, hipEventDisableTiming);
            if (he == hipSuccess) he = hipEventCreateWithFlags((hipEvent_t *)&p.ev_begin, hipEventDisableTiming);
            for (size_t i = 0; i < p.calls.size(); ++i)
                if (p.signals[i] && he == hipSuccess)
                    he = hipEventCreateWithFlags((hipEvent_t *)&p.events[i], hipEventDisableTiming);
            if (he != hipSuccess) {
                p.n_lanes = 1;                         // the partly built set is released with the plan
                return fail(CLG_HIP_ERROR, "creating the plan's streams and events failed: %s", hipGetErrorString(he));
            }
        }
        // the side lanes start after everything already queued on the caller's stream
        he = hipEventRecord((hipEvent_t)p.ev_begin, (hipStream_t)stream);
        for (void *s : p.side_streams)
            if (he == hipSuccess) he = hipStreamWaitEvent((hipStream_t)s, (hipEvent_t)p.ev_begin, 0);
        if (he != hipSuccess) return fail(CLG_HIP_ERROR, "lane fork failed: %s", hipGetErrorString(he));
    }
    auto stream_of = [&](size_t i) -> void * {
        return (lanes && p.lane[i] > 0) ? p.side_streams[(size_t)p.lane[i] - 1] : stream;
    };
    const bool fuse = p.max_lanes <= 1 && !p.handed.empty() && !p.regions.empty();
    Ahead ahead;
    auto in_region = [&](size_t j) {                   // launched with a sibling: reads the region's copy of the weights
        if (!fuse || p.region_of[j] < 0 || !p.handed[j]) return false;
        int n = 0;
        for (int32_t m : p.regions[(size_t)p.region_of[j]].members) n += p.handed[(size_t)m] ? 1 : 0;
        return n >= 2;
    };
    auto ahead_of = [&](size_t i, Ahead *out) -> const Ahead * {
        if (p.ahead.empty() || p.ahead[i].empty()) return nullptr;
        out->n = 0;
        for (int32_t j : p.ahead[i]) {
            const void *w = p.packed[(size_t)j];
            size_t bytes = p.calls[(size_t)j].pack_bytes;
            if (in_region((size_t)j)) {
                const Region &r = p.regions[(size_t)p.region_of[(size_t)j]];
                for (size_t k = 0; k < r.members.size(); ++k)
                    if (r.members[k] == j && r.packed[k]) {
                        w = r.packed[k];
                        bytes = r.fused[k].pack_bytes;
                    }
            }
            if (p.join_of[(size_t)j] >= 0 && p.joins[(size_t)p.join_of[(size_t)j]].packed) {
                const Join &jn = p.joins[(size_t)p.join_of[(size_t)j]];
                w = jn.packed;
                bytes = jn.split.pack_bytes;
            }
            out->p[out->n] = w;
            out->lines[out->n++] = (uint32_t)(bytes / kAheadLine);
        }
        return out;
    };
    int32_t rc = CLG_OK;
    // regions: with one lane, the handed-over members of a region (two or more) go out as one launch
    std::vector<char> &done = p.fuse_mark;             // sized at compile time: nothing is allocated here
    if (fuse) std::fill(done.begin(), done.end(), 0);
    for (size_t i = 0; i < p.calls.size() && rc == CLG_OK; ++i) {
        const KernelCall &c = p.calls[i];
        if (fuse && done[i]) continue;
        if (!kernel_ns && p.join_of[i] >= 0 && p.joins[(size_t)p.join_of[i]].first == (int32_t)i) {
            const Join &j = p.joins[(size_t)p.join_of[i]];
            const size_t end = i + (size_t)j.n;
            void *st = stream_of(i);
            if (lanes)
                for (size_t k = i; k < end; ++k)
                    for (int32_t w : p.waits[k])             // (no kernel of the join is on another lane)
                        if (hipStreamWaitEvent((hipStream_t)st, (hipEvent_t)p.events[w], 0) != hipSuccess)
                            rc = fail(CLG_HIP_ERROR, "hipStreamWaitEvent failed");
            if (rc != CLG_OK) break;
            bool joined = false;
            rc = launch_join(p, j, ptr_of, workspace, ahead_of(end - 1, &ahead), st, &joined);
            if (rc != CLG_OK) break;
            if (joined) {
                for (size_t k = i; k < end; ++k)
                    if (lanes && p.signals[k] && hipEventRecord((hipEvent_t)p.events[k], (hipStream_t)st) != hipSuccess)
                        rc = fail(CLG_HIP_ERROR, "hipEventRecord failed");
                i = end - 1;
                continue;
            }
        }
        if (fuse && p.region_of[i] >= 0 && p.handed[i]) {
            const Region &r = p.regions[(size_t)p.region_of[i]];
            const bool sep = !r.mixed && c.kind == CALL_SEPCONV;
            const bool b3 = r.fused[0].kind == CALL_B3;
            const bool plane = !r.mixed && r.fused[0].kind != CALL_GEMM && !sep && !b3;   // a region of thread-per-output kernels
            GemmArgs members[kMaxRegion];
            B3Args bmembers[kMaxB3Region];
            SepConvArgs smembers[kMaxSepRegion];
            PlaneMultiArgs &pm = p.plane_args;           // (part of the plan: nothing this large goes on the stack per call)
            MixArgs &mm = p.mix_args;
            static_assert(kMaxMixRegion <= kMaxPlaneRegion && kMaxRegion <= kMaxPlaneRegion, "idx holds any region's members");
            size_t idx[kMaxPlaneRegion];
            int nm = 0;
            for (size_t o = 0; o < r.members.size(); ++o) {
                const size_t k = (size_t)r.order[o], ci = (size_t)r.members[k];
                if (ci < i || !p.handed[ci]) continue;
                const KernelCall &fc = r.fused[k];
                const void *fepi[kMaxEpi];
                for (int s = 0; s < kMaxEpi; ++s) fepi[s] = ptr_of(fc.epi_nodes[s]);
                if (r.mixed) {
                    rc = bind_mix(fc, ptr_of(fc.a_node), ptr_of(fc.b_node), ptr_of(fc.c_node), const_cast<void *>(ptr_of(fc.out_node)), fepi,
                                  r.packed[k] ? r.packed[k] : p.packed[ci], &mm.p[nm], &mm.kind[nm]);
                } else if (sep) {
                    if (!p.packed[ci]) rc = fail(CLG_INVALID_ARG, "%s needs packed weights, none were prepared", fc.name.c_str());
                    SepConvArgs &k2 = smembers[nm];
                    k2 = fc.sep;
                    k2.x = (const float *)ptr_of(fc.a_node); k2.wp = (const float *)p.packed[ci];
                    k2.wd = (const float *)ptr_of(fc.c_node);
                    k2.y = (float *)const_cast<void *>(ptr_of(fc.out_node));
                    for (int s = 0; s < k2.epi.n; ++s) k2.epi.s[s].ptr = (const float *)fepi[s];
                } else if (plane) {
                    if (fc.kind == CALL_DIRECT_CONV) {
                        DirectConvArgs &k2 = pm.p[nm].dw;
                        k2 = fc.dconv;
                        k2.x = (const float *)ptr_of(fc.a_node); k2.w = (const float *)ptr_of(fc.b_node);
                        k2.y = (float *)const_cast<void *>(ptr_of(fc.out_node));
                        for (int s = 0; s < k2.epi.n; ++s) k2.epi.s[s].ptr = (const float *)fepi[s];
                        pm.kind[nm] = k2.KH;
                    } else {
                        PoolArgs &k2 = pm.p[nm].pool;
                        k2 = fc.pool;
                        k2.x = (const float *)ptr_of(fc.a_node);
                        k2.y = (float *)const_cast<void *>(ptr_of(fc.out_node));
                        for (int s = 0; s < k2.epi.n; ++s) k2.epi.s[s].ptr = (const float *)fepi[s];
                        pm.kind[nm] = k2.mode == 0 ? 10 : 11;
                    }
                } else if (b3) {
                    const void *pk = r.packed[k] ? r.packed[k] : p.packed[ci];
                    if (!pk) rc = fail(CLG_INVALID_ARG, "%s needs packed weights, none were prepared", fc.name.c_str());
                    B3Args &k2 = bmembers[nm];
                    k2 = fc.b3;
                    k2.x = (const float *)ptr_of(fc.a_node); k2.w = pk;
                    k2.y = (float *)const_cast<void *>(ptr_of(fc.out_node));
                    for (int s = 0; s < k2.epi.n; ++s) k2.epi.s[s].ptr = (const float *)fepi[s];
                } else {
                    const void *pk = r.packed[k] ? r.packed[k] : p.packed[ci];
                    rc = bind_gemm(fc, ptr_of(fc.a_node), ptr_of(fc.b_node), const_cast<void *>(ptr_of(fc.out_node)), fepi,
                                   nullptr, pk, &members[nm]);
                }
                if (rc != CLG_OK) break;
                idx[nm++] = ci;
            }
            if (rc != CLG_OK) break;
            if (nm >= 2) {
                if (kernel_ns) (void)hipEventRecord(ev[2 * i], (hipStream_t)stream);
                pm.n = nm;
                mm.n = nm;
                const int err = r.mixed ? launch_mix_region(mm, stream)
                                : sep ? launch_sepconv_region(smembers, nm, stream)
                                    : (plane ? launch_plane_region(pm, stream)
                                             : (b3 ? launch_b3_region(bmembers, nm, stream) : launch_gemm_region(members, nm, stream)));
                if (kernel_ns) (void)hipEventRecord(ev[2 * i + 1], (hipStream_t)stream);
                if (err != 0) rc = fail(CLG_HIP_ERROR, "launch of the region around %s failed: %s", c.name.c_str(),
                                        hipGetErrorString((hipError_t)err));
                for (int k = 0; k < nm; ++k) done[idx[k]] = 1;
                done[i] = 2;                         // carries the region's time
                continue;
            }
        }
        const void *epi[kMaxEpi];
        for (int s = 0; s < kMaxEpi; ++s) epi[s] = ptr_of(c.epi_nodes[s]);
        void *scratch = p.scratch_offset[i] >= 0 ? (char *)workspace + p.scratch_offset[i] : nullptr;
        void *st = stream_of(i);
        if (lanes)
            for (int32_t w : p.waits[i])
                if (hipStreamWaitEvent((hipStream_t)st, (hipEvent_t)p.events[w], 0) != hipSuccess)
                    rc = fail(CLG_HIP_ERROR, "hipStreamWaitEvent failed");
        if (rc != CLG_OK) break;
        if (kernel_ns && !p.elided[i]) (void)hipEventRecord(ev[2 * i], (hipStream_t)stream);
        if (!p.elided[i])                                // an aliased concatenation: its operands are already in place
            rc = launch_call(c, ptr_of(c.a_node), ptr_of(c.b_node), ptr_of(c.c_node),
                             const_cast<void *>(ptr_of(c.out_node)), epi, scratch, p.packed[i], st, ahead_of(i, &ahead));
        if (kernel_ns && !p.elided[i]) (void)hipEventRecord(ev[2 * i + 1], (hipStream_t)stream);
        if (lanes && p.signals[i] && rc == CLG_OK && hipEventRecord((hipEvent_t)p.events[i], (hipStream_t)st) != hipSuccess)
            rc = fail(CLG_HIP_ERROR, "hipEventRecord failed");
    }
    if (lanes) {
        // join: the caller's stream continues after every side lane (also after a failed launch, so that
        // nothing the plan queued is left running behind the caller's back)
        for (size_t l = 0; l < p.side_streams.size(); ++l) {
            he = hipEventRecord((hipEvent_t)p.ev_end[l], (hipStream_t)p.side_streams[l]);
            if (he == hipSuccess) he = hipStreamWaitEvent((hipStream_t)stream, (hipEvent_t)p.ev_end[l], 0);
            if (he != hipSuccess && rc == CLG_OK) rc = fail(CLG_HIP_ERROR, "lane join failed: %s", hipGetErrorString(he));
        }
    }
    if (kernel_ns) {
        if (rc == CLG_OK && hipStreamSynchronize((hipStream_t)stream) != hipSuccess)
            rc = fail(CLG_HIP_ERROR, "stream synchronisation failed: %s", hipGetErrorString(hipGetLastError()));
        for (size_t i = 0; i < p.calls.size() && rc == CLG_OK; ++i) {
            float ms = 0.f;
            if (p.elided[i] || (fuse && done[i] == 1)) {     // nothing launched, or launched with its region's first kernel
                kernel_ns[i] = 0;
                continue;
            }
            if (hipEventElapsedTime(&ms, ev[2 * i], ev[2 * i + 1]) != hipSuccess)
                rc = fail(CLG_HIP_ERROR, "hipEventElapsedTime failed");
            kernel_ns[i] = (int64_t)((double)ms * 1.0e6 + 0.5);
        }
        for (auto &e : ev) (void)hipEventDestroy(e);
    }
    return rc;
}

}  // namespace clg
