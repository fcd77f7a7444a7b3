// Pattern matcher: enumerates every legal match (v_s, b_i) -> g of the
// registry on a graph (paper Sec. 3 pattern language; the matching step of
// Alg. 1: for a frontier node v_s and a registry entry b_i, the subgraph g).
//
// Readings fixed here (the paper is silent): v_s is the first node of g in the
// order (depth, node id); a match is legal only with a single exit (every
// non-sink node has all consumers inside g and is no graph output), with
// distinct nodes bound to the pattern's operators and with no wildcard bound to
// a non-sink operator of g (a wildcard is an operand from outside the kernel; a
// non-sink value of g lives only inside it); `add` operands are tried as
// written, then swapped; one match is kept per (v_s, pattern), the first found
// scanning sinks in node order; match ids rank (order of v_s, pattern id).
//
// What it costs: a registry lists the same pattern once per kernel-variant
// backend (some twenty times), so patterns are grouped by structure, each
// structure is matched once, only on the operators of its root's kind, and its
// matches are handed to every pattern of the group.  NasNet-A, 891 operators and
// 376 patterns, 14 000 matches: 13 ms per enumeration pattern by pattern,
// 0.9 ms so.
#include <algorithm>

#include "core.h"

namespace clg {

namespace {

bool same_structure(const Pattern &a, const Pattern &b) {
    if (a.nodes.size() != b.nodes.size()) return false;
    for (size_t i = 0; i < a.nodes.size(); ++i) {
        const clg_pattern_node &x = a.nodes[i], &y = b.nodes[i];
        if (x.op != y.op || x.n_args != y.n_args || x.n_constraints != y.n_constraints) return false;
        for (int k = 0; k < x.n_args; ++k)
            if (x.args[k] != y.args[k]) return false;
        for (int k = 0; k < x.n_constraints; ++k)
            if (x.constraints[k].attr != y.constraints[k].attr || x.constraints[k].lo != y.constraints[k].lo ||
                x.constraints[k].hi != y.constraints[k].hi)
                return false;
    }
    return true;
}

struct Matcher {
    const Graph &g;
    const Pattern &p;
    IdList<CLG_MAX_PATTERN_NODES> pre;     // pattern nodes in pre-order: a node, then its arguments left to right
    int32_t bound[CLG_MAX_PATTERN_NODES];  // graph value per pattern node
    Matcher(const Graph &g_, const Pattern &p_) : g(g_), p(p_) {
        std::fill(bound, bound + CLG_MAX_PATTERN_NODES, -1);
        visit((int)p.nodes.size() - 1);
    }
    void visit(int pi) {
        pre.push_back(pi);
        for (int k = 0; k < p.nodes[pi].n_args; ++k) visit(p.nodes[pi].args[k]);
    }

    bool constraints_ok(const clg_pattern_node &pn, int32_t gv) const {
        for (int c = 0; c < pn.n_constraints; ++c) {
            bool ok = false;
            const int64_t v = attr_value(g, gv, pn.constraints[c].attr, &ok);
            if (!ok || v < pn.constraints[c].lo || v > pn.constraints[c].hi) return false;
        }
        return true;
    }

    // Binds the pattern nodes from pre-order position `at` on in every possible way, given that their
    // parents are bound, and calls `found` once per complete binding, depth first.
    template <class F>
    void bind(size_t at, F &&found) {
        if (at == pre.size()) {
            found();
            return;
        }
        const clg_pattern_node &pn = p.nodes[pre[at]];
        if (pn.op == CLG_WILDCARD) {
            bind(at + 1, found);
            return;
        }
        const int32_t gv = bound[pre[at]];
        const Node &nd = g.nodes[gv];
        if (nd.kind != pn.op || (int)nd.in.size() != pn.n_args) return;
        if (!constraints_ok(pn, gv)) return;
        const int n_orders = (pn.op == CLG_OP_ADD && pn.n_args == 2) ? 2 : 1;
        for (int o = 0; o < n_orders; ++o) {
            for (int k = 0; k < pn.n_args; ++k) bound[pn.args[k]] = nd.in[o ? 1 - k : k];
            bind(at + 1, found);
        }
    }

    // Fills r from a complete binding; false if the match is not legal.
    bool legal(MatchRec *r) const {
        r->binding.n = r->wild.n = 0;
        for (size_t i = 0; i < p.nodes.size(); ++i) {
            r->wild.push_back(bound[i]);
            if (p.nodes[i].op != CLG_WILDCARD) r->binding.push_back(bound[i]);
        }
        r->nodes = r->binding;
        std::sort(r->nodes.begin(), r->nodes.end());
        if (std::adjacent_find(r->nodes.begin(), r->nodes.end()) != r->nodes.end()) return false;
        const int32_t sink = r->binding[r->binding.size() - 1];
        auto inside = [&](int32_t v) { return std::find(r->nodes.begin(), r->nodes.end(), v) != r->nodes.end(); };
        for (size_t i = 0; i < p.nodes.size(); ++i)
            if (p.nodes[i].op == CLG_WILDCARD && bound[i] != sink && inside(bound[i])) return false;
        r->first = sink;
        r->sink = sink;
        for (int32_t v : r->nodes) {
            if (g.rank[v] < g.rank[r->first]) r->first = v;
            if (v == sink) continue;
            if (g.is_output[v]) return false;
            for (int32_t c : g.consumers[v])
                if (!inside(c)) return false;
        }
        return true;
    }
};

}  // namespace

int32_t match_all(Context &ctx, Graph &g) {
    g.finalize();
    std::vector<std::vector<int32_t>> by_kind(CLG_OP_COUNT);       // operators of each kind by ascending id
    for (int32_t v : g.op_ids) by_kind[(size_t)g.nodes[v].kind].push_back(v);
    std::vector<std::vector<int32_t>> groups;                      // pattern ids of one structure, ascending
    for (size_t pi = 0; pi < ctx.patterns.size(); ++pi) {
        const Pattern &p = ctx.patterns[pi];
        int n_ops = 0;
        for (auto &pn : p.nodes) n_ops += pn.op != CLG_WILDCARD;
        if (n_ops > CLG_MAX_MATCH_NODES) continue;
        size_t k = 0;
        while (k < groups.size() && !same_structure(ctx.patterns[(size_t)groups[k][0]], p)) ++k;
        if (k == groups.size()) groups.emplace_back();
        groups[k].push_back((int32_t)pi);
    }
    struct Ref { int32_t pattern, rec; };
    std::vector<MatchRec> recs;                                    // one per (first node, structure)
    std::vector<std::vector<Ref>> at(g.order.size());              // matches by the position of their first node
    std::vector<int32_t> taken(g.order.size(), -1);                // structure that last matched from this position
    size_t total = 0;
    for (size_t k = 0; k < groups.size(); ++k) {
        const Pattern &p = ctx.patterns[(size_t)groups[k][0]];
        const int32_t root_op = p.nodes.back().op;
        if (root_op == CLG_WILDCARD) continue;
        Matcher m(g, p);
        MatchRec r;
        for (int32_t sink : by_kind[(size_t)root_op]) {
            m.bound[p.nodes.size() - 1] = sink;
            m.bind(0, [&]() {
                if (!m.legal(&r)) return;
                const int32_t rank = g.rank[r.first];
                if (taken[(size_t)rank] == (int32_t)k) return;
                taken[(size_t)rank] = (int32_t)k;
                for (int32_t pi : groups[k]) at[(size_t)rank].push_back(Ref{pi, (int32_t)recs.size()});
                total += groups[k].size();
                recs.push_back(r);
            });
        }
    }
    g.matches.clear();
    g.matches.reserve(total);
    for (auto &here : at) {
        std::sort(here.begin(), here.end(), [](const Ref &a, const Ref &b) { return a.pattern < b.pattern; });
        for (const Ref &f : here) {
            g.matches.push_back(recs[(size_t)f.rec]);
            g.matches.back().pattern = f.pattern;
            g.matches.back().backend = ctx.patterns[(size_t)f.pattern].backend;
        }
    }
    g.matched = true;
    return CLG_OK;
}

}  // namespace clg
