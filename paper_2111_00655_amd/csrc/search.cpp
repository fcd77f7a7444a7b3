// Op-level placement search: the dynamic programme of paper Sec. 4.2
// (Eq. 3 and Alg. 1) over a cost table of integer nanoseconds.
//
// Stored sub-placements are keyed by the set of operators they cover.  The
// frontier nodes of Alg. 1 are visited in the order (depth, node id); because
// that order is total, the priority queue is a scan over positions that skips
// positions no sub-placement is waiting at (nodes never enqueued).  A match g
// found at frontier v_s relaxes every waiting sub-placement that is disjoint
// from g (the set S); the result waits at its own lowest uncovered node (the
// new frontier nodes F).  Each placement is generated along exactly one path,
// so the result is the minimum over all placements (Eq. 1).
//
// Ties: (total, ascending match-id list) is minimised lexicographically, which
// makes the answer a pure function of the inputs.
//
// What it costs: the number of (sub-placement, distinct operator set) pairs -
// NasNet-A with its separable convolutions operator by operator: 53 000 stored
// sub-placements, 119 000 pairs.
//  * Matches of one frontier node that cover the same operators (the same
//    pattern under every kernel-variant backend) differ in cost only: the
//    cheapest (the earliest among equals) stands for all of them.
//  * A covered set is stored as the window of bits from its lowest uncovered
//    operator on (everything below is covered): a few words instead of one bit
//    per operator of the graph, in one flat array.
//  * Sets are found by hash: every operator has a random 64-bit number, a set's
//    hash is the XOR of its members', so extending a set by a match costs one
//    XOR; equality is decided on the windows, never on the hash.
//  * The loops over a window's words have a constant length up to four words,
//    which leaves a pair without inner loops: 3.6 -> 3.1 ms on that network
//    (three words, 8-CPU host).  Wider windows take the same code with a length
//    read at run time.
// 120 - 230 ms before sets were windows.
#include <algorithm>

#include "core.h"

namespace clg {

namespace {

struct Sub {                 // one stored sub-placement: C_opt(s), P_opt(s)
    int64_t cost;
    uint64_t hash;           // of the covered set
    int32_t parent;          // sub-placement it extends, -1: none
    int32_t match;           // match added last
    int32_t frontier;        // lowest uncovered position
    int32_t next;            // next sub-placement waiting at the same frontier, -1: last
};

// Open-addressing table of sub-placement ids by hash (linear probing, at most half full).
struct Table {
    std::vector<int32_t> slot;
    uint64_t mask = 0;
    explicit Table(size_t n) : slot(n, -1), mask(n - 1) {}
    void grow(const std::vector<Sub> &subs) {
        const size_t n = slot.size() * 2;
        slot.assign(n, -1);
        mask = n - 1;
        for (size_t i = 0; i < subs.size(); ++i) {
            uint64_t at = subs[i].hash & mask;
            while (slot[at] >= 0) at = (at + 1) & mask;
            slot[at] = (int32_t)i;
        }
    }
};

uint64_t mix(uint64_t x) {   // splitmix64
    x += 0x9E3779B97F4A7C15ull;
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    return x ^ (x >> 31);
}

void placement_of(const std::vector<Sub> &subs, int32_t idx, int32_t extra,
                  std::vector<int32_t> *out) {
    out->clear();
    if (extra >= 0) out->push_back(extra);
    for (int32_t s = idx; s >= 0 && subs[s].match >= 0; s = subs[s].parent)
        out->push_back(subs[s].match);
    std::reverse(out->begin(), out->end());
}

// W: words of a window where the compiler is to know them, 0: `any_words`.
template <int W>
int32_t search(Graph &g, size_t any_words, const int64_t *cost, int64_t eps,
               std::vector<int32_t> *chosen, int64_t *total) {
    const size_t words = W ? (size_t)W : any_words;
    const int n = (int)g.order.size();
    const size_t n_matches = g.matches.size();
    std::vector<uint64_t> key((size_t)n);                 // random number of each position
    for (int r = 0; r < n; ++r) key[(size_t)r] = mix((uint64_t)r);

    std::vector<Sub> subs;
    std::vector<uint64_t> bits;                            // windows, `words` per sub-placement
    Table index(1024);
    std::vector<int32_t> head((size_t)n + 1, -1), tail((size_t)n + 1, -1);    // sub-placements waiting at a position, in order of creation
    subs.push_back(Sub{0, 0, -1, -1, 0, -1});              // C_opt(empty) = 0
    bits.resize(words, 0);
    index.slot[0] = 0;
    head[0] = tail[0] = 0;

    struct Group { int32_t match; uint64_t hash; };        // the distinct operator sets at a frontier node: cheapest match
    std::vector<Group> groups;
    std::vector<uint64_t> gbits;
    std::vector<uint64_t> nb(words + 1), mb(words + 1);
    int64_t max_p = 0, max_f = 0, max_s = 0;
    std::vector<int32_t> pa, pb, new_frontiers;
    size_t mi = 0;                                         // matches are sorted by (rank of first node, pattern id)
    for (int pos = 0; pos < n; ++pos) {
        const size_t begin = mi;
        while (mi < n_matches && g.rank[g.matches[mi].first] == pos) ++mi;
        if (head[pos] < 0) continue;                       // never enqueued
        max_p = std::max(max_p, (int64_t)(mi - begin));
        const int base = pos / 64;
        groups.clear();
        gbits.clear();
        for (size_t i = begin; i < mi; ++i) {
            if (cost[i] >= CLG_COST_INF) continue;
            std::fill(mb.begin(), mb.end(), 0);
            uint64_t h = 0;
            for (int32_t v : g.matches[i].nodes) {
                const int r = g.rank[v];
                mb[(size_t)(r / 64 - base)] |= (uint64_t)1 << (r % 64);
                h ^= key[(size_t)r];
            }
            size_t k = 0;
            while (k < groups.size() && !(groups[k].hash == h && std::equal(mb.begin(), mb.begin() + (long)words, gbits.begin() + (long)(k * words)))) ++k;
            if (k == groups.size()) {
                groups.push_back(Group{(int32_t)i, h});
                gbits.insert(gbits.end(), mb.begin(), mb.begin() + (long)words);
            } else if (cost[i] < cost[groups[k].match]) {
                groups[k].match = (int32_t)i;
            }
        }
        for (size_t k = 0; k < groups.size(); ++k) {
            const int32_t m = groups[k].match;
            const uint64_t *const mw = gbits.data() + k * words;
            int64_t s_size = 0;
            new_frontiers.clear();
            for (int32_t si = head[pos]; si >= 0; si = subs[(size_t)si].next) {
                const uint64_t *const sw = bits.data() + (size_t)si * words;
                uint64_t common = 0;
                for (size_t w = 0; w < words; ++w) common |= sw[w] & mw[w];
                if (common) continue;
                ++s_size;
                for (size_t w = 0; w < words; ++w) nb[w] = sw[w] | mw[w];
                const uint64_t h = subs[(size_t)si].hash ^ groups[k].hash;
                const int64_t c = subs[(size_t)si].cost + cost[m] + eps;
                // new frontier: the lowest clear bit at or above pos (the spare word is clear)
                size_t w = 0;
                uint64_t inv = ~nb[0] & (~(uint64_t)0 << (pos % 64));
                while (!inv) inv = ~nb[++w];
                const int f = std::min(n, (int)(base + (int)w) * 64 + __builtin_ctzll(inv));
                const size_t shift = (size_t)(std::min(f, n) / 64 - base);
                // the window from the new frontier's word on (bits of that word below it are all covered)
                uint64_t at = h & index.mask;
                int32_t hit = -1;
                for (; index.slot[at] >= 0; at = (at + 1) & index.mask) {
                    const Sub &o = subs[(size_t)index.slot[at]];
                    if (o.hash != h || o.frontier != f) continue;
                    const uint64_t *const ow = bits.data() + (size_t)index.slot[at] * words;
                    bool same = true;
                    for (size_t u = 0; u < words && same; ++u) same = ow[u] == (u + shift <= words ? nb[u + shift] : 0);
                    if (same) {
                        hit = index.slot[at];
                        break;
                    }
                }
                if (hit < 0) {
                    const int32_t id = (int32_t)subs.size();
                    for (size_t u = 0; u < words; ++u) bits.push_back(u + shift <= words ? nb[u + shift] : 0);
                    subs.push_back(Sub{c, h, si, m, f, -1});
                    index.slot[at] = id;
                    if (subs.size() * 2 > index.slot.size()) index.grow(subs);
                    if (head[f] < 0) head[f] = id;
                    else subs[(size_t)tail[f]].next = id;
                    tail[f] = id;
                    if (std::find(new_frontiers.begin(), new_frontiers.end(), f) == new_frontiers.end()) new_frontiers.push_back(f);
                } else {
                    Sub &old = subs[(size_t)hit];
                    bool better = c < old.cost;
                    if (c == old.cost) {
                        placement_of(subs, si, m, &pa);
                        placement_of(subs, hit, -1, &pb);
                        better = pa < pb;
                    }
                    if (better) {
                        old.cost = c;
                        old.parent = si;
                        old.match = m;
                    }
                }
            }
            max_s = std::max(max_s, s_size);
            max_f = std::max<int64_t>(max_f, (int64_t)new_frontiers.size());
        }
    }
    g.stats[0] = n; g.stats[1] = max_p; g.stats[2] = max_f; g.stats[3] = max_s;
    g.stats[4] = (int64_t)subs.size();

    // the set of all operators is the only one that waits at position n
    const int32_t full = n ? head[n] : 0;
    if (full < 0) return fail(CLG_NOT_A_COVER, "no placement covers every operator of the graph");
    placement_of(subs, full, -1, chosen);
    *total = subs[(size_t)full].cost;
    return CLG_OK;
}

}  // namespace

int32_t search_dp(Graph &g, size_t, const int64_t *cost, int64_t eps,
                  std::vector<int32_t> *chosen, int64_t *total) {
    g.finalize();
    for (size_t i = 0; i < g.matches.size(); ++i)
        if (cost[i] < 0) return fail(CLG_INVALID_ARG, "negative cost for match %zu", i);
    if (eps < 0) return fail(CLG_INVALID_ARG, "negative eps");

    // A set whose lowest uncovered position is f holds no position above f + span: every match in it starts at
    // or below f.  Its window starts at word f / 64 of the bit string and is `words` long; one spare word
    // lets a window that is moved to a later frontier be read past its end.
    int span = 0;
    for (const MatchRec &m : g.matches)
        for (int32_t v : m.nodes) span = std::max(span, g.rank[v] - g.rank[m.first]);
    const size_t words = (size_t)(span + 63) / 64 + 1;
    if (words == 1) return search<1>(g, words, cost, eps, chosen, total);
    if (words == 2) return search<2>(g, words, cost, eps, chosen, total);
    if (words == 3) return search<3>(g, words, cost, eps, chosen, total);
    if (words == 4) return search<4>(g, words, cost, eps, chosen, total);
    return search<0>(g, words, cost, eps, chosen, total);
}

}  // namespace clg
