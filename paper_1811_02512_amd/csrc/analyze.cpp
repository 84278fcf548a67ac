// Host symbolic analysis for the level-scheduled block LDU.
//
// Steps (paper, Sec. II-B): fill-reducing elimination order (our reading:
// exact minimum degree, the paper itself eliminates in the given numbering),
// FormFilledGraph, FormEliminationTree, FormHierarchicalPartition.  The
// filled pattern falls out of the symbolic elimination itself: the neighbours
// a node still has when it is eliminated are exactly its higher neighbours in
// the filled graph.  On top of the paper's structures this builds the index
// maps the kernels need: admittance CSR with its contributing branches,
// position <-> bus maps, Y entry of every filled block, lower-neighbour lists
// and the per-destination update pairs of the left-looking factorisation.
#include <algorithm>
#include <cstdint>
#include <cstring>
#include <queue>
#include <utility>

#include "pf.h"
#include "pf_internal.h"

namespace pf {

namespace {

// Sorted-vector union of a and b without the values x and y.
void merge_without(const std::vector<int32_t>& a, const std::vector<int32_t>& b, int32_t x,
                   int32_t y, std::vector<int32_t>& out)
{
    out.clear();
    out.reserve(a.size() + b.size());
    size_t i = 0, j = 0;
    while (i < a.size() || j < b.size()) {
        int32_t v;
        if (j >= b.size() || (i < a.size() && a[i] < b[j])) {
            v = a[i++];
        } else if (i >= a.size() || b[j] < a[i]) {
            v = b[j++];
        } else {
            v = a[i++];
            ++j;
        }
        if (v != x && v != y) out.push_back(v);
    }
}

size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

// One level's right-looking terms by destination, for the operation lists:
// destinations below `slots` are slots, from there on diagonals.  Layout of
// the positions that place() is given, from 0: every destination's first
// term (slots, padded to a multiple of `pad` where diagonals follow, then
// diagonals), then the second terms of the destinations
// that have one (slots, then diagonals), then the further terms, each
// destination's together.  Within a kind, destinations with more terms come
// first, so a thread finds its second term without reading the first.
struct LevelTerms {
    struct Term {
        int32_t d, a, b, j;
    };
    std::vector<Term> terms;
    std::vector<int32_t> dst, third, count, at, seq;
    std::vector<uint64_t> keys;
    int32_t slots = 0;
    // ns: slots (padded), nd: slots and diagonals, total: all positions; ls, ld:
    // slots and diagonals with more than kTailSerial terms
    int32_t ns = 0, nd = 0, ns2 = 0, nd2 = 0, ls = 0, ld = 0, total = 0;

    LevelTerms(int32_t slots_, int32_t nodes)
        : count((size_t)slots_ + nodes, 0),
          at((size_t)slots_ + nodes, 0),
          seq((size_t)slots_ + nodes, 0),
          slots(slots_)
    {
    }
    void start()
    {
        terms.clear();
        dst.clear();
    }
    void add(int32_t d, int32_t a, int32_t b, int32_t j)
    {
        if (count[d]++ == 0) dst.push_back(d);
        terms.push_back({d, a, b, j});
    }
    // The terms of node j with slots [s0, s1), higher(t) the neighbour of
    // slot t and first(k) the first slot of k: slots are indexed alike.
    template <class H, class F>
    void add_node(int32_t j, int32_t s0, int32_t s1, H&& higher, F&& first)
    {
        for (int32_t b = s0; b < s1; ++b) {
            const int32_t k = higher(b);
            add(slots + k, b, b, j);
            int32_t d = first(k);
            for (int32_t a = b + 1; a < s1; ++a) {
                while (higher(d) != higher(a)) ++d;  // present: the filled pattern is closed
                add(d, a, b, j);
            }
        }
    }
    // place(position, destination, term, offset of its next term or 0, terms
    // of the destination that follow)
    template <class F>
    void place(int32_t pad, F&& fn)
    {
        // slots first, then many terms first, then by destination, as one key
        const int32_t n = (int32_t)dst.size();
        keys.resize(n);
        for (int32_t i = 0; i < n; ++i)
            keys[i] = (uint64_t)(dst[i] >= slots) << 63 |
                      (uint64_t)(INT32_MAX - count[dst[i]]) << 32 | (uint32_t)dst[i];
        std::sort(keys.begin(), keys.end());
        for (int32_t i = 0; i < n; ++i) dst[i] = (int32_t)(uint32_t)keys[i];
        int32_t real = 0;
        ns2 = nd2 = ls = ld = 0;
        for (int32_t d : dst) {
            real += d < slots;
            (d < slots ? ns2 : nd2) += count[d] > 1;
            (d < slots ? ls : ld) += count[d] > kTailSerial;
        }
        ns = n > real ? (real + pad - 1) / pad * pad : real;
        nd = ns + n - real;
        int32_t more = nd + ns2 + nd2;
        for (int32_t i = 0; i < n; ++i) {
            const int32_t d = dst[i];
            at[d] = i;  // index among the destinations
            seq[d] = 0;
        }
        third.assign(n, 0);
        for (int32_t i = 0; i < n; ++i) {
            third[i] = more;
            more += std::max(0, count[dst[i]] - 2);
        }
        total = more;
        for (const Term& q : terms) {
            const int32_t i = at[q.d], k = seq[q.d]++;
            const int32_t first = i < real ? i : ns + i - real;
            const int32_t second = nd + (i < real ? i : ns2 + i - real);
            const int32_t p = k == 0 ? first : k == 1 ? second : third[i] + k - 2;
            const bool last = k + 1 == count[q.d];
            const int32_t nx = k == 0 ? second : third[i] + k - 1;
            fn(p, q.d < slots ? q.d : q.d - slots, q, last ? 0 : nx - p, count[q.d] - 1 - k);
        }
        for (int32_t d : dst) count[d] = 0;
    }
};

}  // namespace

size_t HostSym::dev_bytes() const
{
    const std::vector<int32_t>* arrs[] = {&yptr,      &ycol,      &ybr_ptr, &ybr,    &perm,
                                          &pos,       &Lp,        &Li,      &ydiag,  &level_ptr,
                                          &level_nodes, &level_g, &node_info, &slot_info, &rl,
                                          &upd,       &t_node,    &t_slot,  &t_rl,
                                          &t_lev,     &t_op,      &from,    &to,     &sub_idx,
                                          &sub_ptr,   &sub_cum,   &up.node, &up.slot, &up.rl,
                                          &up.upd,    &up.lev,    &up.op,   &up.next};
    size_t total = 0;
    for (auto* a : arrs) total += align256(std::max<size_t>(a->size(), 1) * sizeof(int32_t));
    return total;
}

int analyze(int n, int m, const int32_t* from, const int32_t* to, int slack, int ordering,
            HostSym& s, std::string& msg)
{
    if (n < 2 || m < 0 || slack < 0 || slack >= n || (m > 0 && (!from || !to))) {
        msg = "pf_analyze: need n >= 2, m >= 0, 0 <= slack < n and branch arrays";
        return PF_E_INVALID;
    }
    if (ordering != PF_ORDER_MINDEG && ordering != PF_ORDER_NATURAL) {
        msg = "pf_analyze: unknown ordering";
        return PF_E_INVALID;
    }
    for (int e = 0; e < m; ++e) {
        if (from[e] < 0 || from[e] >= n || to[e] < 0 || to[e] >= n) {
            msg = "pf_analyze: branch " + std::to_string(e) + " has a bus index out of range";
            return PF_E_INVALID;
        }
        if (from[e] == to[e]) {
            msg = "pf_analyze: branch " + std::to_string(e) + " is a self loop";
            return PF_E_INVALID;
        }
    }
    s = HostSym();
    s.n = n;
    s.m = m;
    s.nn = n - 1;
    s.slack = slack;
    s.ordering = ordering;
    s.from.assign(from, from + m);
    s.to.assign(to, to + m);

    // incidence: (other bus, branch) per bus, sorted: inc[ip[i] .. ip[i + 1])
    using Inc = std::pair<int32_t, int32_t>;
    std::vector<int32_t> ip(n + 1, 0);
    for (int e = 0; e < m; ++e) {
        ++ip[from[e] + 1];
        ++ip[to[e] + 1];
    }
    for (int i = 0; i < n; ++i) ip[i + 1] += ip[i];
    std::vector<Inc> inc(2 * (size_t)m);
    {
        std::vector<int32_t> cur(ip.begin(), ip.end() - 1);
        for (int e = 0; e < m; ++e) {
            inc[cur[from[e]]++] = {to[e], e};
            inc[cur[to[e]]++] = {from[e], e};
        }
    }
    for (int i = 0; i < n; ++i) std::sort(inc.begin() + ip[i], inc.begin() + ip[i + 1]);

    // every bus must reach the slack
    {
        std::vector<char> seen(n, 0);
        std::vector<int32_t> stack{slack};
        seen[slack] = 1;
        int cnt = 1;
        while (!stack.empty()) {
            int v = stack.back();
            stack.pop_back();
            for (int q = ip[v]; q < ip[v + 1]; ++q)
                if (!seen[inc[q].first]) {
                    seen[inc[q].first] = 1;
                    ++cnt;
                    stack.push_back(inc[q].first);
                }
        }
        if (cnt != n) {
            msg = "pf_analyze: " + std::to_string(n - cnt) + " bus(es) not connected to the slack";
            return PF_E_DISCONNECTED;
        }
    }

    // admittance CSR (diagonal always present) and contributing branches, both
    // ascending
    s.yptr.assign(n + 1, 0);
    s.ycol.reserve(n + 2 * (size_t)m);
    s.ybr.reserve(4 * (size_t)m);
    s.ybr_ptr.reserve(n + 2 * (size_t)m + 1);
    s.ybr_ptr.push_back(0);
    for (int i = 0; i < n; ++i) {
        auto diagonal = [&]() {
            s.ycol.push_back(i);
            const size_t b0 = s.ybr.size();
            for (int q = ip[i]; q < ip[i + 1]; ++q) s.ybr.push_back(inc[q].second);
            std::sort(s.ybr.begin() + b0, s.ybr.end());
            s.ybr_ptr.push_back((int32_t)s.ybr.size());
        };
        bool done = false;
        for (int q = ip[i]; q < ip[i + 1];) {
            const int32_t c = inc[q].first;
            if (c > i && !done) {
                diagonal();
                done = true;
            }
            s.ycol.push_back(c);
            for (; q < ip[i + 1] && inc[q].first == c; ++q) s.ybr.push_back(inc[q].second);
            s.ybr_ptr.push_back((int32_t)s.ybr.size());
        }
        if (!done) diagonal();
        s.yptr[i + 1] = (int32_t)s.ycol.size();
    }
    // reduced graph: node v <-> bus, ascending bus order without the slack
    const int nn = s.nn;
    std::vector<int32_t> bus_of(nn), node_of(n, -1);
    for (int i = 0, v = 0; i < n; ++i)
        if (i != slack) {
            node_of[i] = v;
            bus_of[v++] = i;
        }
    std::vector<std::vector<int32_t>> adj(nn);
    for (int v = 0; v < nn; ++v) {
        const int i = bus_of[v];  // its row's columns ascend, and so do their nodes
        adj[v].reserve(s.yptr[i + 1] - s.yptr[i]);
        for (int q = s.yptr[i]; q < s.yptr[i + 1]; ++q) {
            const int w = node_of[s.ycol[q]];
            if (w >= 0 && w != v) adj[v].push_back(w);
        }
    }

    // symbolic elimination: minimum degree (ties to the lowest node, i.e.
    // lowest bus) or the natural order; hi[v] = neighbours left at elimination
    std::vector<std::vector<int32_t>> hi(nn);
    std::vector<int32_t> order(nn);
    {
        std::vector<char> gone(nn, 0);
        using Item = std::pair<int32_t, int32_t>;  // (degree, node)
        std::priority_queue<Item, std::vector<Item>, std::greater<Item>> heap;
        if (ordering == PF_ORDER_MINDEG)
            for (int v = 0; v < nn; ++v) heap.push({(int32_t)adj[v].size(), v});
        std::vector<int32_t> tmp;
        for (int step = 0; step < nn; ++step) {
            int p;
            if (ordering == PF_ORDER_NATURAL) {
                p = step;
            } else {
                for (;;) {
                    Item it = heap.top();
                    heap.pop();
                    if (!gone[it.second] && it.first == (int32_t)adj[it.second].size()) {
                        p = it.second;
                        break;
                    }
                }
            }
            order[step] = p;
            gone[p] = 1;
            hi[p] = std::move(adj[p]);
            adj[p].clear();
            for (int32_t a : hi[p]) {
                merge_without(adj[a], hi[p], a, p, tmp);
                adj[a].swap(tmp);
                if (ordering == PF_ORDER_MINDEG) heap.push({(int32_t)adj[a].size(), a});
            }
        }
    }

    // positions and the filled pattern S(p)
    std::vector<int32_t> pos_of_node(nn);
    for (int p = 0; p < nn; ++p) pos_of_node[order[p]] = p;
    s.perm.resize(nn);
    s.pos.assign(n, -1);
    for (int p = 0; p < nn; ++p) {
        s.perm[p] = bus_of[order[p]];
        s.pos[s.perm[p]] = p;
    }
    s.Lp.assign(nn + 1, 0);
    for (int p = 0; p < nn; ++p) {
        const size_t b0 = s.Li.size();
        for (int32_t v : hi[order[p]]) s.Li.push_back(pos_of_node[v]);
        std::sort(s.Li.begin() + b0, s.Li.end());
        s.Lp[p + 1] = (int32_t)s.Li.size();
    }
    hi.clear();
    const int64_t nnzl = (int64_t)s.Li.size();
    s.owner.resize(nnzl);
    for (int p = 0; p < nn; ++p)
        for (int q = s.Lp[p]; q < s.Lp[p + 1]; ++q) s.owner[q] = p;

    // elimination tree and levels (level = 1 + highest child level)
    s.parent.assign(nn, -1);
    s.level.assign(nn, 1);
    for (int p = 0; p < nn; ++p) {
        if (s.Lp[p + 1] > s.Lp[p]) s.parent[p] = s.Li[s.Lp[p]];
        if (s.parent[p] >= 0)
            s.level[s.parent[p]] = std::max(s.level[s.parent[p]], s.level[p] + 1);
    }
    int nlev = 0;
    for (int p = 0; p < nn; ++p) nlev = std::max(nlev, s.level[p]);
    s.level_ptr.assign(nlev + 1, 0);
    for (int p = 0; p < nn; ++p) s.level_ptr[s.level[p]]++;
    for (int l = 0; l < nlev; ++l) s.level_ptr[l + 1] += s.level_ptr[l];
    s.level_nodes.assign(nn, 0);
    {
        std::vector<int32_t> cur(s.level_ptr.begin(), s.level_ptr.end() - 1);
        for (int p = 0; p < nn; ++p) s.level_nodes[cur[s.level[p] - 1]++] = p;
    }
    s.max_width = 0;
    for (int l = 0; l < nlev; ++l)
        s.max_width = std::max(s.max_width, s.level_ptr[l + 1] - s.level_ptr[l]);

    // admittance entries of every block: at[] marks where the columns of p's
    // row stand; rows ascend, so the entries of a column come in its own
    // row's order and cur[] finds the transposed entry
    s.ydiag.resize(nn);
    s.ylo.resize(nnzl);
    s.yup.resize(nnzl);
    {
        std::vector<int32_t> cur(s.yptr.begin(), s.yptr.end() - 1), at(n, -1);
        std::vector<int32_t> transposed(s.ycol.size());
        for (int i = 0; i < n; ++i)
            for (int q = s.yptr[i]; q < s.yptr[i + 1]; ++q) transposed[q] = cur[s.ycol[q]]++;
        for (int p = 0; p < nn; ++p) {
            const int bp = s.perm[p];
            for (int q = s.yptr[bp]; q < s.yptr[bp + 1]; ++q) at[s.ycol[q]] = q;
            s.ydiag[p] = at[bp];
            for (int q = s.Lp[p]; q < s.Lp[p + 1]; ++q) {
                const int32_t u = at[s.perm[s.Li[q]]];
                s.yup[q] = u;
                s.ylo[q] = u < 0 ? -1 : transposed[u];
            }
            for (int q = s.yptr[bp]; q < s.yptr[bp + 1]; ++q) at[s.ycol[q]] = -1;
        }
    }

    // lower neighbours R(p) with the slot of p inside S(i), ascending i
    s.Rp.assign(nn + 1, 0);
    for (int64_t q = 0; q < nnzl; ++q) s.Rp[s.Li[q] + 1]++;
    for (int p = 0; p < nn; ++p) s.Rp[p + 1] += s.Rp[p];
    s.Ri.resize(nnzl);
    s.Rs.resize(nnzl);
    {
        std::vector<int32_t> cur(s.Rp.begin(), s.Rp.end() - 1);
        for (int i = 0; i < nn; ++i)
            for (int q = s.Lp[i]; q < s.Lp[i + 1]; ++q) {
                int k = s.Li[q];
                s.Ri[cur[k]] = i;
                s.Rs[cur[k]] = q;
                cur[k]++;
            }
    }

    // update pairs per destination slot.  For node j and descendant i with
    // b = slot(i;j), every k after j in S(i) is also in S(j) (the higher
    // neighbours of a node form a clique in the filled graph); the block
    // pair at a = slot(i;k) updates destination slot(j;k).
    s.Up.assign(nnzl + 1, 0);
    {
        std::vector<int32_t> dst;  // destination slots, in the walk's order
        dst.reserve(8 * (size_t)nnzl);
        for (int j = 0; j < nn; ++j)
            for (int r = s.Rp[j]; r < s.Rp[j + 1]; ++r) {
                int d = s.Lp[j];
                for (int a = s.Rs[r] + 1; a < s.Lp[s.Ri[r] + 1]; ++a) {
                    const int k = s.Li[a];
                    while (d < s.Lp[j + 1] && s.Li[d] < k) ++d;
                    if (d >= s.Lp[j + 1] || s.Li[d] != k) {
                        msg = "pf_analyze: internal error, filled pattern is not closed";
                        return PF_E_INVALID;
                    }
                    s.Up[d + 1]++;
                    dst.push_back(d);
                }
            }
        for (int64_t q = 0; q < nnzl; ++q) s.Up[q + 1] += s.Up[q];
        s.Ua.resize(s.Up[nnzl]);
        s.Ub.resize(s.Up[nnzl]);
        std::vector<int32_t> cur(s.Up.begin(), s.Up.end() - 1);
        size_t u = 0;
        for (int64_t r = 0; r < nnzl; ++r)
            for (int a = s.Rs[r] + 1; a < s.Lp[s.Ri[r] + 1]; ++a) {
                const int32_t x = cur[dst[u++]]++;
                s.Ua[x] = a;
                s.Ub[x] = s.Rs[r];
            }
    }

    // packed records (layouts documented with DevSym)
    s.node_info.assign(12 * (size_t)nn, 0);
    for (int x = 0; x < nn; ++x) {
        const int j = s.level_nodes[x];
        int32_t* r = &s.node_info[12 * (size_t)x];
        r[0] = j;
        r[1] = s.perm[j];
        r[2] = s.Rp[j];
        r[3] = s.Rp[j + 1];
        r[4] = s.Lp[j];
        r[5] = s.Lp[j + 1];
        r[6] = s.ydiag[j];
        r[8] = s.yptr[s.perm[j]];
        r[9] = s.yptr[s.perm[j] + 1];
    }
    s.slot_info.assign(8 * (size_t)nnzl, 0);
    for (int64_t q = 0; q < nnzl; ++q) {
        int32_t* r = &s.slot_info[8 * (size_t)q];
        r[0] = s.Li[q];
        r[1] = s.perm[s.Li[q]];
        r[2] = s.ylo[q];
        r[3] = s.yup[q];
        r[4] = s.Up[q];
        r[5] = s.Up[q + 1];
        r[6] = s.owner[q];
        r[7] = s.perm[s.owner[q]];
    }
    s.rl.resize(2 * (size_t)nnzl);
    for (int64_t q = 0; q < nnzl; ++q) {
        s.rl[2 * q] = s.Ri[q];
        s.rl[2 * q + 1] = s.Rs[q];
    }
    s.upd.resize(2 * s.Ua.size());
    for (size_t u = 0; u < s.Ua.size(); ++u) {
        s.upd[2 * u] = s.Ua[u];
        s.upd[2 * u + 1] = s.Ub[u];
    }
    default_mapping(s);
    build_tail(s, s.tail_budget);
    return PF_OK;
}

// The LDS tail: the largest run of top levels whose values, with the
// Newton kernel's PV bitmask, fit the budget.
// Its top may be a clique chain: single-node levels where every node is
// adjacent to all nodes above it in the filled graph.  That part is solved
// densely (column by column on one wavefront).
void build_tail(HostSym& s, int64_t budget)
{
    const int nlev = (int)s.level_ptr.size() - 1;
    const int nn = s.nn;
    int L = nlev;
    int64_t K = 0, TS = 0;
    if (budget > 0) {
        while (L > 0) {
            const int l = L - 1;
            int64_t k2 = K, t2 = TS, ops = 0;
            for (int x = s.level_ptr[l]; x < s.level_ptr[l + 1]; ++x) {
                const int j = s.level_nodes[x];
                const int64_t d = s.Lp[j + 1] - s.Lp[j];
                ++k2;
                t2 += d;
                ops += d * (d + 1) / 2;
            }
            if (tail_bytes(k2, t2) + pv_mask_bytes(s.n) > budget || t2 > kTailIndexMax ||
                k2 > kTailIndexMax || ops > kTailOpsMax)
                break;
            K = k2;
            TS = t2;
            L = l;
        }
    }
    s.tail_level = L;
    s.tail_nodes = (int32_t)K;
    s.tail_slots = (int32_t)TS;
    s.tail_lds = K ? (int32_t)tail_bytes(K, TS) : 0;
    s.tail_clique = 0;
    s.t_node.clear();
    s.t_slot.clear();
    s.t_rl.clear();
    s.t_lev.clear();
    s.tail_longs = 0;
    s.t_op.clear();
    build_subtrees(s);
    s.up = build_upper(s, s.want_whole);
    if (K == 0) return;

    // clique chain at the top of the tail: level nlev-1-d holds one node
    // whose higher neighbours are exactly the d chain nodes above it
    {
        std::vector<int32_t> chain;  // from the root down
        for (int l = nlev - 1; l >= L; --l) {
            if (s.level_ptr[l + 1] - s.level_ptr[l] != 1) break;
            const int j = s.level_nodes[s.level_ptr[l]];
            const int d = (int)chain.size();
            if (s.Lp[j + 1] - s.Lp[j] != d) break;
            bool ok = true;
            for (int q = 0; q < d && ok; ++q) ok = s.Li[s.Lp[j] + q] == chain[d - 1 - q];
            if (!ok) break;
            chain.push_back(j);
        }
        s.tail_clique = chain.size() >= 3 ? (int32_t)chain.size() : 0;
    }

    const int64_t nnzl = (int64_t)s.Li.size();
    std::vector<int32_t> loc(nn, -1), sloc(nnzl, -1);
    std::vector<int32_t> tnodes;
    for (int l = L; l < nlev; ++l) {
        for (int x = s.level_ptr[l]; x < s.level_ptr[l + 1]; ++x) {
            loc[s.level_nodes[x]] = (int32_t)tnodes.size();
            tnodes.push_back(s.level_nodes[x]);
        }
    }
    const int32_t kfirst = (int32_t)K - s.tail_clique;  // first local node of the clique
    auto in_clique = [&](int p) { return loc[p] >= kfirst; };
    int32_t ts = 0;
    for (int j : tnodes)
        for (int q = s.Lp[j]; q < s.Lp[j + 1]; ++q) sloc[q] = ts++;
    s.t_node.assign(8 * (size_t)K, 0);
    s.t_slot.assign(4 * (size_t)TS, 0);
    int32_t run = 0;
    for (size_t jl = 0; jl < tnodes.size(); ++jl) {
        const int j = tnodes[jl];
        int32_t* r = &s.t_node[8 * jl];
        r[0] = j;
        r[1] = s.perm[j];
        r[2] = s.ydiag[j];
        r[3] = run;  // local slots were numbered in this same node order
        run += s.Lp[j + 1] - s.Lp[j];
        r[4] = run;
        r[5] = (int32_t)(s.t_rl.size() / 2);
        for (int q = s.Rp[j]; q < s.Rp[j + 1]; ++q)
            if (loc[s.Ri[q]] < 0) {
                s.t_rl.push_back(s.Ri[q]);
                s.t_rl.push_back(s.Rs[q]);
            }
        r[6] = (int32_t)(s.t_rl.size() / 2);
        for (int q = s.Rp[j]; q < s.Rp[j + 1]; ++q)
            if (in_clique(j) && loc[s.Ri[q]] >= 0 && !in_clique(s.Ri[q])) {
                s.t_rl.push_back(loc[s.Ri[q]]);
                s.t_rl.push_back(sloc[s.Rs[q]]);
            }
        r[7] = (int32_t)(s.t_rl.size() / 2);
        for (int q = s.Lp[j]; q < s.Lp[j + 1]; ++q) {
            int32_t* t = &s.t_slot[4 * (size_t)sloc[q]];
            t[0] = q;
            t[1] = loc[s.Li[q]];
            t[2] = (int32_t)jl;
        }
    }
    build_tail_ops(s);
}

// The upper levels of a spread launch, from mid_level on: the tail and below
// it the levels of at most kMidWidth nodes.  Their updates from lower levels
// (pulled in one pass), and the right-looking operations of those below the
// tail.  Unless `whole`, they end where the lists would pass kUpperTerms
// entries per slot of the factor.
UpperLists build_upper(const HostSym& s, bool whole)
{
    const int nlev = (int)s.level_ptr.size() - 1;
    const int64_t most = kUpperTerms * (int64_t)s.Li.size();
    // a level's right-looking operations and the updates that it pulls
    auto terms = [&](int l) {
        int64_t t = 0;
        for (int x = s.level_ptr[l]; x < s.level_ptr[l + 1]; ++x) {
            const int j = s.level_nodes[x];
            const int64_t d = s.Lp[j + 1] - s.Lp[j];
            t += d * (d + 1) / 2 + s.Up[s.Lp[j + 1]] - s.Up[s.Lp[j]];
        }
        return t;
    };
    UpperLists u;
    u.whole = true;
    int M = s.tail_level;
    int64_t total = 0;
    while (M > 0 && s.level_ptr[M] - s.level_ptr[M - 1] <= kMidWidth) {
        total += terms(M - 1);
        if (total > most) {
            u.whole = whole;
            if (!whole) break;
        }
        --M;
    }
    u.mid_level = M;
    const int x1 = s.level_ptr[M];  // first node (level order) of the upper levels
    // part 0: below the upper levels; part 1: the upper levels below the tail
    auto part = [&](int p) { return s.level[p] <= M ? 0 : s.level[p] <= s.tail_level ? 1 : 2; };
    u.node.reserve(8 * (size_t)(s.nn - x1));
    std::vector<int32_t> rest;  // part 1 of a list, appended to its part 0
    auto close = [&](std::vector<int32_t>& list) {
        const int32_t mid = (int32_t)(list.size() / 2);
        list.insert(list.end(), rest.begin(), rest.end());
        rest.clear();
        return mid;
    };
    for (int x = x1; x < s.nn; ++x) {
        const int j = s.level_nodes[x];
        // the tail alone pulls from the upper levels too (one workgroup)
        const int parts = part(j) == 2 ? 2 : 1;
        const int32_t r0 = (int32_t)(u.rl.size() / 2);
        for (int q = s.Rp[j]; q < s.Rp[j + 1]; ++q) {
            const int k = part(s.Ri[q]);
            if (k >= parts) continue;
            auto& list = k ? rest : u.rl;
            list.push_back(s.Ri[q]);
            list.push_back(s.Rs[q]);
        }
        const int32_t r1 = close(u.rl);
        u.node.insert(u.node.end(), {j, s.perm[j], s.ydiag[j], (int32_t)(u.rl.size() / 2), r0, r1,
                                     s.Lp[j], s.Lp[j + 1]});
        for (int q = s.Lp[j]; q < s.Lp[j + 1]; ++q) {
            const int32_t u0 = (int32_t)(u.upd.size() / 2);
            for (int v = s.Up[q]; v < s.Up[q + 1]; ++v) {
                const int k = part(s.owner[s.Ub[v]]);
                if (k >= parts) continue;
                auto& list = k ? rest : u.upd;
                list.push_back(s.Ua[v]);
                list.push_back(s.Ub[v]);
            }
            const int32_t u1 = close(u.upd);
            u.slot.insert(u.slot.end(), {q, s.perm[j], s.perm[s.Li[q]], s.ylo[q], s.yup[q], u0, u1,
                                         (int32_t)(u.upd.size() / 2)});
        }
    }
    if (M >= s.tail_level) {  // no level between
        u.op.assign(4, -1);
        u.next.assign(1, 0);
        return u;
    }
    LevelTerms lt((int32_t)s.Li.size(), s.nn);
    for (int l = M; l < s.tail_level && l < nlev; ++l) {
        lt.start();
        for (int x = s.level_ptr[l]; x < s.level_ptr[l + 1]; ++x) {
            const int j = s.level_nodes[x];
            lt.add_node(j, s.Lp[j], s.Lp[j + 1], [&](int32_t t) { return s.Li[t]; },
                        [&](int32_t k) { return s.Lp[k]; });
        }
        const int32_t op0 = (int32_t)u.next.size();
        // room for the padding; the destination -1 marks it
        u.op.resize(4 * ((size_t)op0 + lt.terms.size() + 63), -1);
        u.next.resize((size_t)op0 + lt.terms.size() + 63, 0);
        lt.place(64, [&](int32_t i, int32_t d, const LevelTerms::Term& q, int32_t next, int32_t) {
            int32_t* r = &u.op[4 * ((size_t)op0 + i)];
            r[0] = d;
            r[1] = q.a;
            r[2] = q.b;
            r[3] = q.j;
            u.next[(size_t)op0 + i] = next;
        });
        u.op.resize(4 * ((size_t)op0 + lt.total));
        u.next.resize((size_t)op0 + lt.total);
        u.lev.insert(u.lev.end(), {op0, lt.ns, lt.nd, 0, lt.ns2, lt.nd2, 0, 0});
    }
    // stands in for the first operation of an empty last level
    u.op.insert(u.op.end(), 4, -1);
    u.next.push_back(0);
    return u;
}

// The tail's operations by level (layouts documented with DevSym).
void build_tail_ops(HostSym& s)
{
    const int nT = (int)s.level_ptr.size() - 1 - s.tail_level;
    const int K = s.tail_nodes, TS = s.tail_slots, kf = K - s.tail_clique;
    const int x0 = s.level_ptr[s.tail_level];
    auto slot0 = [&](int jl) { return s.t_node[8 * (size_t)jl + 3]; };
    auto slot1 = [&](int jl) { return s.t_node[8 * (size_t)jl + 4]; };
    auto high = [&](int t) { return s.t_slot[4 * (size_t)t + 1]; };
    std::vector<int32_t> own(TS);
    for (int jl = 0; jl < K; ++jl)
        for (int t = slot0(jl); t < slot1(jl); ++t) own[t] = jl;
    s.t_lev.assign(8 * (size_t)nT, 0);
    LevelTerms lt(TS, K);
    auto put = [&](size_t i, uint32_t d, uint32_t a, uint32_t b, uint32_t j, uint32_t next) {
        s.t_op[2 * i] = (int32_t)(d | a << 12 | (b & 255u) << 24);
        s.t_op[2 * i + 1] = (int32_t)(b >> 8 | j << 4 | next << 16);
    };
    for (int tl = 0; tl < nT; ++tl) {
        lt.start();
        for (int x = s.level_ptr[s.tail_level + tl]; x < s.level_ptr[s.tail_level + tl + 1]; ++x)
            lt.add_node(x - x0, slot0(x - x0), slot1(x - x0), high, slot0);
        const size_t op0 = s.t_op.size() / 2;
        s.t_op.resize(s.t_op.size() + 2 * lt.terms.size());
        lt.place(1, [&](int32_t i, int32_t d, const LevelTerms::Term& q, int32_t next,
                        int32_t left) {
            put(op0 + i, d, q.a, q.b, q.j, i < lt.nd + lt.ns2 + lt.nd2 ? next : left);
        });
        int32_t* r = &s.t_lev[8 * (size_t)tl];
        r[0] = (int32_t)op0;
        r[1] = lt.ns;
        r[2] = lt.nd;
        r[3] = lt.ns2 | lt.nd2 << 16;
        r[6] = lt.ls | lt.ld << 16;
        s.tail_longs |= lt.ls + lt.ld > 0;
    }
    // backward: the slots whose higher neighbour is on the level and below
    // the clique, by that neighbour; S(j) lies on one path to the root, so a
    // node has at most one slot into a level
    std::vector<int32_t> ptr(K + 1, 0);
    for (int t = 0; t < TS; ++t) ++ptr[high(t) + 1];
    for (int k = 0; k < K; ++k) ptr[k + 1] += ptr[k];
    const size_t op0 = s.t_op.size() / 2;
    s.t_op.resize(s.t_op.size() + 2 * ((size_t)ptr[kf] + 1));
    for (int tl = 0; tl < nT; ++tl) {
        const int j0 = std::min(kf, s.level_ptr[s.tail_level + tl] - x0);
        const int j1 = std::min(kf, s.level_ptr[s.tail_level + tl + 1] - x0);
        s.t_lev[8 * (size_t)tl + 4] = (int32_t)op0 + ptr[j0];
        s.t_lev[8 * (size_t)tl + 5] = ptr[j1] - ptr[j0];
    }
    for (int t = 0; t < TS; ++t)
        if (high(t) < kf) put(op0 + ptr[high(t)]++, own[t], t, high(t), 0, 0);
    // stands in for the first operation of an empty level
    put(s.t_op.size() / 2 - 1, 0, 0, 0, 0, 0);
}

void build_subtrees(HostSym& s)
{
    const int nlev = (int)s.level_ptr.size() - 1;
    const int nn = s.nn;
    s.sub_cut = 0;
    s.sub_roots = 0;
    s.sub_idx.clear();
    s.sub_ptr.clear();
    s.sub_cum.clear();
    const int top = std::min(s.tail_level, nlev);
    if (top <= 0 || nn == 0) return;
    // roots below cut c (levels 0-based here): nodes p with level(p) < c
    // <= level(parent(p)), or without a parent; counted for every c at once
    std::vector<int64_t> diff(nlev + 2, 0);
    for (int p = 0; p < nn; ++p) {
        const int lp = s.level[p] - 1;
        const int hi = s.parent[p] >= 0 ? s.level[s.parent[p]] - 1 : nlev;
        diff[lp + 1] += 1;
        diff[hi + 1] -= 1;
    }
    int cut = 0;
    int64_t run = 0;
    for (int c = 1; c <= top; ++c) {
        run += diff[c];
        if (run >= kSubMinRoots) cut = c;
    }
    if (cut == 0) return;
    // each node's root (its parent is on a higher level, so top-down works)
    std::vector<int32_t> root(nn, -1);
    for (int l = cut - 1; l >= 0; --l)
        for (int x = s.level_ptr[l]; x < s.level_ptr[l + 1]; ++x) {
            const int p = s.level_nodes[x];
            const int q = s.parent[p];
            root[p] = (q < 0 || s.level[q] - 1 >= cut) ? p : root[q];
        }
    std::vector<int32_t> rid(nn, -1);
    int32_t R = 0;
    for (int p = 0; p < nn; ++p)
        if (root[p] == p) rid[p] = R++;
    // work of a node: its record, descendant list and slots with their pairs
    std::vector<int64_t> W(R, 0);
    for (int p = 0; p < nn; ++p) {
        if (root[p] < 0) continue;
        int64_t w = 4 + (s.Rp[p + 1] - s.Rp[p]);
        for (int q = s.Lp[p]; q < s.Lp[p + 1]; ++q) w += 2 + (s.Up[q + 1] - s.Up[q]);
        W[rid[root[p]]] += w;
    }
    int64_t tot = 0;
    for (int64_t w : W) tot += w;
    if (tot >= ((int64_t)1 << 30)) return;
    s.sub_cum.assign(R + 1, 0);
    for (int k = 0; k < R; ++k) s.sub_cum[k + 1] = s.sub_cum[k] + (int32_t)W[k];
    s.sub_idx.resize(s.level_ptr[cut]);
    s.sub_ptr.assign((size_t)cut * (R + 1), 0);
    for (int l = 0; l < cut; ++l) {
        const int b = s.level_ptr[l], e = s.level_ptr[l + 1];
        std::vector<int32_t> xs(e - b);
        for (int x = b; x < e; ++x) xs[x - b] = x;
        std::stable_sort(xs.begin(), xs.end(), [&](int32_t u, int32_t v) {
            return rid[root[s.level_nodes[u]]] < rid[root[s.level_nodes[v]]];
        });
        int32_t* ptr = &s.sub_ptr[(size_t)l * (R + 1)];
        for (int i = 0; i < e - b; ++i) {
            s.sub_idx[b + i] = xs[i];
            ++ptr[rid[root[s.level_nodes[xs[i]]]] + 1];
        }
        for (int k = 0; k < R; ++k) ptr[k + 1] += ptr[k];
    }
    s.sub_cut = cut;
    s.sub_roots = R;
}

// Lanes per node: enough lanes for the widest per-node loop of the level
// (its destinations, a quarter of its descendants), but no more than keeps
// one pass over the level within a 256-thread workgroup.
void default_mapping(HostSym& s)
{
    const int threads = 256;
    int nlev = (int)s.level_ptr.size() - 1;
    s.level_g.assign(std::max(nlev, 1), 1);
    for (int l = 0; l < nlev; ++l) {
        int w = s.level_ptr[l + 1] - s.level_ptr[l];
        int need = 1;
        for (int x = s.level_ptr[l]; x < s.level_ptr[l + 1]; ++x) {
            int p = s.level_nodes[x];
            int ns = s.Lp[p + 1] - s.Lp[p];
            int nr = (s.Rp[p + 1] - s.Rp[p] + 3) / 4;
            need = std::max(need, std::max(ns, nr));
        }
        int g = 1;
        while (g < need && g < 64) g <<= 1;
        int fit = 1;
        while (fit * 2 * w <= threads && fit < 64) fit <<= 1;
        s.level_g[l] = std::max(1, std::min(g, fit));
    }
}

}  // namespace pf
