// Reads "n m ordering budget", then m branches, and walks the lists of the LDS
// tail and of the upper levels as the kernels do: every update of the
// elimination has to come once, on its level, with its operands.
#include <algorithm>
#include <array>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <string>
#include <vector>

#include "pf_internal.h"

using namespace pf;
using Term = std::array<int, 5>;  // slot or diagonal, destination, a, b, j

static void need(bool ok, const char* what, int at)
{
    if (ok) return;
    std::printf("%s at %d\n", what, at);
    std::exit(1);
}

int main()
{
    int n, m, ordering;
    long long budget;
    if (std::scanf("%d %d %d %lld", &n, &m, &ordering, &budget) != 4) return 2;
    std::vector<int32_t> f(m), t(m);
    for (int e = 0; e < m; ++e)
        if (std::scanf("%d %d", &f[e], &t[e]) != 2) return 2;
    HostSym s;
    std::string msg;
    if (analyze(n, m, f.data(), t.data(), 0, ordering, s, msg) != 0) return 2;
    build_tail(s, budget);
    s.up = build_upper(s, true);
    const int nlev = (int)s.level_ptr.size() - 1, tl = s.tail_level, M = s.up.mid_level;
    const int x0 = s.level_ptr[tl], K = s.tail_nodes;
    std::map<int, int> loc, sloc;  // local node of a position, local slot of a slot
    for (int jl = 0; jl < K; ++jl) {
        need(s.t_node[8 * jl] == s.level_nodes[x0 + jl], "tail node", jl);
        loc[s.t_node[8 * jl]] = jl;
    }
    for (int q = 0; q < s.tail_slots; ++q) sloc[s.t_slot[4 * q]] = q;
    need((int)sloc.size() == s.tail_slots, "tail slots", 0);
    auto slot_of = [&](int j, int k) {
        const auto b = s.Li.begin() + s.Lp[j], e = s.Li.begin() + s.Lp[j + 1];
        const auto it = std::lower_bound(b, e, k);
        need(it != e && *it == k, "slot", j);
        return (int)(it - s.Li.begin());
    };
    // a level's updates, in local or global numbers
    auto wanted = [&](int l, bool local) {
        std::vector<Term> w;
        for (int x = s.level_ptr[l]; x < s.level_ptr[l + 1]; ++x) {
            const int j = s.level_nodes[x];
            for (int b = s.Lp[j]; b < s.Lp[j + 1]; ++b)
                for (int a = b; a < s.Lp[j + 1]; ++a) {
                    const bool diag = a == b;
                    const int d = diag ? s.Li[b] : slot_of(s.Li[b], s.Li[a]);
                    if (local)
                        w.push_back({diag, diag ? loc.at(d) : sloc.at(d), sloc.at(a), sloc.at(b),
                                     loc.at(j)});
                    else
                        w.push_back({diag, d, a, b, j});
                }
        }
        std::sort(w.begin(), w.end());
        return w;
    };
    size_t longest = 0;
    for (int l = tl; l < nlev; ++l) {
        const int32_t* h = &s.t_lev[8 * (size_t)(l - tl)];
        const int op0 = h[0], ns = h[1], nd = h[2], ns2 = h[3] & 0xffff, nd2 = h[3] >> 16;
        const int ls = h[6] & 0xffff, ld = h[6] >> 16;
        std::vector<Term> got;
        auto take = [&](int at, bool diag, int& next) {
            need(at >= 0 && 2 * (size_t)at + 1 < s.t_op.size(), "tail operation's place", l);
            const uint32_t x = s.t_op[2 * (size_t)at], y = s.t_op[2 * (size_t)at + 1];
            got.push_back({diag, (int)(x & 0xfff), (int)(x >> 12 & 0xfff),
                           (int)(x >> 24 | (y & 15) << 8), (int)(y >> 4 & 0xfff)});
            next = (int)(y >> 16);
        };
        for (int i = 0; i < nd; ++i) {
            const bool diag = i >= ns;
            const int k = diag ? i - ns : i;
            const size_t before = got.size();
            int next;
            take(op0 + i, diag, next);
            if (next) {
                need(k < (diag ? nd2 : ns2), "second operation", l);
                const int two = op0 + nd + (diag ? ns2 : 0) + k;
                need(two == op0 + i + next, "second operation's place", l);
                take(two, diag, next);
                if (next) {
                    int at = two + next, left;
                    take(at, diag, left);
                    while (left) {
                        const int was = left;
                        take(++at, diag, left);
                        need(left == was - 1, "operations left", l);
                    }
                }
            }
            const size_t c = got.size() - before;
            longest = std::max(longest, c);
            need((c > kTailSerial) == (k < (diag ? ld : ls)), "long destination", l);
            for (size_t g = before; g < got.size(); ++g)
                need(got[g][1] == got[before][1], "destination", l);
        }
        std::sort(got.begin(), got.end());
        need(got == wanted(l, true), "tail operations", l);
    }
    for (int l = M; l < tl; ++l) {
        const int32_t* h = &s.up.lev[8 * (size_t)(l - M)];
        const int op0 = h[0], ns = h[1], nd = h[2], ns2 = h[4], nd2 = h[5];
        std::vector<Term> got;
        for (int i = 0; i < nd; ++i) {
            const bool diag = i >= ns;
            int at = op0 + i;
            if (s.up.op[4 * (size_t)at] < 0) continue;  // padding
            const int k = diag ? i - ns : i;
            for (bool first = true;; first = false) {
                const int32_t* o = &s.up.op[4 * (size_t)at];
                got.push_back({diag, o[0], o[1], o[2], o[3]});
                const int next = s.up.next[at];
                if (!next) break;
                at += next;
                if (first)
                    need(k < (diag ? nd2 : ns2) && at == op0 + nd + (diag ? ns2 : 0) + k,
                         "second upper operation's place", l);
            }
        }
        std::sort(got.begin(), got.end());
        need(got == wanted(l, false), "upper operations", l);
    }
    // what the upper levels pull: from below them, and the tail from all below it
    const int x1 = s.level_ptr[M];
    size_t u = 0;
    for (int x = x1; x < s.nn; ++x) {
        const int32_t* r = &s.up.node[8 * (size_t)(x - x1)];
        const int j = r[0];
        auto below = [&](int i, int l) { return s.level[i] <= l; };
        auto check = [&](const std::vector<int32_t>& list, int a, int b, int c,
                         std::vector<std::pair<int, int>> all, auto&& of) {
            std::vector<std::pair<int, int>> got, want;
            const bool tail = s.level[j] > tl;
            for (int q = a; q < c; ++q) {
                got.push_back({list[2 * (size_t)q], list[2 * (size_t)q + 1]});
                need(below(of(got.back()), q < b ? M : tl), "part", j);
            }
            for (auto& p : all)
                if (below(of(p), tail ? tl : M)) want.push_back(p);
            std::sort(got.begin(), got.end());
            std::sort(want.begin(), want.end());
            need(got == want, "pulled", j);
        };
        std::vector<std::pair<int, int>> all;
        for (int q = s.Rp[j]; q < s.Rp[j + 1]; ++q) all.push_back({s.Ri[q], s.Rs[q]});
        check(s.up.rl, r[4], r[5], r[3], all, [](const std::pair<int, int>& p) { return p.first; });
        for (int q = s.Lp[j]; q < s.Lp[j + 1]; ++q, ++u) {
            const int32_t* t = &s.up.slot[8 * u];
            need(t[0] == q, "upper slot", j);
            all.clear();
            for (int v = s.Up[q]; v < s.Up[q + 1]; ++v) all.push_back({s.Ua[v], s.Ub[v]});
            check(s.up.upd, t[5], t[6], t[7], all,
                  [&](const std::pair<int, int>& p) { return s.owner[p.second]; });
        }
    }
    std::printf("ok: %d tail nodes, %d upper levels, longest %zu\n", K, tl - M, longest);
}
