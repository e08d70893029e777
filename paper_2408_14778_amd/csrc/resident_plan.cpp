// Host plan of the resident iteration: see resident_plan.hpp.
#include "resident_plan.hpp"

#include <algorithm>
#include <atomic>
#include <functional>
#include <memory>
#include <new>
#include <thread>

#include "sum_order.hpp"

namespace cfr {

namespace {

// Nodes that a bin should hold at least, when there are CUs to spare: below this its levels are
// all latency, and more workgroups only make the barrier dearer.
constexpr int64_t kBinNodes = 3000;

// Runs the jobs, each on a thread of its own where n (the nodes they go over) is large. False: one
// threw.
bool run_all(int64_t n, const std::vector<std::function<void()>>& jobs) {
    std::atomic<bool> failed{false};
    auto guarded = [&](const std::function<void()>& job) {
        try {
            job();
        } catch (...) {
            failed = true;
        }
    };
    std::vector<std::thread> pool;
    size_t i = 0;
    if (n >= 200000) try {
            for (; i + 1 < jobs.size(); ++i) pool.emplace_back([&, i] { guarded(jobs[i]); });
        } catch (...) {  // fewer threads
        }
    for (; i < jobs.size(); ++i) guarded(jobs[i]);
    for (std::thread& th : pool) th.join();
    return !failed;
}

int64_t columns(const ResSizes& z) { return z.players > 0 ? z.players : 1; }
int64_t planes(const ResSizes& z) { return z.players > 0 ? z.players : 2; }

}  // namespace

// Whether the public-block engine is the alternative.
bool block_game(const ResSizes& z) { return z.players == 0 && z.real_bytes == 4 && z.level_pure; }

int32_t resident_max_bins(const ResSizes& z) {
    return 1 + (z.forest ? kResRoundsForest : block_game(z) ? kResRoundsBlock : kResRounds) * (kResTeam - 1);
}

bool resident_fits(const ResSizes& z) {
    const int64_t room = kResLds * resident_max_bins(z);
    // what the bins of a team hold in all
    const int64_t team = z.real_bytes * ((columns(z) + 1) * z.nodes + planes(z) * z.decision) + 8 * z.decision;
    return z.decision > 0 && z.depth >= 1 && z.depth <= kResMaxDepth &&
           z.max_actions <= kResMaxActions && z.pairs + z.chance_pairs < (int64_t{1} << 28) &&
           z.players < 15 &&
           z.real_bytes * (columns(z) * z.nodes + planes(z) * z.decision) <= room &&
           (!block_game(z) || z.nodes <= (z.passes > 1 ? kResNodesBlock2 : kResNodesBlock)) &&
           // (bins that have no room to be uneven are not worth the search, nor the workspace: of a poker
           // game's in double precision 8.3 million nodes at 0.66 of the room fit, 9.1 at 0.73 do not)
           ((z.nodes <= 65535 && !z.forest) || (block_game(z) && !z.forest) || 4 * team <= 3 * room);
}

int64_t resident_max_table(const ResSizes& z) { return int64_t{resident_max_bins(z)} * (z.depth + 3); }
int64_t resident_max_roots(const ResSizes& z) { return std::min<int64_t>(kResTrunk, z.decision); }
int64_t resident_max_path(const ResSizes& z) { return kResPath * resident_max_roots(z); }

Layout forest_layout(const std::vector<Layout>& games) {
    const size_t n = games.size();
    Layout L;
    L.N = 1;
    std::vector<int64_t> h_base(n), q_base(n), q0_base(n), m_base(n);
    for (size_t g = 0; g < n; ++g) {
        h_base[g] = L.Hp; q_base[g] = L.Qp; q0_base[g] = L.Q0; m_base[g] = L.n_members;
        L.N += games[g].N; L.Hp += games[g].Hp; L.Qp += games[g].Qp; L.Q0 += games[g].Q0;
        L.n_members += games[g].n_members;
        L.D = std::max(L.D, games[g].D + 1);
    }
    // level l + 1: level l of every game, game after game
    std::vector<std::vector<int64_t>> base(n, std::vector<int64_t>(L.D + 1, 0));
    L.level_offset = {0};
    int64_t at = 1;
    for (int32_t l = 0; l <= L.D; ++l) {
        L.level_offset.push_back(static_cast<int32_t>(at));
        for (size_t g = 0; g < n; ++g) {
            base[g][l] = at;
            if (l <= games[g].D) at += games[g].level_offset[l + 1] - games[g].level_offset[l];
        }
    }
    L.parent.resize(L.N);
    L.child_begin.resize(L.N + 1);
    L.node_player.resize(L.N);
    L.node_infoset.resize(L.N);
    L.node_edge.resize(L.N);
    L.payoff.resize(L.N);
    L.q_offset.resize(L.Hp + 1);
    L.member_offset.resize(L.Hp + 1);
    L.infoset_player.resize(L.Hp);
    L.members.resize(L.n_members);
    L.parent[0] = L.node_infoset[0] = L.node_edge[0] = -1;
    L.node_player[0] = 0;
    L.payoff[0] = 0.0f;
    L.child_begin[0] = 1;
    L.child_begin[L.N] = static_cast<int32_t>(L.N);
    L.q_offset[L.Hp] = static_cast<int32_t>(L.Qp);
    L.member_offset[L.Hp] = static_cast<int32_t>(L.n_members);
    for (const Layout& G : games)
        L.chance_prob.insert(L.chance_prob.end(), G.chance_prob.begin(), G.chance_prob.end());
    const int32_t Qp = static_cast<int32_t>(L.Qp), Q0 = static_cast<int32_t>(L.Q0);
    for (size_t g = 0; g < n; ++g) {
        const Layout& G = games[g];
        for (int32_t l = 0; l <= G.D; ++l) {
            const int32_t lo = G.level_offset[l];
            const int32_t down = static_cast<int32_t>(base[g][l + 1]) - G.level_offset[l + 1];
            const int32_t up = l > 0 ? static_cast<int32_t>(base[g][l - 1]) - G.level_offset[l - 1] : 0;
            const int32_t here = static_cast<int32_t>(base[g][l]) - lo;
            for_ranges(G.level_offset[l + 1] - lo, [&, l, lo, down, up, here](int64_t i0, int64_t i1) {
                for (int64_t v = lo + i0; v < lo + i1; ++v) {
                    const int64_t i = v + here;
                    const int32_t e = G.node_edge[v];
                    L.parent[i] = l > 0 ? G.parent[v] + up : 0;
                    L.child_begin[i] = G.child_begin[v] + down;
                    L.node_player[i] = G.node_player[v];
                    L.node_infoset[i] = G.node_player[v] > 0
                                            ? G.node_infoset[v] + static_cast<int32_t>(h_base[g]) : -1;
                    L.node_edge[i] = l == 0 ? Qp + Q0 + static_cast<int32_t>(g)
                                     : e < G.Qp ? e + static_cast<int32_t>(q_base[g])
                                                : Qp + static_cast<int32_t>(q0_base[g] + (e - G.Qp));
                    L.payoff[i] = G.payoff[v];
                }
            });
        }
        for (int64_t h = 0; h < G.Hp; ++h) {
            const int64_t i = h_base[g] + h;
            L.q_offset[i] = G.q_offset[h] + static_cast<int32_t>(q_base[g]);
            L.member_offset[i] = G.member_offset[h] + static_cast<int32_t>(m_base[g]);
            L.infoset_player[i] = G.infoset_player[h];
            int32_t l = 0;
            for (int32_t m = G.member_offset[h]; m < G.member_offset[h + 1]; ++m) {
                const int32_t v = G.members[m];
                while (v >= G.level_offset[l + 1]) ++l;
                L.members[m_base[g] + m] = v - G.level_offset[l] + static_cast<int32_t>(base[g][l]);
            }
        }
    }
    L.Q0 += static_cast<int64_t>(n);
    L.chance_prob.resize(L.Q0, 1.0f);
    return L;
}

namespace {

bool plan_resident(const Layout& L, const std::vector<int32_t>& q_of, const ResSizes& z, ResPlan& P) {
    const int64_t N = L.N;
    const int32_t D = L.D;
    const int64_t cols = columns(z), pl = planes(z), real = z.real_bytes;
    P = ResPlan{};
    if (!resident_fits(z)) return false;
    // every node's level, and each level's largest fan-out of a chance node
    const std::unique_ptr<int8_t[]> level(new int8_t[N]);
    std::vector<int32_t> fan(D + 1, 1);
    for (int32_t l = 0; l <= D; ++l) {
        std::atomic<int32_t> most{1};
        const int32_t lo = L.level_offset[l];
        for_ranges(L.level_offset[l + 1] - lo, [&, l, lo](int64_t i0, int64_t i1) {
            int32_t k = 1;
            for (int64_t v = lo + i0; v < lo + i1; ++v) {
                level[v] = static_cast<int8_t>(l);
                if (L.node_player[v] == 0) k = std::max(k, L.child_begin[v + 1] - L.child_begin[v]);
            }
            for (int32_t seen = most; seen < k && !most.compare_exchange_weak(seen, k);) {
            }
        });
        fan[l] = most;
        if (fan[l] > kResMaxFan) return false;
    }
    int64_t con = 0;
    for (int64_t h = 0; h < L.Hp; ++h)
        con += static_cast<int64_t>(L.member_offset[h + 1] - L.member_offset[h]) *
               res_stride(L.q_offset[h + 1] - L.q_offset[h], z.real_bytes);
    if (con >= (int64_t{1} << 31)) return false;
    P.contributions = con;
    const int64_t nd = z.decision;
    // a bin's LDS: values and edge probabilities, reach and short records
    auto bin_bytes = [&](int64_t n, int64_t d) { return real * ((cols + 1) * n + pl * d) + 8 * d; };
    auto edge_of = [&](int64_t v) {
        const int32_t p = L.parent[v];
        if (L.node_player[p] == 0) return L.node_edge[v];
        const int32_t h = L.node_infoset[p];
        return q_of[h] + (L.node_edge[v] - L.q_offset[h]);
    };
    // owner of every node: its bin (0: the trunk); bins' roots in order
    std::vector<int32_t> roots, bin_root{0, 0}, in_trunk;
    std::unique_ptr<int32_t[]> sn, sd;
    std::vector<int8_t> trunk(N, 0);
    const int64_t solo = real * (cols * N + pl * nd + 3 * z.pairs + z.chance_pairs + con) + 16 * nd;
    if (N <= 65535 && solo <= kResLds) {
        P.mode = RES_SOLO;
        P.bins = 1;
        roots.push_back(0);
        bin_root = {0, 1};
    } else {
        // nodes and decision nodes of every subtree, level by level from below
        sn.reset(new int32_t[N]);
        sd.reset(new int32_t[N]);
        for (int32_t l = D; l >= 0; --l) {
            const int32_t lo = L.level_offset[l];
            for_ranges(L.level_offset[l + 1] - lo, [&, lo](int64_t i0, int64_t i1) {
                for (int64_t v = lo + i0; v < lo + i1; ++v) {
                    int32_t n = 1, d = L.node_player[v] >= 0 ? 1 : 0;
                    for (int32_t c = L.child_begin[v]; c < L.child_begin[v + 1]; ++c) {
                        n += sn[c];
                        d += sd[c];
                    }
                    sn[v] = n;
                    sd[v] = d;
                }
            });
        }
        int64_t first_want = std::min<int64_t>(kResTeam - 1, std::max<int64_t>(1, N / kBinNodes));
        // one XCD with the trunk
        if (first_want >= kResXcd && first_want < 2 * kResXcd) first_want = kResXcd - 1;
        bool found = false;
        // more bins until they fit: up to one per workgroup, then whole rounds of them
        for (int64_t want = first_want; want < resident_max_bins(z) && !found;
             want = want < kResTeam - 1 ? std::min<int64_t>(kResTeam - 1, want + want / 8 + 1)
                                        : want + kResTeam - 1) {
            // subtrees of at most a fraction of a bin: small ones balance, large ones leave a
            // small trunk
            const int64_t even = (N + want - 1) / want;
            // (then sizes between them: 2.58 million nodes fit one bin per workgroup at one of these
            // only, 58 us per iteration against 70 with two)
            std::vector<int64_t> sizes;
            for (const int64_t num : {2, 3})
                for (int64_t t = std::max<int64_t>(even / 16, 16); t * num / 2 <= even; t *= 2)
                    sizes.push_back(t * num / 2);
            for (size_t k = 0; k < sizes.size() && !found; ++k) {
                const int64_t t = sizes[k];
                // the trunk, level by level from the root
                roots.clear();
                for (int32_t v : in_trunk) trunk[v] = 0;
                in_trunk.assign(1, 0);
                trunk[0] = 1;
                int64_t tn = 1;
                int32_t deepest = 0;
                for (size_t i = 0; i < in_trunk.size() && tn <= 65535; ++i) {
                    const int32_t p = in_trunk[i];
                    for (int32_t v = L.child_begin[p]; v < L.child_begin[p + 1]; ++v) {
                        ++tn;
                        if (L.node_player[v] < 0) continue;
                        if (sn[v] > t) {
                            trunk[v] = 1;
                            in_trunk.push_back(v);
                        } else {
                            roots.push_back(v);
                            deepest = std::max<int32_t>(deepest, level[v]);
                        }
                    }
                }
                const int64_t td = static_cast<int64_t>(in_trunk.size());
                if (roots.size() < 2 || static_cast<int64_t>(roots.size()) > kResTrunk ||
                    deepest > kResPath || tn > 65535 || bin_bytes(tn, td) > kResLds)
                    continue;
                // by level and first edge: in the public-block order the members of an infoset
                // then lie in few bins
                std::sort(roots.begin(), roots.end(), [&](int32_t a, int32_t b) {
                    if (level[a] != level[b]) return level[a] < level[b];
                    const int32_t ea = edge_of(L.child_begin[a]), eb = edge_of(L.child_begin[b]);
                    return ea != eb ? ea < eb : a < b;
                });
                int64_t total = 0, most = 0, most_d = td;
                for (int32_t v : roots) {
                    total += sn[v];
                    most = std::max<int64_t>(most, sn[v]);
                    most_d = std::max<int64_t>(most_d, sd[v]);
                }
                for (int64_t cap = std::max((total + want - 1) / want, most); cap < 2 * total + 2;
                     cap += cap / 32 + 1) {
                    // every workgroup's arrays have room for `cap` nodes and for the decision nodes that
                    // LDS holds beside them; a bin ends at either (by nodes alone, 2.58 million nodes
                    // took two bins per workgroup: where many of them decide the bins overflowed)
                    const int64_t cap_n = std::max(cap, tn);
                    const int64_t cap_d = std::min<int64_t>(
                        65535, (kResLds - bin_bytes(cap_n, 0)) / bin_bytes(0, 1));
                    if (cap_n > 65535 || bin_bytes(cap_n, most_d) > kResLds) break;
                    bin_root.assign(1, 0);
                    int64_t n = 0, d = 0;
                    for (size_t i = 0; i < roots.size(); ++i) {
                        const int32_t v = roots[i];
                        if (i == 0 || n + sn[v] > cap || d + sd[v] > cap_d) {
                            bin_root.push_back(static_cast<int32_t>(i));
                            n = d = 0;
                        }
                        n += sn[v];
                        d += sd[v];
                    }
                    if (static_cast<int64_t>(bin_root.size()) - 1 <= want) {
                        found = true;
                        P.mode = RES_TEAM;
                        break;
                    }
                }
            }
        }
        if (!found) return false;
        P.bins = static_cast<int32_t>(bin_root.size());
        bin_root.push_back(static_cast<int32_t>(roots.size()));
        P.roots = static_cast<int32_t>(roots.size());
        for (int32_t v : roots) P.path_len = std::max<int32_t>(P.path_len, level[v]);
    }
    const bool team = P.mode == RES_TEAM;
    const int32_t W = D + 3;
    P.table.assign(static_cast<size_t>(P.bins) * W, Rec4{0, 0, 0, 0});
    P.root_rank.resize(P.roots);
    P.ext.resize(P.roots);
    P.path.assign(static_cast<size_t>(P.roots) * P.path_len, 0);
    std::vector<int32_t> glog(D + 1, 0);
    for (int32_t l = 0; l < D; ++l) {
        // lanes per chance node: the level's largest fan-out rounded up to a power of two, at most a
        // wavefront
        const int32_t nodes = L.level_offset[l + 1] - L.level_offset[l];
        const bool grouped = z.players > 0 && nodes <= kWideNodes;
        int32_t g = 0;
        while (g < 6 && (1 << g) < fan[l]) ++g;
        const bool wide = grouped && nodes <= kWideTop && fan[l] > 64;
        glog[l] = g | (grouped ? kResGrouped : 0) | (wide ? kResWide : 0);
    }
    // per node, set where it is read: its first contribution, local node and local rank
    std::unique_ptr<int32_t[]> slot, lnode, lrank;
    // chance products (rounded to float after every factor in single precision, as the level by
    // level launches form them): x at v's parent to v
    const auto chance_step = [&](double x, int64_t v) {
        if (L.node_player[L.parent[v]] != 0) return x;
        const int64_t i = L.node_edge[v] - L.Qp;
        return real == 8 ? x * L.chance_prob64[i]
                         : static_cast<double>(static_cast<float>(x) * L.chance_prob[i]);
    };
    const auto chance_product = [&](int64_t v) {
        int64_t path[kResMaxDepth];
        int32_t n = 0;
        for (; v > 0; v = L.parent[v]) path[n++] = v;
        double x = 1.0;
        while (n > 0) x = chance_step(x, path[--n]);
        return x;
    };
    // infosets: the trunk's first, then by pair (through the pairs: no sort); their contribution
    // slots in that order
    const auto number_sets = [&] {
        std::vector<int8_t> of_trunk(L.Hp, 0);
        if (team)
            for (int32_t v : in_trunk)
                if (L.node_player[v] > 0) of_trunk[L.node_infoset[v]] = 1;
        std::vector<int32_t> order, at_pair(L.Qp, -1);
        order.reserve(L.Hp);
        for (int64_t h = 0; h < L.Hp; ++h) at_pair[q_of[h]] = static_cast<int32_t>(h);
        for (int pass = 1; pass >= 0; --pass)
            for (int64_t q = 0; q < L.Qp; ++q)
                if (at_pair[q] >= 0 && of_trunk[at_pair[q]] == pass) order.push_back(at_pair[q]);
        P.sets.resize(L.Hp);
        std::vector<int32_t> base(L.Hp);
        int64_t at = 0;
        for (int64_t i = 0; i < L.Hp; ++i) {
            const int32_t h = order[i];
            const int32_t n = L.member_offset[h + 1] - L.member_offset[h];
            const int32_t k = L.q_offset[h + 1] - L.q_offset[h];
            P.trunk_sets += of_trunk[h];
            P.max_actions = std::max(P.max_actions, k);
            P.sets[i] = Rec4{q_of[h], static_cast<int32_t>(at), n, k | (L.infoset_player[h] << 24)};
            base[h] = static_cast<int32_t>(at);
            at += static_cast<int64_t>(n) * res_stride(k, z.real_bytes);
        }
        slot.reset(new int32_t[N]);
        for_ranges(L.n_members, [&](int64_t m0, int64_t m1) {
            int64_t h = std::upper_bound(L.member_offset.begin(), L.member_offset.end(), m0) -
                        L.member_offset.begin() - 1;
            for (int64_t m = m0; m < m1; ++m) {
                while (m >= L.member_offset[h + 1]) ++h;
                const int32_t k = L.q_offset[h + 1] - L.q_offset[h];
                slot[L.members[m]] = base[h] + static_cast<int32_t>(m - L.member_offset[h]) *
                                                   res_stride(k, z.real_bytes);
            }
        });
        P.mean_members = L.Hp > 0 ? static_cast<int32_t>(L.n_members / L.Hp) : 0;
        P.waves = gather_waves(L.n_members, L.Hp);
    };
    std::vector<std::function<void()>> jobs;
    jobs.emplace_back([&] { P.rec.resize(nd); });
    jobs.emplace_back([&] { P.slot.assign(nd, 0); });
    jobs.emplace_back([&] { P.reach_c.resize(nd); });
    jobs.emplace_back([&] {
        P.rank_node.resize(nd);
        P.node.resize(N + P.roots);
    });
    jobs.emplace_back([&] {
        lnode.reset(new int32_t[N]);
        lrank.reset(new int32_t[N]);
    });
    jobs.emplace_back(number_sets);
    if (!run_all(N, jobs)) return false;
    // where each bin's ranks and nodes begin
    std::vector<int64_t> rbase_of(P.bins, 0), nbase_of(P.bins, 0);
    if (team) {
        int64_t rb = static_cast<int64_t>(in_trunk.size()), nb = 1;
        for (int32_t v : in_trunk) nb += L.child_begin[v + 1] - L.child_begin[v];
        for (int32_t b = 1; b < P.bins; ++b) {
            rbase_of[b] = rb;
            nbase_of[b] = nb;
            for (int32_t x = bin_root[b]; x < bin_root[b + 1]; ++x) {
                rb += sd[roots[x]];
                nb += sn[roots[x]];
            }
        }
    }
    // the bins: local numbers level by level, records (the trunk first: its leaves are numbered
    // again in their own bins; the others on several threads)
    std::vector<int32_t> bin_nodes(P.bins, 0), bin_ranks(P.bins, 0);
    auto fill_bin = [&](int32_t b) {
        std::vector<int32_t> now, next;
        const int64_t rbase = rbase_of[b], nbase = nbase_of[b];
        Rec4* t = P.table.data() + static_cast<size_t>(b) * W;
        const bool is_trunk = team && b == 0;
        int32_t r0 = is_trunk ? 0 : team ? bin_root[b] : 0, r1 = is_trunk ? 0 : team ? bin_root[b + 1] : 1;
        const int32_t first_root = r0, end_root = r1;
        int32_t n = 0, r = 0, l0 = -1, l1 = -1;
        now.clear();
        for (int32_t l = 0; l <= D; ++l) {
            // the children of the bin's nodes of the level above, then the roots of this one
            next.clear();
            for (int32_t p : now)
                for (int32_t c = L.child_begin[p]; c < L.child_begin[p + 1]; ++c) next.push_back(c);
            if (is_trunk && l == 0) next.push_back(0);
            while (r0 < r1 && level[roots[r0]] == l) next.push_back(roots[r0++]);
            t[l] = Rec4{n, r, l < D ? glog[l] : 0, 0};
            for (int32_t v : next) {
                lnode[v] = n;
                P.node[nbase + n++] = v;
            }
            // (the roots of other bins are leaves of the trunk)
            now.clear();
            for (int32_t v : next)
                if (L.node_player[v] >= 0 && (!is_trunk || trunk[v])) now.push_back(v);
            for (int32_t v : now)
                if (L.node_player[v] > 0) lrank[v] = r++;
            for (int32_t v : now)
                if (L.node_player[v] == 0) {
                    lrank[v] = r++;
                    ++t[l].w;
                }
            for (int32_t v : now) {
                const bool apart = v == 0 || (team && !is_trunk && trunk[L.parent[v]]);
                P.reach_c[rbase + lrank[v]] =
                    apart ? chance_product(v) : chance_step(P.reach_c[rbase + lrank[L.parent[v]]], v);
            }
            if (!now.empty()) {
                l0 = l0 < 0 ? l : l0;
                l1 = l;
            }
        }
        if (is_trunk)
            for (int32_t x = 0; x < P.roots; ++x) P.ext[x] = lnode[roots[x]];
        t[D + 1] = Rec4{static_cast<int32_t>(rbase), n, r, static_cast<int32_t>(nbase)};
        t[D + 2] = Rec4{l0, l1 - l0 + 1, team ? first_root : 0, team ? end_root : 0};
        bin_nodes[b] = n;
        bin_ranks[b] = r;
        for (int32_t i = 0; i < n; ++i) {
            const int64_t v = P.node[nbase + i];
            if (L.node_player[v] < 0 || (is_trunk && !trunk[v])) continue;
            const int32_t d = lrank[v];
            const int32_t c0 = L.child_begin[v], k = L.child_begin[v + 1] - c0;
            const int32_t who = L.node_player[v];
            const int32_t p = L.parent[v];
            // a subtree's root has no parent in its bin
            const bool root = v > 0 && team && !is_trunk && trunk[p];
            const uint32_t actor = root ? 15u : v == 0 ? 15u : static_cast<uint32_t>(L.node_player[p]);
            Rec4& q = P.rec[rbase + d];
            q.x = static_cast<int32_t>(static_cast<uint32_t>(lnode[c0]) |
                                       (static_cast<uint32_t>(lnode[v]) << 16));
            q.y = static_cast<int32_t>(static_cast<uint32_t>(edge_of(c0)) |
                                       (static_cast<uint32_t>(who) << 28));
            q.z = static_cast<int32_t>((root || v == 0 ? 0u : static_cast<uint32_t>(lrank[p])) |
                                       (actor << 16) | (static_cast<uint32_t>(k) << 20));
            q.w = v == 0 ? 0 : edge_of(v);
            P.slot[rbase + d] = who > 0 ? slot[v] : 0;
            P.rank_node[rbase + d] = static_cast<int32_t>(v);
        }
        if (team && !is_trunk)
            for (int32_t x = first_root; x < end_root; ++x) {
                int64_t u = roots[x];
                P.root_rank[x] = lrank[u];
                for (int32_t q = level[u] - 1; q >= 0; --q) {
                    const int32_t p = L.parent[u];
                    P.path[static_cast<size_t>(q) * P.roots + x] =
                        static_cast<int32_t>(static_cast<uint32_t>(edge_of(u)) |
                                             (static_cast<uint32_t>(L.node_player[p]) << 28));
                    u = p;
                }
            }
    };
    fill_bin(0);
    std::atomic<int32_t> at_bin{1};
    std::atomic<bool> failed{false};
    auto work = [&] {
        try {
            for (int32_t b; (b = at_bin.fetch_add(8)) < P.bins;)
                for (int32_t i = b; i < std::min(P.bins, b + 8); ++i) fill_bin(i);
        } catch (...) {  // out of memory: the game is not resident
            failed = true;
        }
    };
    std::vector<std::thread> pool;
    if (N > 100000)
        try {
            for (unsigned i = 1; i < std::min(8u, std::thread::hardware_concurrency()); ++i)
                pool.emplace_back(work);
        } catch (...) {  // fewer threads
        }
    work();
    for (std::thread& th : pool) th.join();
    if (failed) return false;
    for (int32_t b = 0; b < P.bins; ++b) {
        P.max_nodes = std::max(P.max_nodes, bin_nodes[b]);
        P.max_ranks = std::max(P.max_ranks, bin_ranks[b]);
    }
    return true;
}

}  // namespace

bool build_resident(const Layout& L, const std::vector<int32_t>& q_of, const ResSizes& z,
                    ResPlan& P) {
    try {
        if (plan_resident(L, q_of, z, P)) return true;
    } catch (const std::bad_alloc&) {
    }
    P = ResPlan{};
    return false;
}

}  // namespace cfr
