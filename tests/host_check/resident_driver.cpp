// Host-only driver of the resident iteration's plan, built by tests/test_host_resident.py with the
// address and undefined-behaviour sanitizers. Every game of a file (the format of plan_driver.cpp;
// infosets of more than two players: a general-sum game) is planned in both precisions, and the
// two-player ones together as a batch; every record of every bin is followed as the kernel follows it and
// compared with the canonical layout. With "starve" as a second argument, the first games are planned
// with the n-th allocation failing, for every n: the planner then says that the game is not resident.
#include <atomic>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <new>
#include <string>
#include <vector>

#include "../../include/cfr.h"
#include "../../paper_2408_14778_amd/csrc/flatten.hpp"
#include "../../paper_2408_14778_amd/csrc/resident_plan.hpp"
#include "../../paper_2408_14778_amd/csrc/sum_order.hpp"

using namespace cfr;

namespace {
std::atomic<int64_t> g_left{-1};  // allocations until one fails (negative: none does)
}

void* operator new(std::size_t n) {
    int64_t left = g_left.load();
    while (left >= 0 && !g_left.compare_exchange_weak(left, left - 1)) {
    }
    void* p = left == 0 ? nullptr : std::malloc(n > 0 ? n : 1);
    if (p == nullptr) throw std::bad_alloc();
    return p;
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }

namespace {

struct GameData {
    std::vector<int32_t> parent, node_infoset, node_action, nact;
    std::vector<int8_t> player;
    std::vector<double> chance, payoff;
    cfr_game g{};
};

template <class T>
bool read(FILE* f, std::vector<T>& v, int64_t n) {
    v.resize(static_cast<size_t>(n));
    return n == 0 || std::fread(v.data(), sizeof(T), static_cast<size_t>(n), f) == static_cast<size_t>(n);
}

int64_t g_bad = 0;
#define EXPECT(ok)                                                                             \
    do {                                                                                       \
        if (!(ok) && g_bad++ < 20) std::printf("line %d: %s\n", __LINE__, #ok);                \
    } while (0)

ResSizes sizes_of(const Layout& L, int32_t players, int32_t real, bool forest) {
    ResSizes z;
    z.nodes = L.N;
    for (int64_t v = 0; v < L.N; ++v) z.decision += L.node_player[v] >= 0;
    z.members = L.n_members; z.infosets = L.Hp; z.pairs = L.Qp; z.chance_pairs = L.Q0;
    z.depth = L.D; z.players = players; z.real_bytes = real; z.forest = forest;
    z.max_actions = 1;
    for (int64_t h = 0; h < L.Hp; ++h) z.max_actions = std::max(z.max_actions, L.q_offset[h + 1] - L.q_offset[h]);
    z.level_pure = L.level_pure;
    return z;
}

void check_plan(const Layout& L, const ResSizes& z, const std::vector<int32_t>& q_of, const ResPlan& P) {
    const int32_t D = L.D, W = D + 3;
    const bool team = P.mode == RES_TEAM;
    const int64_t cols = z.players > 0 ? z.players : 1, planes = z.players > 0 ? z.players : 2;
    auto edge_of = [&](int64_t v) {
        const int32_t p = L.parent[v];
        return L.node_player[p] == 0 ? L.node_edge[v]
                                     : q_of[L.node_infoset[p]] + L.node_edge[v] - L.q_offset[L.node_infoset[p]];
    };
    std::vector<int32_t> level(L.N, 0);
    for (int32_t l = 0; l <= D; ++l)
        for (int32_t v = L.level_offset[l]; v < L.level_offset[l + 1]; ++v) level[v] = l;
    // array bounds and LDS
    EXPECT(static_cast<int64_t>(P.table.size()) == int64_t{P.bins} * W && static_cast<int64_t>(P.table.size()) <= resident_max_table(z));
    EXPECT(P.roots <= resident_max_roots(z) && static_cast<int64_t>(P.path.size()) <= resident_max_path(z));
    EXPECT(static_cast<int64_t>(P.node.size()) == L.N + P.roots && P.path_len <= kResPath);
    EXPECT(static_cast<int64_t>(P.rec.size()) == z.decision && P.slot.size() == P.rec.size() &&
           P.reach_c.size() == P.rec.size() && P.rank_node.size() == P.rec.size());
    EXPECT(team ? P.bins >= 2 : P.bins == 1 && P.roots == 0);
    const int64_t reals = cols * P.max_nodes + planes * P.max_ranks +
                          (team ? P.max_nodes : 3 * z.pairs + z.chance_pairs + P.contributions);
    EXPECT(z.real_bytes * reals + (team ? 8 : 16) * int64_t{P.max_ranks} <= kResLds);
    // infosets and contribution slots
    std::vector<int32_t> set_of(L.Hp, -1), slot(L.N, -1), of_pair(L.Qp, -1);
    for (int64_t h = 0; h < L.Hp; ++h) of_pair[q_of[h]] = static_cast<int32_t>(h);
    int64_t at = 0;
    for (int64_t i = 0; i < L.Hp; ++i) {
        const Rec4& s = P.sets.at(i);
        const int32_t h = of_pair.at(s.x), k = L.q_offset[h + 1] - L.q_offset[h];
        EXPECT(h >= 0 && set_of[h] < 0);
        set_of[h] = static_cast<int32_t>(i);
        EXPECT(s.y == at && s.z == L.member_offset[h + 1] - L.member_offset[h]);
        EXPECT((s.w & 0xFFFFFF) == k && (s.w >> 24) == L.infoset_player[h]);
        EXPECT(s.y % (16 / z.real_bytes) == 0 && res_stride(k, z.real_bytes) >= k + 1);
        for (int32_t j = 0; j < s.z; ++j) slot[L.members[L.member_offset[h] + j]] = s.y + j * res_stride(k, z.real_bytes);
        at += int64_t{s.z} * res_stride(k, z.real_bytes);
    }
    EXPECT(at == P.contributions && P.waves == gather_waves(L.n_members, L.Hp));
    // bins
    std::vector<int8_t> seen(L.N, 0), placed(L.N, 0), in_trunk(L.Hp, 0);
    int64_t ranks = 0, nodes = 0;
    int32_t root_end = 0;
    for (int32_t b = 0; b < P.bins; ++b) {
        const Rec4* t = P.table.data() + static_cast<size_t>(b) * W;
        const int64_t rbase = t[D + 1].x, nbase = t[D + 1].w;
        const int32_t n = t[D + 1].y, r = t[D + 1].z, l0 = t[D + 2].x, nl = t[D + 2].y;
        const bool trunk = team && b == 0;
        EXPECT(rbase == ranks && nbase == nodes && n <= P.max_nodes && r <= P.max_ranks && n <= 65535);
        ranks += r;
        nodes += n;
        if (team && b > 0) EXPECT(t[D + 2].z == root_end && t[D + 2].w > root_end);
        if (team && b > 0) root_end = t[D + 2].w;
        if (!team) EXPECT(t[D + 2].z == 0 && t[D + 2].w == 0);
        for (int32_t i = 0; i < n; ++i) placed.at(P.node.at(nbase + i)) += trunk ? 0 : 1;
        for (int32_t d = 0; d < r; ++d) {
            const int64_t x = rbase + d, v = P.rank_node.at(x);
            const Rec4& q = P.rec.at(x);
            const uint32_t ux = q.x, uy = q.y, uz = q.z;
            const int32_t own = ux >> 16, c0 = ux & 0xFFFF, who = uy >> 28, e0 = uy & 0x0FFFFFFF;
            const int32_t pr = uz & 0xFFFF, actor = (uz >> 16) & 15, k = uz >> 20, l = level[v];
            ++seen[v];
            EXPECT(L.node_player[v] >= 0 && own < n && P.node[nbase + own] == v);
            EXPECT(own >= t[l].x && own < t[l + 1].x + (l == D ? n : 0));
            EXPECT(k == L.child_begin[v + 1] - L.child_begin[v] && who == L.node_player[v]);
            for (int32_t a = 0; a < k; ++a)
                EXPECT(c0 + a < n && P.node[nbase + c0 + a] == L.child_begin[v] + a &&
                       edge_of(L.child_begin[v] + a) == e0 + a);
            EXPECT(l >= l0 && l < l0 + nl && d >= t[l].y && d < t[l + 1].y + (l == D ? r : 0));
            EXPECT((d >= t[l + 1].y - t[l].w) == (who == 0));
            if (actor != 15) {
                EXPECT(pr < d && P.rank_node[rbase + pr] == L.parent[v] && actor == L.node_player[L.parent[v]]);
                EXPECT(q.w == edge_of(v));
            } else {
                EXPECT(v == 0 || (team && !trunk && seen[L.parent[v]] == 1));
            }
            if (who > 0) EXPECT(P.slot[x] == slot[v] && slot[v] >= 0);
            if (who > 0 && trunk) in_trunk[L.node_infoset[v]] = 1;
            double rc = 1.0;
            std::vector<int64_t> up;
            for (int64_t u = v; u > 0; u = L.parent[u]) up.push_back(u);
            for (size_t i = up.size(); i-- > 0;)
                if (L.node_player[L.parent[up[i]]] == 0) {
                    const int64_t c = L.node_edge[up[i]] - L.Qp;
                    rc = z.real_bytes == 8 ? rc * L.chance_prob64[c]
                                           : double{static_cast<float>(rc) * L.chance_prob[c]};
                }
            EXPECT(P.reach_c[x] == rc);
        }
        // the order of each level's sums
        for (int32_t l = 0; l < D; ++l) {
            const int32_t in_level = L.level_offset[l + 1] - L.level_offset[l], s = t[l].z;
            int32_t fan = 1;
            for (int32_t v = L.level_offset[l]; v < L.level_offset[l + 1]; ++v)
                if (L.node_player[v] == 0) fan = std::max(fan, L.child_begin[v + 1] - L.child_begin[v]);
            const bool grouped = z.players > 0 && in_level <= kWideNodes;
            EXPECT(((s & kResGrouped) != 0) == grouped);
            EXPECT(((s & kResWide) != 0) == (grouped && in_level <= kWideTop && fan > 64));
            EXPECT((s & kResLanes) <= 6 && (1 << (s & kResLanes)) >= std::min(fan, 64));
        }
        for (int32_t x = t[D + 2].z; x < t[D + 2].w; ++x) {
            const int64_t root = P.rank_node.at(rbase + P.root_rank.at(x));
            EXPECT(((static_cast<uint32_t>(P.rec[rbase + P.root_rank[x]].z) >> 16) & 15) == 15);
            EXPECT(P.node.at(P.ext.at(x)) == root);  // a leaf of the trunk, which is bin 0
            int64_t u = root;
            for (int32_t i = P.path_len - 1; i >= 0; --i) {
                const uint32_t e = P.path[static_cast<size_t>(i) * P.roots + x];
                if (i >= level[root]) {
                    EXPECT(e == 0);
                    continue;
                }
                EXPECT(static_cast<int32_t>(e & 0x0FFFFFFF) == edge_of(u) &&
                       static_cast<int32_t>(e >> 28) == L.node_player[L.parent[u]]);
                u = L.parent[u];
            }
            EXPECT(u == 0);
        }
    }
    EXPECT(ranks == z.decision && nodes == L.N + P.roots && root_end == P.roots);
    for (int64_t v = 0; v < L.N; ++v) {
        EXPECT(seen[v] == (L.node_player[v] >= 0 ? 1 : 0));
        // every node in a bin of its own but the trunk's, which come once there
        if (!team) EXPECT(placed[v] == 1);
        else EXPECT(placed[v] <= 1);
    }
    for (int64_t h = 0; h < L.Hp; ++h) EXPECT((set_of[h] < P.trunk_sets) == (in_trunk[h] != 0));
}

int32_t g_solo = 0, g_team = 0, g_none = 0;

void plan_and_check(const Layout& L, int32_t players, int32_t real, bool forest) {
    const ResSizes z = sizes_of(L, players, real, forest);
    const std::vector<int32_t> q_of(L.q_offset.begin(), L.q_offset.begin() + L.Hp);
    ResPlan P;
    if (!build_resident(L, q_of, z, P)) {
        EXPECT(P.rec.empty() && P.bins == 0);
        ++g_none;
        return;
    }
    ++(P.mode == RES_SOLO ? g_solo : g_team);
    check_plan(L, z, q_of, P);
}

// Plans with allocation n failing, for n = 0, 1, .. (in growing steps past 200) until none fails.
void starve(const Layout& L, int32_t players, int32_t real) {
    const ResSizes z = sizes_of(L, players, real, false);
    const std::vector<int32_t> q_of(L.q_offset.begin(), L.q_offset.begin() + L.Hp);
    ResPlan full;
    const bool fits = build_resident(L, q_of, z, full);
    for (int64_t n = 0;; n += 1 + n / 200) {
        ResPlan P;
        g_left = n;
        const bool ok = build_resident(L, q_of, z, P);
        const bool failed = g_left.exchange(-1) < 0;
        EXPECT(ok ? P.rec.size() == full.rec.size() && P.bins == full.bins : P.rec.empty() && P.bins == 0);
        if (!failed) {
            EXPECT(ok == fits);
            break;
        }
    }
}

}  // namespace

int main(int argc, char** argv) {
    FILE* f = argc >= 2 ? std::fopen(argv[1], "rb") : nullptr;
    int32_t n_games = 0;
    if (f == nullptr || std::fread(&n_games, 4, 1, f) != 1) return 2;
    const bool starved = argc > 2 && std::string(argv[2]) == "starve";
    std::vector<Layout> batch;
    for (int32_t i = 0; i < n_games; ++i) {
        GameData d;
        int64_t n = 0, nc = 0;
        int32_t h = 0;
        if (std::fread(&n, 8, 1, f) != 1 || !read(f, d.parent, n) || !read(f, d.node_infoset, n) ||
            !read(f, d.node_action, n) || std::fread(&h, 4, 1, f) != 1 || !read(f, d.player, h) ||
            !read(f, d.nact, h) || std::fread(&nc, 8, 1, f) != 1 || !read(f, d.chance, nc) ||
            !read(f, d.payoff, n))
            return 2;
        if (d.chance.empty()) d.chance.push_back(0.0);
        d.g.n_nodes = n;
        d.g.parent = d.parent.data();
        d.g.node_infoset = d.node_infoset.data();
        d.g.node_action = d.node_action.data();
        d.g.n_infosets = h;
        d.g.infoset_player = d.player.data();
        d.g.infoset_num_actions = d.nact.data();
        d.g.chance_prob = d.chance.data();
        d.g.payoff_u1 = d.payoff.data();
        int32_t players = 0;
        for (const int8_t p : d.player) players = std::max<int32_t>(players, p);
        const bool general = players > 2;
        for (const bool f64 : {false, true}) {
            Layout L;
            std::string err;
            if (flatten(d.g, L, err, f64, general ? players : 2) != CFR_OK) return 1;
            if (starved) {
                starve(L, general ? players : 0, f64 ? 8 : 4);
                continue;
            }
            plan_and_check(L, general ? players : 0, f64 ? 8 : 4, false);
            if (!general) plan_and_check(L, 2, f64 ? 8 : 4, false);  // as a general-sum game
            if (!f64 && !general && L.level_pure) batch.push_back(std::move(L));
        }
    }
    std::fclose(f);
    if (!starved) {
        plan_and_check(forest_layout(batch), 0, 4, true);
        plan_and_check(forest_layout({batch.front()}), 0, 4, true);
        plan_and_check(forest_layout({batch.back(), batch.front()}), 0, 4, true);
    }
    std::printf("%d of one workgroup, %d of teams, %d not resident, %lld mismatches\n%s\n", g_solo, g_team,
                g_none, static_cast<long long>(g_bad), g_bad == 0 ? "ok" : "bad");
    return g_bad == 0 ? 0 : 1;
}
