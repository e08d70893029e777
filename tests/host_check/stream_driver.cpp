// Host-only driver of the out-of-core stream's plan and of a batch joined under one root, built by
// tests/test_host_stream.py with the address and undefined-behaviour sanitizers. Every game of a file
// (the format of plan_driver.cpp) is cut at every level with several window sizes in both
// precisions; every record of every run is decoded as the kernel decodes it (bits, codes, children
// by running sums of fan-outs) and compared with the canonical node it stands for, and every node
// from the first cut down must come once. The games' batch layout is compared with their own.
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

#include "../../include/cfr.h"
#include "../../paper_2408_14778_amd/csrc/flatten.hpp"
#include "../../paper_2408_14778_amd/csrc/resident_plan.hpp"
#include "../../paper_2408_14778_amd/csrc/stream_plan.hpp"

using namespace cfr;

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
void expect(bool ok) { g_bad += ok ? 0 : 1; }

int32_t code_of(const Layout& L, int64_t v) {
    return L.node_player[v] < 0 ? -1
           : L.node_player[v] > 0 ? L.node_infoset[v]
                                  : static_cast<int32_t>(L.Hp) + L.node_infoset[v];
}
int32_t fan(const Layout& L, int32_t code) {
    const int64_t c = code - L.Hp;
    return c < 0 ? L.q_offset[code + 1] - L.q_offset[code] : L.cq_offset[c + 1] - L.cq_offset[c];
}

template <class W, class F>
void check_stream(const Layout& L, const PartPlan& P, const StreamPlan& S, const std::vector<W>& words,
                  const std::vector<F>& pay) {
    std::vector<int8_t> seen(L.N, 0);
    const int32_t nl = S.split - S.cut + 1;
    expect(S.window <= P.window && static_cast<int64_t>(words.size()) == S.words);
    int64_t cut_next = L.level_offset[S.cut];
    for (int32_t g = 0; g < S.groups; ++g) {
        const size_t at = static_cast<size_t>(g) * nl;
        // canonical first node of each level of the group; local ids follow by level
        std::vector<int64_t> first{cut_next};
        expect(S.id[at] == cut_next);
        for (int32_t i = 1; i < nl; ++i) first.push_back(L.child_begin[first[i - 1]]);
        cut_next += S.count[at];
        for (int32_t i = 0; i < nl; ++i)
            expect(S.id[at + i] >= (i == 0 ? 0 : S.base) &&
                   S.id[at + i] + S.count[at + i] <= S.base + (i == 0 ? 0 : S.window));
        for (int32_t i = 0; i + 1 < nl; ++i)
            for (int32_t j = 0; j < S.count[at + i]; ++j) {
                const int64_t v = first[i] + j, q = S.rec[at + i] + j;
                ++seen[v];
                expect(S.mid_code.at(q) == code_of(L, v));
                if (S.mid_code[q] < 0) expect(static_cast<F>(S.mid_pay.at(q)) == pay[v]);
                else expect(S.mid_child.at(q) - S.id[at + i + 1] == L.child_begin[v] - first[i + 1]);
            }
        int64_t id = S.id[at + nl - 1];
        for (int32_t u = S.unit0[g]; u < S.unit0[g + 1]; ++u) {
            const StreamUnit& U = S.units.at(u);
            expect(U.id0 == id && U.n <= S.max_unit && U.n <= kStreamMax && U.at % kStreamPart == 0);
            const int64_t root = first[nl - 1] + (id - S.id[at + nl - 1]);
            id += U.roots;
            // the run's canonical nodes, breadth first
            std::vector<int64_t> node;
            for (int64_t x = root, y = root + U.roots; x < y;) {
                for (int64_t v = x; v < y; ++v) node.push_back(v);
                const int64_t cx = L.child_begin[x], cy = L.child_begin[y];
                x = cx;
                y = cy;
            }
            expect(static_cast<int32_t>(node.size()) == U.n);
            const int64_t bit_words = ((((U.n + 31) / 32 * 4) + static_cast<int64_t>(sizeof(W)) - 1) /
                                           static_cast<int64_t>(sizeof(W)) + kStreamPart - 1) /
                                      kStreamPart * kStreamPart;
            std::vector<uint32_t> bits((U.n + 31) / 32);
            std::memcpy(bits.data(), &words.at(U.at), bits.size() * 4);
            int64_t child = U.roots;
            for (int32_t i = 0; i < U.n; ++i) {
                const int64_t v = node.at(i);
                const W w = words.at(U.at + bit_words + i);
                ++seen[v];
                const bool decision = (bits[i / 32] >> (i % 32)) & 1;
                expect(decision == (L.node_player[v] >= 0));
                if (decision) {
                    expect(static_cast<int32_t>(w) == code_of(L, v));
                    expect(node.at(child) == L.child_begin[v]);
                    child += fan(L, static_cast<int32_t>(w));
                } else {
                    F p;
                    std::memcpy(&p, &w, sizeof p);
                    expect(p == pay[v]);
                }
            }
            expect(child == U.n);
        }
        expect(id == S.id[at + nl - 1] + S.count[at + nl - 1]);
    }
    for (int64_t v = 0; v < L.N; ++v) expect(seen[v] == (v >= L.level_offset[S.cut] ? 1 : 0));
}

void check_forest(const std::vector<Layout>& games) {
    const Layout F = forest_layout(games);
    std::vector<int64_t> at(games.size());
    int64_t h = 0, q = 0, q0 = 0, m = 0;
    for (size_t g = 0; g < games.size(); ++g) {
        const Layout& L = games[g];
        // walk both trees together from the game's root
        std::vector<int64_t> to(L.N, -1);
        to[0] = F.child_begin[0] + static_cast<int64_t>(g);
        expect(F.parent[to[0]] == 0 && F.node_edge[to[0]] == F.Qp + F.Q0 - static_cast<int64_t>(games.size() - g));
        for (int64_t v = 0; v < L.N; ++v) {
            const int64_t f = to[v];
            expect(F.node_player[f] == L.node_player[v] && F.payoff[f] == L.payoff[v]);
            if (L.node_player[v] > 0) expect(F.node_infoset[f] == L.node_infoset[v] + h);
            expect(F.child_begin[f + 1] - F.child_begin[f] == L.child_begin[v + 1] - L.child_begin[v]);
            for (int64_t c = L.child_begin[v]; c < L.child_begin[v + 1]; ++c) {
                to[c] = F.child_begin[f] + (c - L.child_begin[v]);
                expect(F.parent[to[c]] == f);
                const int32_t e = L.node_edge[c];
                expect(F.node_edge[to[c]] == (e < L.Qp ? e + q : F.Qp + q0 + (e - L.Qp)));
            }
        }
        for (int64_t i = 0; i < L.n_members; ++i) expect(F.members[m + i] == to[L.members[i]]);
        for (int64_t i = 0; i < L.Hp; ++i)
            expect(F.q_offset[h + i] == L.q_offset[i] + q && F.member_offset[h + i] == L.member_offset[i] + m &&
                   F.infoset_player[h + i] == L.infoset_player[i]);
        h += L.Hp; q += L.Qp; q0 += L.Q0; m += L.n_members;
    }
    expect(F.level_offset.back() == F.N && static_cast<int32_t>(F.level_offset.size()) == F.D + 2);
}

}  // namespace

int main(int argc, char** argv) {
    FILE* f = argc == 2 ? std::fopen(argv[1], "rb") : nullptr;
    int32_t n_games = 0;
    if (f == nullptr || std::fread(&n_games, 4, 1, f) != 1) return 2;
    std::vector<Layout> all;
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
        for (const bool f64 : {false, true}) {
            Layout L;
            std::string err;
            if (flatten(d.g, L, err, f64) != CFR_OK) return 1;
            for (int32_t cut = 1; cut < L.D; ++cut)
                for (const int64_t window : {int64_t{1}, int64_t{97}, int64_t{3000}, int64_t{1} << 40}) {
                    PartPlan P;
                    StreamPlan S, sizes;
                    if (plan_partitions(L, cut, window, P, err) != CFR_OK) return 1;
                    plan_stream(L, P, f64, S);
                    plan_stream(L, P, f64, sizes, true);
                    expect(sizes.window == S.window && sizes.host_bytes(f64) == S.host_bytes(f64));
                    if (f64) check_stream(L, P, S, S.stream64, L.payoff64);
                    else check_stream(L, P, S, S.stream32, L.payoff);
                }
            if (!f64 && L.level_pure) all.push_back(std::move(L));
        }
    }
    std::fclose(f);
    check_forest(all);
    check_forest({all.front()});
    std::printf("%lld mismatches\n%s\n", static_cast<long long>(g_bad), g_bad == 0 ? "ok" : "bad");
    return g_bad == 0 ? 0 : 1;
}
