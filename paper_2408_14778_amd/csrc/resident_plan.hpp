// Resident iteration (host plan, no HIP): a small or middle-sized game split into a trunk and small
// subtrees, the subtrees grouped into bins whose values and reach fit one workgroup's LDS, with the
// records that one launch iterates from start to end.
#pragma once

#include <algorithm>
#include <cstdint>
#include <string>
#include <thread>
#include <vector>

#include "flatten.hpp"

namespace cfr {

// 16-byte records as plain integers (loaded as one vector each on the device).
struct Rec4 {
    int32_t x, y, z, w;
};

constexpr int32_t kResMaxDepth = 120;   // levels of a resident game
constexpr int32_t kResMaxActions = 16;  // actions of its infosets
constexpr int32_t kResMaxFan = 4095;    // children of a chance node
constexpr int32_t kResTeam = 256;       // workgroups of a team: one per CU
// Bins of a workgroup at most (it then loads each anew in every pass). Where the line lies: with the
// public-block engine as the alternative (two players, single precision) three bins still win, up to
// kResNodesBlock nodes (5.5 million nodes: 124 against 140 us per iteration; 6.38 million of ten
// ranks 136 against 135, 6.48 million of thirteen 135 against 147, 6.60 million of twelve 143 against
// 135), and with two passes per iteration up to all that three bins hold, kResNodesBlock2 (6.60
// million: 235 against 251 us, 6.89 million 236 against 282). The node engine's alternatives are two
// times slower up to where eight bins end (2.2 million nodes in double precision: 78 against 229 us,
// 8.3 million 286 against 518).
// A batch keeps to one: its records cost more to lay out than its iterations gain beyond (10 games of
// 2.8 million nodes in all, two bins: 103 -> 79 us per iteration for 66 ms; 12 of 1.6 million, one
// bin: 84 -> 44 us).
// A single game pays for its records when it is built: 2.2 million nodes in double precision 57 -> 67
// ms, 3.3 million 87 -> 107 ms, 100,993 nodes 1.8 -> 2.6 ms, what 70, 120 and 13 iterations gain;
// three players 64 ms and single precision, whose plan of public blocks takes several times as long,
// the same within 2 %.
constexpr int32_t kResRoundsBlock = 3, kResRounds = 8, kResRoundsForest = 1;
constexpr int64_t kResNodesBlock = 6400000, kResNodesBlock2 = 7000000;
constexpr int32_t kResMaxBins = 1 + kResRounds * (kResTeam - 1);
constexpr int32_t kResTrunk = 32768;    // subtrees
constexpr int32_t kResPath = 24;        // levels above them
constexpr int32_t kResXcd = 32;         // CUs of one XCD
constexpr int64_t kResLds = 150 * 1024; // bytes of a bin's arrays (160 KB less the kernel's own)
// What a level's entry of ResPlan::table holds in its third word: log2 of the lanes that share a
// node's children, and how a general-sum game's level sums (sum_order.hpp; a two-player game's
// chance nodes always sum over their lanes and a butterfly, as the public-block engine's do)
constexpr int32_t kResLanes = 0xFF;
constexpr int32_t kResGrouped = 1 << 8;  // over 64 lanes (at most kWideNodes nodes), else in child order
constexpr int32_t kResWide = 1 << 9;     // at most kWideTop nodes, one with children for a second wavefront
enum ResMode { RES_SOLO = 0, RES_TEAM = 1 };

// A member's contributions and own reach, padded to 16 bytes.
constexpr int32_t res_stride(int32_t k, int32_t real_bytes) {
    return (k + 1 + 16 / real_bytes - 1) / (16 / real_bytes) * (16 / real_bytes);
}

struct ResSizes {
    int64_t nodes = 0, decision = 0, members = 0, infosets = 0, pairs = 0, chance_pairs = 0;
    int32_t depth = 0, max_actions = 0, players = 0, real_bytes = 4;
    int32_t passes = 1;  // per iteration
    bool level_pure = true, forest = false;
};
// f(begin, end) over parts of 0 .. n - 1, on several threads where n is large. f does not throw.
template <class Fn>
void for_ranges(int64_t n, const Fn& f) {
    const int64_t parts =
        n < 200000 ? 1 : std::max(1u, std::min(8u, std::thread::hardware_concurrency()));
    std::vector<std::thread> pool;
    int64_t i = 0;
    try {
        for (; i + 1 < parts; ++i)
            pool.emplace_back([&f, n, parts, i] { f(n * i / parts, n * (i + 1) / parts); });
    } catch (...) {  // fewer threads
    }
    f(n * i / parts, n);
    for (std::thread& th : pool) th.join();
}

// Whether a game of these sizes may run resident (the plan then decides); the plan's arrays are
// bounded by these sizes alone.
bool resident_fits(const ResSizes& z);
// Entries of ResPlan::table and ::path at most.
int64_t resident_max_table(const ResSizes& z);
int64_t resident_max_path(const ResSizes& z);
int64_t resident_max_roots(const ResSizes& z);

// Bins: bin 0 is the trunk (every node whose subtree is larger than a bin's share, and their other
// children as leaves: terminal nodes, and the subtrees' roots, whose values the other bins
// compute); every other bin is a run of subtrees. A game that fits one workgroup is one bin without
// a trunk (RES_SOLO). A bin's nodes and decision nodes are numbered locally, level by level (a
// node's children consecutively; of a level's decision nodes the players' first, then chance's).
struct ResPlan {
    int32_t mode = RES_SOLO, bins = 0;
    int32_t trunk_sets = 0;       // infosets with a member in the trunk: sets[0 .. trunk_sets)
    int32_t roots = 0, path_len = 0;
    // per decision node, bin-major in local order: {first child | own node << 16, edge of action
    // 0 | player << 28, parent's rank | actor into the node << 16 (15: a subtree's root) | k << 20,
    // edge into the node} (local nodes and ranks; edges index [sigma | sigma_0] in the engine's
    // pair order)
    std::vector<Rec4> rec;
    std::vector<int32_t> slot;    // per decision node: its first contribution (player nodes)
    std::vector<double> reach_c;  // per decision node: the chance probabilities on its path
    std::vector<int32_t> rank_node;  // per decision node: its canonical node
    std::vector<int32_t> node;    // per node, bin-major in local order: its canonical node
    // per infoset, the trunk's first, then by first pair: {first pair, first contribution,
    // members, k | player << 24}; member j's k contributions and its own reach lie from first
    // contribution + j res_stride(k, real_bytes)
    std::vector<Rec4> sets;
    // per root, in the order of the bins: its local rank, its leaf in the trunk (local node), and
    // path_len edges from the game's root down (edge | actor << 28; entry i of root x at i roots +
    // x, actor 0 past its end)
    std::vector<int32_t> root_rank, ext, path;
    // per bin from table[bin * (depth + 3)], per level of the game: {first local node, first local
    // rank, lanes and order of the sums (kRes...), chance nodes}; then {rank base in rec, nodes, ranks, node base in node} and
    // {first level, levels with decision nodes, first root, end of roots}
    std::vector<Rec4> table;
    int32_t max_nodes = 0, max_ranks = 0;  // of a bin
    int64_t contributions = 0;
    int32_t max_actions = 1, mean_members = 0;
    int32_t waves = 1;  // general sums: gather_waves of the infosets
};

// A batch as one game: a chance node above the games' roots deals each of them with probability 1, on
// edges past the games' own (its value is a sum that nobody reads). Infosets, pairs and chance pairs
// game after game in their canonical orders.
Layout forest_layout(const std::vector<Layout>& games);

// Plans layout L; q_of[h]: the first pair of canonical rational infoset h in the engine's order.
// False, and an empty plan: no split whose bins fit, or no memory for it (the game stays on the
// level-by-level launches).
bool build_resident(const Layout& L, const std::vector<int32_t>& q_of, const ResSizes& z,
                    ResPlan& out);

}  // namespace cfr
