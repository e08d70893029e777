// Resident iteration (device): one launch runs many iterations of a game whose bins
// (resident_plan.hpp) fit the LDS of the chip's CUs.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "kernels.hpp"
#include "resident_plan.hpp"

namespace cfr {

constexpr int kResGroup = 16;  // arrivals that meet on one counter before the barrier's own

// State of a launch's team of workgroups; zero between launches. Every counter on a line of its own.
struct ResTeam {
    struct Line {
        uint32_t v;
        uint32_t pad[31];
    };
    Line xcc;     // 1 + the XCD that the team forms on (one-XCD teams)
    Line reg;     // registered workgroups; the top bit is set once the team is complete
    Line size;    // the complete team's size
    Line exited;  // workgroups of the launch that have left
    Line bar;     // complete groups at the team's barrier
    Line group[kResTeam / kResGroup];  // arrivals of a group
};

// All pointers are device memory; F the arithmetic type. N nodes, ND decision nodes.
template <class F>
struct Resident {
    int64_t N = 0;
    int32_t ND = 0, Hp = 0, Qp = 0, Q0 = 0, D = 0;
    int32_t players = 0;   // general-sum game of n players, or 0 (two players, zero sum)
    int32_t mode = 0, bins = 0, team_size = 1, trunk_sets = 0;
    int32_t team_limit = 0;  // at most so many workgroups (0: team_size of them)
    int32_t roots = 0, path_len = 0;
    int32_t max_nodes = 0, max_ranks = 0;
    int64_t n_con = 0;
    int32_t alog = 0;      // log2 of the lanes per infoset: over its actions
    int32_t mlog = 0;      // and over its members
    int32_t waves = 1;     // general sums: wavefronts whose order the members' sums follow
    int32_t threads = 0;   // threads per workgroup
    Rec4* rec = nullptr;
    int32_t* slot = nullptr;
    F* reach_c = nullptr;  // ND, in the order of rec
    Rec4* sets = nullptr;
    int32_t *root_rank = nullptr, *ext = nullptr, *path = nullptr;
    Rec4* table = nullptr;
    F* con = nullptr;      // contributions (RES_SOLO: in LDS)
    F* root_val = nullptr; // column i of root x at i * roots + x
    // payoffs and the last iteration's node values (in the order of ResPlan::node, column i at i
    // NB) and the players' reach (in the order of rec, plane i at i ND)
    int64_t NB = 0;        // N + roots
    F* pay = nullptr;
    F* val = nullptr;
    F* reach = nullptr;
    ResTeam* team = nullptr;
    // the engine's state
    F *prob = nullptr, *R = nullptr, *S = nullptr;
    int64_t* T = nullptr;
};

// Takes a plan's sizes and sets the launch shape.
template <class F>
void resident_shape(Resident<F>& r, const ResPlan& p);
// Fills r.pay from the payoff columns in canonical order (column i at i N); r.val holds ResPlan::node
// as int32 (it is not read before an iteration has written it).
template <class F>
void launch_resident_pay(const Resident<F>& r, const F* payoff, hipStream_t st);
// Clears the team, once, when the solver is set up.
template <class F>
void launch_resident_reset(const Resident<F>& r, hipStream_t st);
// Workgroups of a launch's team at most.
template <class F>
int32_t resident_workgroups(const Resident<F>& r) {
    if (r.mode == RES_SOLO) return 1;
    return r.team_limit > 0 && r.team_limit < r.team_size ? r.team_limit : r.team_size;
}
// The most iterations of one launch: about 5 ms of a full team's work. A launch keeps the team that it
// formed; one that formed while other work held the CUs is slower, and the next launch forms anew. A
// launch costs 6 to 10 us, so shorter ones would show. An iteration's time is taken as 4 us and 22 ps a
// node and pass (617 nodes and three passes 3.3 us, 2.6 million nodes 58 us, 5.5 million 124 us).
template <class F>
int32_t resident_launch_iterations(const Resident<F>& r, int32_t passes) {
    const double us = 4.0 + 22e-6 * static_cast<double>(r.N) * passes;
    return static_cast<int32_t>(5000.0 / us) > 16 ? static_cast<int32_t>(5000.0 / us) : 16;
}
// n iterations (alternating: a pass per player each), T += n.
template <class F>
void launch_resident(const Resident<F>& r, const UpdateRule& rule, bool alternating, int32_t n,
                     hipStream_t st);

}  // namespace cfr
