// The stream of an out-of-core iteration (host side, no HIP): the partitions of partition_plan.hpp
// cut once more, at the first level whose subtrees fit a workgroup's LDS. The subtrees below that
// level travel as runs of node records that a kernel reads once per iteration, straight from
// pinned host memory; the few levels between the two cuts keep records that are read level by level.
#pragma once

#include <cstdint>
#include <vector>

#include "flatten.hpp"
#include "partition_plan.hpp"

namespace cfr {

// Nodes of the largest subtree below the second cut, and of a run of smaller ones. A node takes 28
// bytes of LDS (48 in double precision): 1,024 leave room for five workgroups on a CU, which hide
// each other's reads over the host link.
constexpr int32_t kStreamMax = 2048, kStreamRun = 1024;
constexpr int32_t kStreamPart = 4;  // records per load (16 bytes of single precision)

// One run: n nodes below and with `roots` consecutive nodes of the second cut (the first has local id
// id0), breadth first over all of them, so the children of a node follow those of the nodes
// before it. At word `at` of the stream: a bit per node (1: decision) in 32-bit units, padded to a
// whole part, then a word per node, padded likewise: a decision's code (below), a terminal's payoff.
struct StreamUnit {
    int64_t at = 0;
    int32_t n = 0, roots = 0, id0 = 0, pad = 0;
};

// A code: the canonical infoset, or Hp + the chance infoset.
struct StreamPlan {
    int32_t cut = 0, split = 0;  // the second cut: cut .. D
    int64_t base = 0;            // first local id past the resident levels
    int64_t window = 0;          // nodes of the levels cut + 1 .. split of the largest group
    int32_t max_unit = 0;        // nodes of the largest run
    int64_t units_n = 0;         // runs
    // groups of consecutive partitions whose nodes between the cuts fit the window together
    int32_t groups = 0;
    std::vector<int32_t> unit0;     // groups + 1: first run
    // per group and level cut .. split: first local id, nodes, first record (levels before split)
    std::vector<int32_t> id, count;
    std::vector<int64_t> rec;
    int64_t mid = 0;  // records of the levels cut .. split - 1
    std::vector<int32_t> mid_code, mid_child;  // code (-1: terminal), local id of the first child
    std::vector<double> mid_pay;
    std::vector<StreamUnit> units;
    int64_t words = 0;           // stream length, in 32-bit (double precision: 64-bit) words
    std::vector<uint32_t> stream32;
    std::vector<uint64_t> stream64;
    // pinned host memory that a solver of this plan allocates
    int64_t host_bytes(bool f64) const {
        return words * (f64 ? 8 : 4) + mid * (f64 ? 16 : 12) +
               units_n * static_cast<int64_t>(sizeof(StreamUnit));
    }
};

// Fills S from a layout and its partitions. f64: records hold double-precision payoffs. sizes_only:
// without the records, units and stream themselves.
void plan_stream(const Layout& L, const PartPlan& P, bool f64, StreamPlan& S, bool sizes_only = false);

}  // namespace cfr
