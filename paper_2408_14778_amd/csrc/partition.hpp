// Subtree-partitioned, out-of-core iteration (device side): the pinned host memory that holds the
// stream of a plan (stream_plan.hpp), and one pass of the iteration over it.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <vector>

#include "kernels.hpp"
#include "stream_plan.hpp"

namespace cfr {

// A partitioned solver of real type F: its plan and the pinned host copies that every pass reads.
template <class F>
struct PartDev {
    StreamPlan plan;
    // pinned host memory (hipHostMalloc), released by release()
    void* h_stream = nullptr;
    StreamUnit* h_units = nullptr;
    int32_t *h_code = nullptr, *h_child = nullptr;
    F* h_pay = nullptr;
    std::vector<int32_t> level_offset;  // canonical, D + 2 (the resident levels)
    int upload();                       // plan -> pinned buffers (once, at build)
    void release();
};

// One pass of the partitioned iteration on d (N = base + window local nodes; structure of the
// resident levels uploaded at build): resident top-down, then per group of partitions the levels
// between the cuts top-down, every run of subtrees below them, and those levels bottom-up; the
// resident bottom-up; the infoset pass.
template <class F>
void launch_partitioned_pass(const DevT<F>& d, const PartDev<F>& P, const UpdateRule& rule,
                             hipStream_t st);

}  // namespace cfr
