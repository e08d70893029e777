// The order in which a general-sum game's sums are formed, by level and infoset sizes (host rules, no
// HIP): the level-by-level kernels and the resident iteration both follow it, so that their results
// agree bit for bit.
#pragma once

#include <cstdint>

namespace cfr {

// A level of at most kWideNodes nodes sums each node's children over 64 lanes (lane t takes children
// t, t + 64, ..., then a butterfly); of at most kWideTop nodes (a root dealing many private types,
// the levels just below it) over kWideWaves wavefronts, whose sums are added in order; other
// levels in child order.
constexpr int32_t kWideNodes = 4096;
constexpr int32_t kWideTop = 16;
constexpr int32_t kWideWaves = 16;

// An infoset sums its members over so many wavefronts (thread t takes members t, t + threads, ...;
// a butterfly in each wavefront, then the wavefronts in order): one pass over the members of an
// average infoset, at most four wavefronts.
constexpr int32_t gather_waves(int64_t members, int64_t infosets) {
    const int64_t mean = infosets > 0 ? (members + infosets - 1) / infosets : 0;
    return mean <= 64 ? 1 : mean <= 128 ? 2 : 4;
}

}  // namespace cfr
