// Pinned host words that kernels write their results into (a check's values, a step's loss), for one
// solver or network each. Freeing pinned memory waits for everything that the device runs, so the
// words are lines of one slab that the process allocates once and keeps, given back when their owner
// is destroyed; what does not fit the slab is an allocation of its own.
#pragma once

#include <cstddef>

namespace cfr {

// At least `bytes` of zeroed pinned memory, 64-byte aligned and in no line of another owner's; null: none
// to be had. Any thread; no stream is touched, and a capture that the thread is in goes on.
void* pinned_take(size_t bytes);
// Returns it (null: nothing). No kernel may still write there.
void pinned_give(void* p);

}  // namespace cfr
