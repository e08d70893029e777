// Pinned result words: see pinned.hpp.
#include "pinned.hpp"

#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstring>
#include <mutex>

namespace cfr {

namespace {

constexpr size_t kLine = 64, kLines = 4096;  // 256 KiB: a thousand solvers, or 16,384 games' values

struct Slab {
    std::mutex mu;
    unsigned char* base = nullptr;
    uint16_t run[kLines] = {};  // lines of the block that starts here (0: none does)
    bool used[kLines] = {};
};

// (never destroyed: the runtime may be gone before the process's static objects are)
Slab& slab() {
    static Slab* const s = new Slab();
    return *s;
}

void* allocate(size_t bytes) {
    // (allocating touches no stream: a capture that this thread is in the middle of goes on)
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    (void)hipThreadExchangeStreamCaptureMode(&mode);
    void* p = nullptr;
    const hipError_t e = hipHostMalloc(&p, bytes, hipHostMallocPortable);
    (void)hipThreadExchangeStreamCaptureMode(&mode);
    if (e == hipSuccess) return p;
    (void)hipGetLastError();
    return nullptr;
}

}  // namespace

void* pinned_take(size_t bytes) {
    Slab& s = slab();
    const size_t n = bytes > 0 ? (bytes + kLine - 1) / kLine : 1;
    void* p = nullptr;
    {
        const std::lock_guard<std::mutex> lock(s.mu);
        if (n <= kLines && s.base == nullptr)
            s.base = static_cast<unsigned char*>(allocate(kLine * kLines));
        if (n <= kLines && s.base != nullptr)
            for (size_t i = 0, free = 0; i < kLines && p == nullptr; ++i) {
                free = s.used[i] ? 0 : free + 1;
                if (free < n) continue;
                const size_t first = i + 1 - n;
                for (size_t j = first; j <= i; ++j) s.used[j] = true;
                s.run[first] = static_cast<uint16_t>(n);
                p = s.base + first * kLine;
            }
    }
    if (p == nullptr) p = allocate(n * kLine);
    if (p != nullptr) std::memset(p, 0, n * kLine);
    return p;
}

void pinned_give(void* p) {
    if (p == nullptr) return;
    Slab& s = slab();
    {
        const std::lock_guard<std::mutex> lock(s.mu);
        const unsigned char* c = static_cast<unsigned char*>(p);
        if (s.base != nullptr && c >= s.base && c < s.base + kLine * kLines) {
            const size_t first = static_cast<size_t>(c - s.base) / kLine;
            for (size_t j = first; j < first + s.run[first]; ++j) s.used[j] = false;
            s.run[first] = 0;
            return;
        }
    }
    (void)hipHostFree(p);
}

}  // namespace cfr
