// A launch's one-time preparation, per device (plain C++).
#pragma once

#include <atomic>
#include <cstdint>

namespace po {

// A kernel's limit of dynamic LDS belongs to the kernel on ONE device: raised for the first device a process launches on,
// it is not raised for the next.  Threads may come here together: each runs f unless it sees that somebody has finished it.
struct OncePerDevice {
    std::atomic<uint64_t> done{0};
    template <typename F>
    void run(int device, F f) {
        const uint64_t bit = 1ull << (device & 63);
        if (done.load(std::memory_order_acquire) & bit) return;
        f();
        done.fetch_or(bit, std::memory_order_release);
    }
};

}  // namespace po
