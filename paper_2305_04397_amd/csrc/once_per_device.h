// Something to be asked for once on every device of a process, whatever thread
// or context comes first there.
#pragma once

#include <atomic>
#include <cstdint>

namespace morap {

class OncePerDevice {
public:
    // ask() unless it has returned for that device before (it throws to be asked
    // again; two threads at once may both ask)
    template <class F>
    void operator()(int device, F&& ask) {
        const uint64_t bit = device >= 0 && device < 64 ? uint64_t(1) << device : 0;   // (others: every time)
        if (done_.load(std::memory_order_acquire) & bit) return;
        ask();
        done_.fetch_or(bit, std::memory_order_release);
    }

private:
    std::atomic<uint64_t> done_{0};
};

}  // namespace morap
