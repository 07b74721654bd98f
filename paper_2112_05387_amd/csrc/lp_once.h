// Work that a process does once per device before it launches a kernel there (raising the kernel's LDS limit): a function
// attribute belongs to the device that is current when it is set, and launches come from any thread.
#pragma once
#include <atomic>

namespace lp {

class OncePerDevice {
    std::atomic<unsigned long long> done_{0};      // bit d: done on device d (devices beyond 63: done every time)

public:
    // get(&device) and work() return an error code, 0 for success.  Work that fails is done again by the next call; threads
    // that come at the same time may both do it, so it has to be repeatable.
    template <class Get, class Work> auto run(Get get, Work work) -> decltype(work()) {
        int device = 0;
        const auto err = get(&device);
        if (err != decltype(err)(0)) return err;
        const unsigned long long bit = device >= 0 && device < 64 ? 1ull << device : 0;
        if (done_.load(std::memory_order_acquire) & bit) return decltype(work())(0);
        const auto e = work();
        if (e == decltype(e)(0)) done_.fetch_or(bit, std::memory_order_release);
        return e;
    }
};

}  // namespace lp
