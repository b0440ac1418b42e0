// device_once.hpp -- a setting that is made once on each device.
#pragma once
#include <atomic>
#include <cstdint>

namespace pa {

// Calls set() on the first use for each device (of 64; it is called each time
// on others) and returns its result, 0 for success and from then on.  A failure
// is not kept: the next use tries again.  Two threads that meet on a first use
// may both call set().
class DeviceOnce {
    std::atomic<std::uint64_t> done_{0};

  public:
    template <class F>
    auto operator()(int device, F&& set) -> decltype(set()) {
        const std::uint64_t bit = device >= 0 && device < 64 ? std::uint64_t(1) << device : 0;
        if (done_.load(std::memory_order_acquire) & bit) return decltype(set())(0);
        const auto e = set();
        if (e == decltype(set())(0)) done_.fetch_or(bit, std::memory_order_release);
        return e;
    }
};

}  // namespace pa
