// Something that has to be asked of the runtime once on every GPU a process uses.
#pragma once
#include <atomic>
#include <stdint.h>

namespace cr {

class PerDevice {
    std::atomic<uint64_t> done_{0};      // bit d: granted on device d (the devices from 64 on ask every time)

public:
    // Whether ask() has been granted on `device`: asks if it has not.  Threads that meet here may ask twice.
    template <typename Ask>
    bool once(int device, Ask &&ask)
    {
        const uint64_t bit = device >= 0 && device < 64 ? 1ull << device : 0ull;
        if (done_.load(std::memory_order_acquire) & bit) return true;
        if (!ask()) return false;
        done_.fetch_or(bit, std::memory_order_release);
        return true;
    }
};

}  // namespace cr
