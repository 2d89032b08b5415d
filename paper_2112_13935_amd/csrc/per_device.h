// Something that is set or found out once per GPU and kernel: the permission for more than 64 KB
// of LDS, an occupancy.  A process can hold a context on every GPU and drive each from a thread
// of its own, so "once" is per device, and threads may come at the same time.  Host code
// without HIP, so that a CPU test can include it.
#pragma once
#include <atomic>

namespace aet {

constexpr int kMaxDevices = 64;

class PerDevice {
    std::atomic<int> value_[kMaxDevices] = {};   // 0: not known yet

 public:
    // *value of device dev.  find(value) works it out (a positive number; returns 0 for
    // success): the first time on each device, again after a failure, and in every thread that
    // comes before the first is done (all store the same).
    template <class Find>
    auto get(int dev, int *value, Find find) -> decltype(find(value)) {
        const bool known = dev >= 0 && dev < kMaxDevices;
        if (known && (*value = value_[dev].load(std::memory_order_acquire)) > 0) return decltype(find(value))(0);
        const auto status = find(value);
        if (known && status == decltype(find(value))(0)) value_[dev].store(*value, std::memory_order_release);
        return status;
    }
};

}  // namespace aet
