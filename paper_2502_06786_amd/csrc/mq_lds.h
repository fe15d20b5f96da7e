// How much dynamic LDS a kernel has been allowed, per device (host code, no HIP in it).
#pragma once
#include <atomic>
#include <mutex>

namespace mq {

class LdsGrants {
    static constexpr int kDevices = 64;
    std::atomic<int> allowed_[kDevices] = {};  // the largest size granted so far
    std::mutex mutex_;

  public:
    // Makes sure that `bytes` are allowed on device `dev`.  set(bytes) asks the runtime, replacing what was allowed before, and
    // says whether it agreed.  Asking and recording are one step: between two threads with two sizes the smaller one would
    // otherwise be what the runtime keeps and the larger one what is recorded.
    template <typename Set>
    bool ensure(int dev, int bytes, Set set) {
        if (dev < 0) return false;
        if (dev < kDevices && allowed_[dev].load(std::memory_order_acquire) >= bytes) return true;
        std::lock_guard<std::mutex> lock(mutex_);
        if (dev >= kDevices) return set(bytes);
        if (allowed_[dev].load(std::memory_order_relaxed) >= bytes) return true;
        if (!set(bytes)) return false;
        allowed_[dev].store(bytes, std::memory_order_release);
        return true;
    }
};

}  // namespace mq
