// Per-device set-up of a process: which devices have had it.
#pragma once

#include <stdint.h>

#include <atomic>

namespace pyro {

// One per thing to be set up.  run(dev, f) calls f, unless it has succeeded
// for device dev before, and returns its status (0: success); a failure is
// not kept.  Threads that come first together may each call f.
class DeviceOnce {
public:
    template <typename F>
    auto run(int dev, F f) -> decltype(f())
    {
        const bool known = dev >= 0 && dev < 64;
        const uint64_t bit = known ? (uint64_t)1 << dev : 0;
        if (done_.load(std::memory_order_acquire) & bit) return decltype(f())(0);
        const auto e = f();
        if (e == decltype(f())(0)) done_.fetch_or(bit, std::memory_order_release);
        return e;
    }

private:
    std::atomic<uint64_t> done_{0};
};

}  // namespace pyro
