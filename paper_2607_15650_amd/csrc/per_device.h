// per_device.h - something done once on every device of the process (host code).
#pragma once

#include <stdint.h>

#include <atomic>

namespace ditango {

// run(dev, f) calls f() on the first call for each device, and again until it
// has returned 0 there; returns f's value, 0 once it is done.  f may run twice
// when threads meet on a device's first call.
class OncePerDevice {
 public:
  template <class F>
  auto run(int dev, F f) -> decltype(f()) {
    const uint64_t bit = dev >= 0 && dev < 64 ? uint64_t(1) << dev : 0;
    if (bit != 0 && (done_.load(std::memory_order_acquire) & bit) != 0) return decltype(f())(0);
    const auto e = f();
    if (e == decltype(f())(0)) done_.fetch_or(bit, std::memory_order_release);
    return e;
  }

 private:
  std::atomic<uint64_t> done_{0};
};

}  // namespace ditango
