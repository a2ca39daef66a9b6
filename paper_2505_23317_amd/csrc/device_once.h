// Something to be done once for every device of the process (no HIP here: the tests build it
// for the host).
#pragma once
#include <atomic>
#include <cstdint>

namespace cfdetr {

// run(device, f) calls f() until it has returned 0 for that device, and returns what it
// returned.  Any number of threads; two that come first together both call.  Devices from 64 on
// are not remembered.
class DeviceOnce {
 public:
  template <typename F>
  auto run(int device, F f) -> decltype(f()) {
    const uint64_t bit = device >= 0 && device < 64 ? uint64_t(1) << device : 0;
    if (done_.load(std::memory_order_relaxed) & bit) return decltype(f())(0);
    const auto r = f();
    if (r == decltype(f())(0)) done_.fetch_or(bit, std::memory_order_relaxed);
    return r;
  }

 private:
  std::atomic<uint64_t> done_{0};
};

}  // namespace cfdetr
