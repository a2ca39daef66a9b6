// Something to be done, or found out, once for every device of the process (no HIP here: the
// tests build it for the host).
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

// get(device, f): what f() returned for that device, a positive number; one that is not is returned and
// asked for again the next time.  Threads and devices as above.
class DeviceNumber {
 public:
  template <typename F>
  int get(int device, F f) {
    const bool known = device >= 0 && device < 64;
    if (known)
      if (const int n = of_[device].load(std::memory_order_relaxed); n > 0) return n;
    const int n = f();
    if (known && n > 0) of_[device].store(n, std::memory_order_relaxed);
    return n;
  }

 private:
  std::atomic<int> of_[64] = {};
};

}  // namespace cfdetr
