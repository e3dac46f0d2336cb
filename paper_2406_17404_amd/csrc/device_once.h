// Something to be done once on every device of the process, from any thread.
#pragma once
#include <stdint.h>

#include <atomic>

namespace trj {

// Threads that come at the same time may each do it; it counts as done when it returned 0.
// Devices from 64 on have no place to remember it: there it is done every time.
class DeviceOnce {
  std::atomic<uint64_t> done_{0};

 public:
  template <class F>
  int run(int device, F f) {
    const uint64_t bit = device >= 0 && device < 64 ? 1ull << device : 0;
    if (done_.load(std::memory_order_acquire) & bit) return 0;
    const int rc = f();
    if (rc == 0) done_.fetch_or(bit, std::memory_order_release);
    return rc;
  }
};

}  // namespace trj
