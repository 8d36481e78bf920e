// Set-up that a kernel needs once on every device (function attributes belong to a device).
#pragma once

#include <atomic>

namespace gw {

// What is known to be set up: a bit per device.  run(device, set): set() where that device has not been seen,
// and again after a failure; devices beyond the bits each time.  Safe with several threads (set() may then run
// more than once).
class OncePerDevice {
 public:
  template <typename Set> auto run(int device, Set set) -> decltype(set()) {
    const unsigned long long bit = device >= 0 && device < 64 ? 1ull << device : 0;
    if (done_.load(std::memory_order_acquire) & bit) return {};
    const auto e = set();
    if (e == decltype(set()){}) done_.fetch_or(bit, std::memory_order_release);
    return e;
  }

 private:
  std::atomic<unsigned long long> done_{0};
};

}  // namespace gw
