// Set-up that a kernel needs once on every device (no HIP here).
#pragma once
#include <stdint.h>

#include <atomic>

namespace upir {

// run(device, f): f() until it has succeeded (returned zero) once for the
// device, then zero. Any thread may call it; two that come first may both run
// f. A failure is returned and not kept: the next call tries again.
class OncePerDevice {
  std::atomic<uint64_t> done_{0};

 public:
  template <class F>
  auto run(int device, F &&f) -> decltype(f()) {
    const uint64_t bit = device >= 0 && device < 64 ? 1ULL << device : 0;
    if (done_.load(std::memory_order_acquire) & bit) return decltype(f())(0);
    const auto e = f();
    if (e == decltype(f())(0)) done_.fetch_or(bit, std::memory_order_release);
    return e;
  }
};

}  // namespace upir
