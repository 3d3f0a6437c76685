// Something that has to be done once on every device, such as a kernel's attributes: a launch does it before its first
// one there.  (Done once in the process, a second device would go without.)
#pragma once
#include <stdint.h>
#include <atomic>

namespace asl {

class OncePerDevice {
 public:
  // f() on device `device`, unless it has returned `ok` there; returns what f does, or `ok`.  Any threads at once: f may then
  // run more than once.  Devices from the 64th on are not remembered.
  template <typename R, typename F>
  R operator()(int device, R ok, F f) {
    const uint64_t bit = device >= 0 && device < 64 ? uint64_t(1) << device : 0;
    if ((done_.load(std::memory_order_acquire) & bit) != 0) return ok;
    const R r = f();
    if (r == ok) done_.fetch_or(bit, std::memory_order_release);
    return r;
  }

 private:
  std::atomic<uint64_t> done_{0};
};

}  // namespace asl
