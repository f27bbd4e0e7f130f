// Set-up that each device needs once (kernel attributes).
#pragma once

#include <stdint.h>

#include <atomic>

namespace lx {

// run() calls set() on the first call for a device and after a call that
// failed; its result is returned, `ok` where nothing was left to do. Threads
// that meet here each call set(), which therefore has to be repeatable. Devices
// from 64 on have no bit and call it every time.
class DeviceOnce {
 public:
  template <class Err, class F>
  Err run(int device, Err ok, F&& set) {
    const uint64_t bit = device >= 0 && device < 64 ? uint64_t{1} << device : 0;
    if (done_.load(std::memory_order_acquire) & bit) return ok;
    const Err e = set();
    if (e == ok) done_.fetch_or(bit, std::memory_order_release);
    return e;
  }

 private:
  std::atomic<uint64_t> done_{0};
};

}  // namespace lx
