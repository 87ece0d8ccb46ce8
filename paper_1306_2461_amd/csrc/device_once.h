// Per-device set-up of a kernel (host code).
#pragma once

#include <atomic>
#include <cstdint>

namespace ofmi {

// set() once for each device: a kernel's attributes belong to the device that was current, so a process
// that drives several sets them on each.  `done` holds a bit per device (those past 63 set on every
// call); a failure is returned and tried again on the next call.
template <class Error, class Set>
Error once_per_device(std::atomic<uint64_t>& done, int device, Error success, Set set) {
  const uint64_t bit = device >= 0 && device < 64 ? uint64_t{1} << device : 0;
  if (done.load(std::memory_order_acquire) & bit) return success;
  const Error e = set();
  if (e == success) done.fetch_or(bit, std::memory_order_release);
  return e;
}

}  // namespace ofmi
