// Set-up that has to happen once on every device (host only, no HIP).
#pragma once

#include <atomic>

namespace shot {

// Runs set() on behalf of device dev until it has returned 0 there, and returns its
// status (0 where it was done before).  Threads that meet here all run set(), in any
// order and at the same time: it has to do the same whoever runs it.
template <typename Set>
auto once_per_device(std::atomic<unsigned long long>& done, int dev, Set set) -> decltype(set()) {
  const unsigned long long bit = dev >= 0 && dev < 64 ? 1ull << dev : 0;  // (no memory of devices beyond 63)
  if (done.load(std::memory_order_acquire) & bit) return decltype(set())();
  const auto status = set();
  if (status == decltype(set())()) done.fetch_or(bit, std::memory_order_release);
  return status;
}

}  // namespace shot
