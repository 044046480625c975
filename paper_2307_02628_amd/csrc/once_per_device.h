// Settings that a kernel needs once on every device before its first launch there (host only, no HIP).
#pragma once
#include <atomic>
#include <cstdint>

namespace skd {

// Runs set() until it has succeeded once for `device`; false if it failed now.  Threads may race to the first call: each
// of them runs set() (which is the same for all) before it goes on.
template <typename F>
bool once_per_device(std::atomic<uint64_t> &done, int device, F set) {
  const uint64_t bit = device >= 0 && device < 64 ? 1ull << device : 0;  // others: every time
  if (done.load(std::memory_order_acquire) & bit) return true;
  if (!set()) return false;
  done.fetch_or(bit, std::memory_order_release);
  return true;
}

}  // namespace skd
