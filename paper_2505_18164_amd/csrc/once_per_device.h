// Work that is due once per GPU of the process: a kernel's attributes belong to the copy of it that a device has loaded.
// Plain C++, for the library and for a host test.
#pragma once

#include <atomic>
#include <cstdint>

namespace mdi {

class OncePerDevice {
  std::atomic<uint64_t> done_{0};                          // one bit per device ordinal

 public:
  static constexpr int kDevices = 64;
  // Calls work() unless it has succeeded for this device before; false if it fails, or the ordinal has no bit.  Threads
  // that meet on one device may both call it.
  template <typename Work>
  bool run(int device, Work&& work) {
    if (device < 0 || device >= kDevices) return false;
    const uint64_t bit = 1ull << device;
    if (done_.load(std::memory_order_acquire) & bit) return true;
    if (!work()) return false;
    done_.fetch_or(bit, std::memory_order_release);
    return true;
  }
};

}  // namespace mdi
