// The devices something has been done on, for set-up that belongs to a device and not to the process.
#pragma once
#include <atomic>
#include <cstdint>

namespace mtla {

// Any thread may ask and add at any time; a device past the 64th is never remembered, so its set-up is simply repeated.
class DeviceSet {
 public:
  bool has(int device) const { return (bits_.load(std::memory_order_acquire) & bit(device)) != 0; }
  void add(int device) { bits_.fetch_or(bit(device), std::memory_order_release); }

 private:
  static uint64_t bit(int device) { return device >= 0 && device < 64 ? uint64_t(1) << device : 0; }
  std::atomic<uint64_t> bits_{0};
};

}  // namespace mtla
