// A setting that a device keeps once it has been made, and that has to be made on each device by itself.
#pragma once

#include <atomic>
#include <cstdint>

namespace lime {

class PerDevice {
 public:
  // Calls `make` (0 = success) unless it has succeeded for this device before; returns what it returned.  A failure is not
  // remembered.  Threads that come at the same time may each call it, and a device past the 64th calls it every time.
  template <typename Make>
  auto ensure(int device, Make make) -> decltype(make()) {
    const uint64_t bit = device >= 0 && device < 64 ? uint64_t{1} << device : 0;
    if (made_.load(std::memory_order_acquire) & bit) return {};
    const auto status = make();
    if (static_cast<int>(status) == 0) made_.fetch_or(bit, std::memory_order_release);
    return status;
  }

 private:
  std::atomic<uint64_t> made_{0};
};

}  // namespace lime
