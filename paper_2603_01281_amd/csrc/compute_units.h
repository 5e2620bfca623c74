// A small count per device, asked for on a device's first use.  Host only, no HIP: `ask` does the asking.
#pragma once
#include <atomic>

namespace seka {

class PerDeviceCount {
 public:
  // Any number of threads may call this at once: those that come first all ask, and get the same answer.
  template <class Ask>
  int of(int device, Ask&& ask) {
    if (device < 0 || device >= kDevices) return ask(device);
    int n = known_[device].load(std::memory_order_relaxed);
    if (n == 0) {
      n = ask(device);
      known_[device].store(n, std::memory_order_relaxed);
    }
    return n;
  }

 private:
  static constexpr int kDevices = 64;
  std::atomic<int> known_[kDevices] = {};      // 0: not asked yet
};

}  // namespace seka
