// What launches look up or arrange once per device, safe with several host threads.  No HIP in here: the calls come in as
// arguments.
#pragma once
#include <atomic>

namespace ppll {

constexpr int MAX_DEVICES = 64;

// Runs `set` (0 on success) on a device until it has succeeded there once.  A device counts as done only then: a thread that
// finds it not done runs `set` itself, so that nobody goes on before it has taken effect.
class OncePerDevice {
  std::atomic<bool> done_[MAX_DEVICES] = {};

 public:
  template <class Set> int operator()(int dev, Set set) {
    const bool known = dev >= 0 && dev < MAX_DEVICES;
    if (known && done_[dev].load(std::memory_order_acquire)) return 0;
    const int status = set();
    if (status == 0 && known) done_[dev].store(true, std::memory_order_release);
    return status;
  }
};

// A positive number that `query` gives for a device (0 or less: it could not say), asked for once.
class PerDevice {
  std::atomic<int> value_[MAX_DEVICES] = {};

 public:
  template <class Query> int operator()(int dev, Query query) {
    const bool known = dev >= 0 && dev < MAX_DEVICES;
    if (known) {
      const int v = value_[dev].load(std::memory_order_relaxed);
      if (v > 0) return v;
    }
    const int v = query();
    if (known && v > 0) value_[dev].store(v, std::memory_order_relaxed);
    return v;
  }
};

}  // namespace ppll
