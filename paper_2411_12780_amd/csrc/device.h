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

}  // namespace ppll
