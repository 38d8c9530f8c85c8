// What a process asks of every device once (more LDS for a kernel than it has by itself).
#pragma once

#include <atomic>

namespace kvm {

// E: an error type whose zero is success.  A static one of these stands for one thing asked for.
template <typename E>
class OncePerDevice {
 public:
  // current(&number): the calling thread's device; ask(): asks it.  Only what was granted is remembered, and for that device: a
  // failure is the call's, and the next one asks again.  (Asking twice, from two threads, does no harm.)
  template <typename Current, typename Ask>
  E operator()(Current current, Ask ask) {
    int dev = -1;
    E e = current(&dev);
    if (e != E{}) return e;
    const bool known = dev >= 0 && dev < kDevices;
    if (known && granted_[dev].load(std::memory_order_acquire)) return E{};
    e = ask();
    if (e == E{} && known) granted_[dev].store(true, std::memory_order_release);
    return e;
  }

 private:
  static constexpr int kDevices = 64;   // others are asked every time
  std::atomic<bool> granted_[kDevices] = {};
};

}  // namespace kvm
