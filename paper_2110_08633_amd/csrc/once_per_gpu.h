// An action that has to be done once on every GPU a process uses, such as setting an attribute of a kernel: the
// attribute belongs to the code object as loaded on one GPU.
#pragma once
#include <stdint.h>

#include <atomic>

namespace hydra {

class OncePerGpu {
 public:
  // f() -> int, 0 = done.  Called unless an earlier call for this GPU returned 0; a failure is not remembered.  Threads
  // that come first at the same time may each call it.  GPUs past the 64th are not remembered either.
  template <typename F>
  int run(int gpu, F f) {
    const uint64_t bit = gpu >= 0 && gpu < 64 ? (uint64_t)1 << gpu : 0;
    if (done_.load(std::memory_order_acquire) & bit) return 0;
    const int e = f();
    if (e == 0) done_.fetch_or(bit, std::memory_order_release);
    return e;
  }

 private:
  std::atomic<uint64_t> done_{0};
};

}  // namespace hydra
