// Which results hardware atomic additions may be used for.
#pragma once
#include <hip/hip_runtime_api.h>

namespace hydra {

// Plain memory of the GPU that the kernel runs on.  Not another GPU's, whose additions would have to be carried out across the
// link, nor fine-grained or uncached device memory (both allocation flags have bit 0, signal memory bit 1), where the hardware may
// leave floating-point additions out, nor host or managed memory.
inline bool atomic_adds_ok(const hipPointerAttribute_t &at, int gpu) {
  return at.type == hipMemoryTypeDevice && at.device == gpu && !(at.allocationFlags & hipDeviceMallocUncached);
}

}  // namespace hydra
