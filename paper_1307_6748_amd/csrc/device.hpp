// Per-device kernel set-up shared by the solver's and the network's launches.
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>

namespace isis {

// Raises a kernel's dynamic LDS limit to `bytes` on the current device, once
// per device (the attribute is per device); `done` is the kernel's bitmask of
// devices already set up.
inline hipError_t ensure_dynamic_lds(const void* kern, int bytes, std::atomic<unsigned>& done)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const unsigned bit = dev < 32 ? 1u << dev : 0u;
    if (bit && (done.load(std::memory_order_acquire) & bit)) return hipSuccess;
    e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e == hipSuccess && bit) done.fetch_or(bit, std::memory_order_release);
    return e;
}

}  // namespace isis
