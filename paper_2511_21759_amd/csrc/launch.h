// Host-side helpers of the kernel launches.
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>

namespace odb {

// Lets a kernel use more dynamic LDS than the default limit of 64 KiB: once per kernel and GPU.
template <auto Kernel>
inline void allow_lds(int bytes) {
    static std::atomic<unsigned long long> done{0};
    int dev = 0;
    (void)hipGetDevice(&dev);
    const unsigned long long bit = 1ull << (dev & 63);
    if (done.load(std::memory_order_acquire) & bit) return;
    (void)hipFuncSetAttribute(reinterpret_cast<const void *>(Kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    done.fetch_or(bit, std::memory_order_release);
}

}  // namespace odb
