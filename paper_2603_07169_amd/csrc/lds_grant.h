// The limit up to which a kernel may be launched with dynamic LDS.  Host code.
#pragma once
#include <hip/hip_runtime_api.h>

#include <atomic>
#include <cstddef>
#include <cstdint>

namespace spmv {

constexpr size_t kLdsOfUnit = 160 * 1024;  // LDS of a compute unit
// Launches of up to this many bytes need no grant.  The runtime's limit is 64 KB with the kernel's own arrays, which take 2.2 KB at most.
constexpr size_t kLdsUngranted = 60 * 1024;

// One per kernel, with static storage.  The limit is a property of the kernel on a device: whoever raises it raises it for all threads, and
// whoever set it to what one launch needs could take from another thread what that had been given.  So it is set to all that the kernel's own
// arrays leave of a compute unit, once per device, whatever the launch at hand needs.
class LdsGrant {
   public:
    hipError_t operator()(const void* kernel, size_t lds) {
        if (lds <= kLdsUngranted) return hipSuccess;
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        const uint64_t bit = dev < 64 ? uint64_t{1} << dev : 0;  // a device beyond those is told every time
        if ((devices_.load(std::memory_order_acquire) & bit) == 0) {
            hipFuncAttributes own{};
            if ((e = hipFuncGetAttributes(&own, kernel)) != hipSuccess) return e;
            const size_t most = kLdsOfUnit - own.sharedSizeBytes;
            if ((e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(most))) != hipSuccess) return e;
            most_.store(most, std::memory_order_relaxed);  // the same number on every device
            devices_.fetch_or(bit, std::memory_order_release);
        }
        return lds <= most_.load(std::memory_order_relaxed) ? hipSuccess : hipErrorInvalidValue;
    }

   private:
    std::atomic<uint64_t> devices_{0};
    std::atomic<size_t> most_{0};
};

}  // namespace spmv
