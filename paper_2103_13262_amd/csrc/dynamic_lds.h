// Kernels whose dynamic LDS exceeds the default limit (internal).
#pragma once
#include <hip/hip_runtime_api.h>

#include <mutex>

namespace moe {

constexpr int kMaxDevices = 64;   // per-device caches (function attributes, compute-unit counts) are indexed by the HIP device id
int current_device();             // the calling thread's HIP device, or -1 (after fail_launch)
// A launcher that could not launch (a function attribute was refused, no usable device): records the text and makes
// the next check_launch on this thread return MOE_ERR_HIP.
void fail_launch(const char* fmt, ...);

// Raises the limit of one kernel, once per device.  The kernel itself is the template's parameter: its type is no key, the
// instances of a kernel template have one type between them.  False after fail_launch.
template <auto Kern> bool allow_dynamic_lds(int bytes)
{
    static std::mutex mu;
    static int allowed[kMaxDevices] = {};
    const int dev = current_device();
    if (dev < 0) return false;
    std::lock_guard<std::mutex> lk(mu);
    if (allowed[dev] < bytes) {
        const hipError_t e = hipFuncSetAttribute((const void*)Kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        if (e != hipSuccess) { fail_launch("%d bytes of dynamic LDS refused on device %d: %s", bytes, dev, hipGetErrorString(e)); return false; }
        allowed[dev] = bytes;
    }
    return true;
}

}  // namespace moe
