// Dynamic LDS of the patch kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <map>
#include <mutex>
#include <utility>

namespace cf {

// LDS bytes a block may take on the current device.
inline size_t device_lds_limit() {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 65536;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess) return 65536;
    return (size_t)v;
}

// Dynamic LDS above 64 KB needs the kernel's attribute raised first (a cap,
// only ever raised, under a lock); false when the runtime refuses.
inline bool lds_allow(const void* kernel, size_t lds) {
    if (lds <= 65536) return true;
    static std::mutex mu;
    static std::map<std::pair<int, const void*>, size_t> cap;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return false;
    std::lock_guard<std::mutex> lk(mu);
    size_t& c = cap[{dev, kernel}];
    if (lds <= c) return true;
    if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    c = lds;
    return true;
}

}  // namespace cf
