// Leave for a kernel to take more dynamic LDS than 64 KB (internal).
#pragma once
#include <hip/hip_runtime.h>

namespace tsr {

// To be called before each launch: the attribute belongs to the kernel on the current device, and is set on the
// first call there (remembered per host thread; kernels beyond the table set it each time).
inline hipError_t allow_lds(const void* kernel, int bytes) {
    if (bytes <= 64 * 1024) return hipSuccess;
    struct Entry { const void* kernel; unsigned long long devices; };
    static thread_local Entry seen[64] = {};
    int device = 0;
    hipError_t e = hipGetDevice(&device);
    if (e != hipSuccess) return e;
    const unsigned long long bit = device < 64 ? 1ull << device : 0;
    Entry* at = nullptr;
    for (Entry& x : seen)
        if (x.kernel == kernel || x.kernel == nullptr) { at = &x; break; }
    if (at && at->kernel == kernel && (at->devices & bit)) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e != hipSuccess) return e;
    if (at) { at->kernel = kernel; at->devices |= bit; }
    return hipSuccess;
}

}  // namespace tsr
