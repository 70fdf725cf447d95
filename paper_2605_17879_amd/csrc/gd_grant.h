// Leave for a kernel to be launched with more dynamic LDS than launches may ask for without
// more ado: asked for once per kernel and GPU, whichever of the process's threads comes first.
#ifndef GD_GRANT_H_
#define GD_GRANT_H_

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <atomic>

// granted: one word of a kernel's own, bit d for GPU d (a GPU beyond the 64th asks every time).
inline hipError_t gd_grant_lds(std::atomic<uint64_t>& granted, const void* kernel, size_t bytes) {
    int device = 0;
    hipError_t e = hipGetDevice(&device);
    if (e != hipSuccess) return e;
    const uint64_t bit = device >= 0 && device < 64 ? 1ull << device : 0ull;
    if (granted.load(std::memory_order_acquire) & bit) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e == hipSuccess) granted.fetch_or(bit, std::memory_order_release);
    return e;
}

#endif  // GD_GRANT_H_
