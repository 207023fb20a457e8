// Dynamic LDS limits of kernels.
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>
#include <map>
#include <mutex>
#include <utility>

namespace fsic {

// Allows kernel f at least `bytes` of dynamic LDS on the current device.  A
// limit is only ever raised: one set to the size of a smaller launch, or of an
// occupancy query, would outlast the shape it was meant for and could come
// between another thread's call and its launch.
inline hipError_t allow_lds(const void *f, size_t bytes) {
    if (bytes <= 32768) return hipSuccess;
    static std::mutex mu;
    static std::map<std::pair<int, const void *>, size_t> limit;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lk(mu);
    size_t &have = limit[{dev, f}];
    if (bytes <= have) return hipSuccess;
    e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e == hipSuccess) have = bytes;
    return e;
}

}  // namespace fsic
