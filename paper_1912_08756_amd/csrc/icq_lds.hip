// Opt-in for more dynamic LDS than the default.
#include "icq_lds.h"

#include <map>
#include <mutex>
#include <utility>

hipError_t icq_allow_lds(const void *fn, int bytes, bool no_static_lds) {
    static std::mutex mu;
    static std::map<std::pair<int, const void *>, int> allowed;        // most bytes asked for so far
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lock(mu);
    const auto it = allowed.find({dev, fn});
    if (it != allowed.end() && it->second >= bytes) return hipSuccess;
    if (no_static_lds) {
        hipFuncAttributes attr;
        e = hipFuncGetAttributes(&attr, fn);
        if (e != hipSuccess) return e;
        if (attr.sharedSizeBytes != 0) return hipErrorInvalidValue;
    }
    e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e == hipSuccess) allowed[{dev, fn}] = bytes;
    return e;
}
