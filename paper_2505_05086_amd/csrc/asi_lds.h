// More LDS for a kernel than the 64 KB that a launch may ask for without saying so first.
#pragma once
#include <hip/hip_runtime_api.h>

#include <atomic>
#include <cstddef>
#include <cstdint>

namespace asi {

// A kernel's allowance belongs to the kernel AND the GPU, so it is asked for once for every GPU that the kernel is launched
// on, whichever threads do so: `done` has a bit per device, set once the call has succeeded there.  `bytes` is the most that any
// launch of the kernel takes (the same in every call: an allowance that a second thread could lower again is none).
struct LdsAllowed {
    std::atomic<uint64_t> devices{0};
};
inline hipError_t allow_lds(const void* kernel, size_t bytes, LdsAllowed& done) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = dev >= 0 && dev < 64 ? uint64_t(1) << dev : 0;      // (past the 64th device: asked for every time)
    if (done.devices.load() & bit) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e == hipSuccess) done.devices.fetch_or(bit);
    return e;
}

}  // namespace asi
