// How many workgroups of a kernel the current device holds at once: the persistent kernels' workgroups wait on each other,
// so a grid of them is launched only if all fit.
#pragma once
#include <hip/hip_runtime.h>

namespace blstm {

// The answer depends on the kernel and the device only and is kept per kernel and thread for the device last asked about.
template <auto KERNEL>
hipError_t resident_workgroups(int threads, size_t dyn_lds, int* count) {
    static thread_local int device = -1, held = 0;
    int dev = 0, cus = 0, per_cu = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev != device) {
        e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        if (e == hipSuccess && dyn_lds > 0)
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(KERNEL), hipFuncAttributeMaxDynamicSharedMemorySize, (int)dyn_lds);
        if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, KERNEL, threads, dyn_lds);
        if (e != hipSuccess) return e;
        held = cus * per_cu;
        device = dev;
    }
    *count = held;
    return hipSuccess;
}

}  // namespace blstm
