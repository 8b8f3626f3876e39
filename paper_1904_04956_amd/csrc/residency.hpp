// The persistent kernels' workgroups wait on each other, so all of a grid must be resident at once: a grid is launched only
// if the device holds it, and behind the persistent launches that it cannot run beside, whatever streams they are on.
#pragma once
#include <hip/hip_runtime.h>

namespace blstm {

// LDS a workgroup may ask for: a CU's 160 KB but for what __syncthreads_or takes.
constexpr int LDS_MOST = 159 * 1024;

// How many workgroups of a kernel the current device holds at once.  The answer depends on the kernel, its LDS and the device only
// and is kept per kernel and thread for the last few of those asked about (the LDS differs between learners: see recurrent_multi.hip).
template <auto KERNEL>
hipError_t resident_workgroups(int threads, size_t dyn_lds, int* count) {
    constexpr int KEPT = 4;
    struct Asked { int device; size_t lds; int held; };
    static thread_local Asked asked[KEPT] = {{-1, 0, 0}, {-1, 0, 0}, {-1, 0, 0}, {-1, 0, 0}};
    static thread_local int oldest = 0;
    int dev = 0, cus = 0, per_cu = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    for (const Asked& k : asked)
        if (k.device == dev && k.lds == dyn_lds) { *count = k.held; return hipSuccess; }
    e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess && dyn_lds > 0)
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(KERNEL), hipFuncAttributeMaxDynamicSharedMemorySize, LDS_MOST);   // (not dyn_lds: other threads may launch it with more)
    if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, KERNEL, threads, dyn_lds);
    if (e != hipSuccess) return e;
    asked[oldest] = {dev, dyn_lds, cus * per_cu};
    oldest = (oldest + 1) % KEPT;
    *count = cus * per_cu;
    return hipSuccess;
}

// Launches a kernel behind those launched here on this device that would not fit beside it (on a stream that is being captured:
// without that).  grid: a multiple of eight.
hipError_t launch_in_turn(const void* kernel, int grid, int threads, size_t dyn_lds, void** args, hipStream_t st);

// Launches `grid` workgroups of KERNEL (`real` of which wait on each other, the others leave at once) if those can all be
// resident, or (a.ask) only says whether they can.
template <auto KERNEL, typename A>
hipError_t launch_resident(const A& a, int threads, size_t dyn_lds, int grid, int real, hipStream_t st, bool* launched) {
    int resident = 0;
    const hipError_t e = resident_workgroups<KERNEL>(threads, dyn_lds, &resident);
    if (e != hipSuccess || resident < real) return e;
    *launched = true;
    if (a.ask) return hipSuccess;
    A copy = a;
    void* args[] = {&copy};
    return launch_in_turn(reinterpret_cast<const void*>(KERNEL), grid, threads, dyn_lds, args, st);
}

}  // namespace blstm
