// Two persistent launches at once, each half resident, would starve each other until their waits are abandoned.  So one
// waits for the other on the device: every persistent launch carries an event as its completion signal, which the next one
// waits for.  On one stream the wait costs nothing (the order is there already) and the event 0.5 us a launch (a marker
// behind the launch: 1.5 us, with a system fence 3 us).
// Not covered, because nothing here can order them: launches in replays of captured graphs, and other processes.
#include "residency.hpp"
#include <hip/hip_ext.h>
#include <mutex>

namespace blstm {
namespace {

constexpr int MAX_DEVICES = 64;
std::mutex g_mutex;                                // held from the wait to the launch
hipEvent_t g_last[MAX_DEVICES];                    // completion of the device's last persistent launch; null: none yet.  Kept until the process ends

}  // namespace

hipError_t launch_in_turn(const void* kernel, int grid, int threads, size_t dyn_lds, void** args, hipStream_t st) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (dev >= MAX_DEVICES || hipStreamIsCapturing(st, &capture) != hipSuccess || capture != hipStreamCaptureStatusNone) {
        (void)hipGetLastError();                   // (of the query)
        e = hipLaunchKernel(kernel, dim3(grid), dim3(threads), args, dyn_lds, st);
        return e != hipSuccess ? e : hipGetLastError();
    }
    std::lock_guard<std::mutex> lock(g_mutex);
    if (g_last[dev]) e = hipStreamWaitEvent(st, g_last[dev], 0);
    else e = hipEventCreateWithFlags(&g_last[dev], hipEventDisableTiming | hipEventDisableSystemFence);
    if (e != hipSuccess) return e;
    e = hipExtLaunchKernel(kernel, dim3(grid), dim3(threads), args, dyn_lds, st, nullptr, g_last[dev], 0);
    return e != hipSuccess ? e : hipGetLastError();
}

}  // namespace blstm
