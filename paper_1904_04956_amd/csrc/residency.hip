// Persistent launches at once, each resident in part only, would starve each other until their waits are abandoned.  So those
// that may run at the same time never have more workgroups together than the device has CUs: each workgroup then finds a CU
// without another one (grids are whole rounds of the eight XCDs, so this holds on every XCD).  A launch beyond that waits on
// the device for as many of the others as it takes (one with more than a workgroup a CU, for all of them).  Every launch carries an event as its completion signal for that (0.5 us
// a launch; a marker behind it 1.5 us, with a system fence 3 us).  Three learners of 4 x 512 cells and 8 sequences (64
// workgroups a launch), a thread and a stream each: 801 us a step of all three, 1284 with every launch behind the last one,
// 470 for one learner alone.
// Not covered, because nothing here can order them: launches in replays of captured graphs, and other processes.  Two replays at once of 64 sequences of 512 cells, 256 workgroups
// each, fill the device twice: the kernels with wavefronts for what is not the exchange have 512 threads and, backward at 385 to 512 cells, forward beyond 512, in float forward at 257
// to 512 and backward at 129 to 256, registers for one workgroup a CU (four wavefronts alone left room for two).
#include "residency.hpp"
#include <hip/hip_ext.h>
#include <mutex>

namespace blstm {
namespace {

constexpr int MAX_DEVICES = 64, LANES = 8;

// Launches that run one behind the other: those of one stream, or of several where there are more streams than lanes (each
// launch waits for its lane's last one).  done[now]: completion of the last one; held[now]: the most workgroups of one since the lane turned
// to this event.  The larger ones before that are complete with the other event, and had held[!now] at most.
struct Lane { hipStream_t stream; unsigned long long used; int now; hipEvent_t done[2]; int held[2]; };   // used: number of its last launch, 0: none
struct Device { int cus; unsigned long long launches; Lane lane[LANES]; };
std::mutex g_mutex;                                // held from the waits to the launch
Device g_device[MAX_DEVICES];                      // (the events are kept until the process ends)

hipError_t wait_for(Lane& l, int which, hipStream_t st) { return l.done[which] ? hipStreamWaitEvent(st, l.done[which], 0) : hipSuccess; }

// The stream's lane, or the one that has been idle for longest.
Lane& lane_of(Device& d, hipStream_t st) {
    Lane* oldest = &d.lane[0];
    for (Lane& l : d.lane) {
        if (l.used && l.stream == st) return l;
        if (l.used < oldest->used) oldest = &l;
    }
    return *oldest;
}

// Puts `grid` workgroups on the lane of the stream behind what they cannot run beside; *done is to signal their completion.
hipError_t take_turn(Device& d, int grid, hipStream_t st, hipEvent_t* done) {
    Lane& own = lane_of(d, st);
    own.used = ++d.launches;
    own.stream = st;
    hipError_t e = wait_for(own, own.now, st);     // (on one stream the order is there already, and this costs nothing)
    long long held = grid;
    for (Lane& l : d.lane) if (&l != &own) held += l.held[0] > l.held[1] ? l.held[0] : l.held[1];
    for (Lane& l : d.lane) {                       // the large launches of lanes that have gone over to smaller ones
        const int less = l.held[!l.now] - l.held[l.now];
        if (held <= d.cus || &l == &own || less <= 0 || e != hipSuccess) continue;
        e = wait_for(l, !l.now, st);
        held -= less;
    }
    bool behind[LANES] = {};
    while (held > d.cus && e == hipSuccess) {      // whole lanes, the one idle for longest (most likely complete) first
        int k = -1;
        for (int i = 0; i < LANES; ++i)
            if (&d.lane[i] != &own && !behind[i] && (k < 0 || d.lane[i].used < d.lane[k].used)) k = i;
        if (k < 0) break;                          // (behind all of them)
        behind[k] = true;
        e = wait_for(d.lane[k], d.lane[k].now, st);
        held -= d.lane[k].held[d.lane[k].now];
    }
    if (e != hipSuccess) return e;
    if (grid < own.held[own.now]) {                // (the last launch's completion is that of all before it)
        if (own.held[!own.now] > own.held[own.now]) own.held[own.now] = own.held[!own.now];
        own.now = !own.now;
    }
    if (!own.done[own.now]) e = hipEventCreateWithFlags(&own.done[own.now], hipEventDisableTiming | hipEventDisableSystemFence);
    own.held[own.now] = grid;
    *done = own.done[own.now];
    return e;
}

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
    Device& d = g_device[dev];
    if (d.cus == 0) e = hipDeviceGetAttribute(&d.cus, hipDeviceAttributeMultiprocessorCount, dev);
    hipEvent_t done = nullptr;
    if (e == hipSuccess) e = take_turn(d, grid, st, &done);
    if (e != hipSuccess) return e;
    e = hipExtLaunchKernel(kernel, dim3(grid), dim3(threads), args, dyn_lds, st, nullptr, done, 0);
    return e != hipSuccess ? e : hipGetLastError();
}

}  // namespace blstm
