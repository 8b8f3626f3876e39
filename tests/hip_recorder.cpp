// A stand-in for the HIP runtime's entry points that the library uses: no device, every launch is written down.  Loaded
// before the library, it lets the host code that picks and prepares launches be tested without a GPU.
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>
#include <vector>

struct dim3 { uint32_t x, y, z; };
struct Launch { std::string name; dim3 grid; bool timed; };
static std::map<const void*, std::string> g_names;
static std::vector<Launch> g_launches;
static std::map<int, int> g_cus;
static std::vector<std::pair<std::string, int>> g_occupancy;
static std::string g_fail;
// Persistent launches in the order they were made: each one's workgroups and the earlier ones it is behind; the ones that are
// complete with an event, and before whatever is next on a stream.
static std::vector<std::pair<int, std::set<int>>> g_persistent;
static std::map<void*, std::set<int>> g_with_event, g_before;
static void* g_capturing = nullptr;
static unsigned long long g_captures = 0;
static int g_device = 0, g_error = 0, g_events = 0, g_occupancy_asked = 0;
static struct { dim3 grid, block; size_t lds; void* stream; } g_config;

extern "C" {

void recorder_reset() { g_launches.clear(); g_cus.clear(); g_occupancy.clear(); g_fail.clear(); g_device = 0; g_error = 0; g_events = 0; }
void recorder_clear() { g_launches.clear(); g_events = 0; }
void recorder_device(int device) { g_device = device; }
void recorder_cus(int device, int cus) { g_cus[device] = cus; }
void recorder_occupancy(const char* part_of_name, int per_cu) { g_occupancy.emplace_back(part_of_name, per_cu); }
void recorder_fail(const char* part_of_name) { g_fail = part_of_name; }   // "" = none
int recorder_count() { return (int)g_launches.size(); }
const char* recorder_name(int i) { return g_launches[i].name.c_str(); }
unsigned recorder_grid(int i, int axis) { const dim3& g = g_launches[i].grid; return axis == 0 ? g.x : axis == 1 ? g.y : g.z; }
int recorder_persistent() { return (int)g_persistent.size(); }
int recorder_workgroups(int i) { return g_persistent[i].first; }
int recorder_behind(int i, int j) { return (int)g_persistent[i].second.count(j); }
void recorder_capturing(void* stream) { g_capturing = stream; ++g_captures; }   // a capture of its own
int recorder_occupancy_asked() { return g_occupancy_asked; }
int recorder_timed(int i) { return g_launches[i].timed; }         // between the two events of a pair

void** __hipRegisterFatBinary(const void*) { static void* handle; return &handle; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { g_names[host] = name; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void* stream) { g_config = {grid, block, lds, stream}; return 0; }
int __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, void** stream) {
    *grid = g_config.grid; *block = g_config.block; *lds = g_config.lds; *stream = g_config.stream;
    return 0;
}
int hipLaunchKernel(const void* f, dim3 grid, dim3, void**, size_t, void* stream) {
    const std::string name = g_names.count(f) ? g_names[f] : "?";
    if (!g_fail.empty() && name.find(g_fail) != std::string::npos) return g_error = 719;
    if (name.find("rec_") != std::string::npos || name.find("rec32_") != std::string::npos) {
        const int n = (int)g_persistent.size();
        g_persistent.push_back({(int)grid.x, g_before[stream]});
        g_before[stream].insert(n);
    }
    g_launches.push_back({name, grid, (g_events & 1) != 0});
    return 0;
}
int hipExtLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t lds, void* stream, void*, void* stop, int) {
    const int e = hipLaunchKernel(f, grid, block, args, lds, stream);
    if (e == 0 && stop) g_with_event[stop] = g_before[stream];
    return e;
}
int hipStreamWaitEvent(void* stream, void* event, unsigned) {
    g_before[stream].insert(g_with_event[event].begin(), g_with_event[event].end());
    return 0;
}
int hipStreamIsCapturing(void* stream, int* status) { *status = stream != nullptr && stream == g_capturing; return 0; }
int hipStreamGetCaptureInfo(void* stream, int* status, unsigned long long* id) { *status = stream != nullptr && stream == g_capturing; *id = g_captures; return 0; }
int hipEventCreateWithFlags(void** e, unsigned) { *e = malloc(1); return 0; }
int hipGetLastError() { const int e = g_error; g_error = 0; return e; }
const char* hipGetErrorString(int) { return "recorded failure"; }
int hipGetDevice(int* d) { *d = g_device; return 0; }
int hipDeviceGetAttribute(int* v, int, int device) { *v = g_cus.count(device) ? g_cus[device] : 256; return 0; }
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int, size_t) {
    *n = 1;
    ++g_occupancy_asked;
    for (auto& o : g_occupancy) if (g_names[f].find(o.first) != std::string::npos) *n = o.second;
    return 0;
}
int hipEventCreate(void** e) { *e = malloc(1); return 0; }
int hipEventDestroy(void* e) { free(e); return 0; }
int hipEventRecord(void*, void*) { ++g_events; return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*) { *ms = 1.0f; return 0; }
int hipGetSymbolAddress(void** p, const void*) { *p = reinterpret_cast<void*>(uintptr_t(1) << 40); return 0; }
int hipMemcpy(void* dst, const void*, size_t n, int) { memset(dst, 0, n); return 0; }
int hipMemcpyAsync(void*, const void*, size_t, int, void*) { g_launches.push_back({"hipMemcpyAsync", {1, 1, 1}, (g_events & 1) != 0}); return 0; }
int hipStreamSynchronize(void*) { return 0; }

}  // extern "C"
