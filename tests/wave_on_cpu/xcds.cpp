// one_xcd of csrc/xcd.hpp as host code: prints the answer, whether it was given up, the abort word, the loads.  xcds WHAT: a wavefront of one lane;
// xcds WHAT LANES: of several, a thread each.
#include <hip/hip_runtime.h>
#include <atomic>
#include <barrier>
#include <cstdio>
#include <string>
#include <thread>
#include <vector>
static int on_xcd = 3;
static std::barrier<>* wave = nullptr;                         // (several lanes)
static std::atomic<int> votes;
static thread_local struct { unsigned x; } this_lane;
static thread_local unsigned long long this_clock = 0;
static bool vote(bool v) {
    if (!wave) return v;
    if (!v) ++votes;
    wave->arrive_and_wait();
    const bool all = votes == 0;
    wave->arrive_and_wait();
    votes = 0;
    wave->arrive_and_wait();
    return all;
}
template <typename T> static T load_word(const T* p) { return wave ? __atomic_load_n(p, __ATOMIC_SEQ_CST) : past_the_caches(p); }
#undef __all
#define __all(x) vote(x)
#undef __hip_atomic_load
#define __hip_atomic_load(p, order, scope) load_word(p)
#define threadIdx this_lane
#define wall_clock64() (wave ? ++this_clock : ++clock_now)
#define __builtin_amdgcn_s_getreg(what) on_xcd
#define inline static inline
#include "xcd.hpp"
#undef inline
using namespace blstm;

static void several(const std::string& what, int lanes) {
    // groups of three slices: what each of them wrote
    unsigned table[3] = {3, 3, what == "other" ? 5u : what == "late" || what == "nothing" ? 0xFFFFFFFFu : 3u}, abort_word = what == "aborted" ? 1 : 0;
    if (what == "aborted") table[1] = 0xFFFFFFFFu;
    std::barrier<> all(lanes);
    wave = &all;
    std::vector<std::thread> threads;
    std::vector<int> near(lanes), gave_up(lanes);
    for (int k = 0; k < lanes; ++k) threads.emplace_back([&, k] {
        this_lane.x = k;
        bool g = true;
        // (every lane's clock goes the same way, as a wavefront's branches do)
        near[k] = one_xcd(table, 3, &abort_word, what == "late" ? 1000000 : 20, &g);
        gave_up[k] = g;
    });
    if (what == "late") __atomic_store_n(&table[2], 3u, __ATOMIC_SEQ_CST);
    for (std::thread& t : threads) t.join();
    for (int k = 1; k < lanes; ++k) if (near[k] != near[0] || gave_up[k] != gave_up[0]) { printf("lanes disagree\n"); return; }
    printf("%d %d %u 0\n", near[0], gave_up[0], abort_word);
}

int main(int argc, char** argv) {
    const std::string what = argv[1];
    if (argc > 2) { several(what, atoi(argv[2])); return 0; }
    unsigned table[2] = {0xFFFFFFFFu, 0xFFFFFFFFu}, abort_word = what == "aborted" ? 1 : 0;
    if (what == "same") tell_xcd(table, 0);
    if (what == "other") { on_xcd = 5; tell_xcd(table, 0); on_xcd = 3; }
    if (what == "late") on_load = [&](unsigned long long n) { if (n == 100) table[0] = 3; };
    bool gave_up = true;
    try {
        const bool near = one_xcd(what == "none" ? nullptr : table, what == "many" ? XCD_GROUP_MAX + 1 : 1, &abort_word, 20, &gave_up);
        printf("%d %d %u %llu\n", near, gave_up, abort_word, loads);
    } catch (too_many_loads) { printf("unbounded\n"); }
}
