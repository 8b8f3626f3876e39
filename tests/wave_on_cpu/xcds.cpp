// one_xcd of csrc/xcd.hpp as host code, a wavefront of one lane: prints the answer, whether it was given up, the abort word, the loads.
#include <hip/hip_runtime.h>
#include <cstdio>
#include <string>
static int on_xcd = 3;
#define __builtin_amdgcn_s_getreg(what) on_xcd
#define inline static inline
#include "xcd.hpp"
#undef inline
using namespace blstm;

int main(int argc, char** argv) {
    const std::string what = argv[1];
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
