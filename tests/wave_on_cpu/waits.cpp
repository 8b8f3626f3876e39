// The bounded waits of the persistent kernels, one call each: prints result, abort word, loads, whether the data came whole.  waits WHAT [few | float]: a
// first look, by ordinary loads, then what the kernels call behind it: wait_written without a nap, as on 16-row tiles, in the wide layers and, through the
// L2, for few sequences; with one, as for few sequences elsewhere; or wait_written32, as in float.
#include "exchange.hpp"
#include <cstdio>
#include <cstring>
#include <string>
using namespace blstm;

int main(int argc, char** argv) {
    const std::string what = argv[1];
    const std::string who = argc > 2 ? argv[2] : "";
    constexpr int N = 4;
    alignas(16) static bf16_t data[N * 8];
    for (bf16_t& e : data) e = 0x3F80;
    unsigned abort_word = 0;
    bool gave_up = false;
    if (what == "nothing") memset(data, 0xFF, sizeof data);                                            // nobody writes
    if (what == "rest" || what == "rest, aborted") data[11] = 0xFFFF;                                  // one element never comes
    if (what == "rest, aborted") on_load = [&](unsigned long long n) { if (n == 500) abort_word = 1; };   // (raised by another workgroup)
    if (what == "late") { memset(data, 0xFF, sizeof data); on_load = [&](unsigned long long n) { if (n == 100) data[24] = data[25] = 0; if (n == 300) memset(data, 0, sizeof data); }; }
    if (what == "given up") { data[3] = 0xFFFF; gave_up = true; }
    if (who == "float" && (what == "rest" || what == "rest, aborted" || what == "given up")) data[2] = data[3] = data[10] = data[11] = 0xFFFF;   // (half a word is not the pattern)
    const unsigned long long limit = what == "rest, aborted" ? ~0ull >> 1 : 20;
    uint4 f[N];
    try {
        memcpy(f, data, sizeof f);
        auto look = [&]() { for (int q = 0; q < N; ++q) f[q] = ld_coh_16B(data + q * 8); };
        const bool r = who == "few" ? wait_written<true, N>(f, look, gave_up, &abort_word, limit)
                     : who == "float" ? wait_written32<N>(f, look, gave_up, &abort_word, limit) : wait_written<false, N>(f, look, gave_up, &abort_word, limit);
        printf("%d %u %llu %d\n", r, abort_word, loads, who == "float" ? all_written32<N>(f) : all_written<N>(f));
    } catch (too_many_loads) { printf("unbounded\n"); }
}
