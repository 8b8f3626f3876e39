// The bounded waits of the persistent kernels, one call each: prints result, abort word, loads, whether the data came whole.  waits WHAT [few | float]: as the
// kernels on 16-row tiles and of the wide layers wait (a first look, then wait_written), or as those for few sequences do (the probe of the
// producers, a look, then settle16), or as the float ones do (a look, then wait_written32; every element is half of a word).
#include "exchange.hpp"
#include <cstdio>
#include <cstring>
#include <string>
using namespace blstm;

int main(int argc, char** argv) {
    const std::string what = argv[1];
    const std::string who = argc > 2 ? argv[2] : "";
    constexpr int N = 4;
    alignas(16) static bf16_t data[N * 8 + 8];
    for (bf16_t& e : data) e = 0x3F80;
    const bf16_t* probe = data + N * 8;                        // (a word of its own: the last a producer writes)
    auto off = [](int q) { return q * 8; };
    unsigned abort_word = 0;
    bool gave_up = false;
    if (what == "nothing") memset(data, 0xFF, sizeof data);                                            // nobody writes
    if (what == "rest" || what == "rest, aborted") data[11] = 0xFFFF;                                  // the probed word is there, one other element never comes
    if (what == "rest, aborted") on_load = [&](unsigned long long n) { if (n == 500) abort_word = 1; };   // (raised by another workgroup)
    if (what == "late") { memset(data, 0xFF, sizeof data); on_load = [&](unsigned long long n) { if (n == 100) data[32] = data[33] = 0; if (n == 300) memset(data, 0, sizeof data); }; }
    if (what == "given up") { data[3] = 0xFFFF; gave_up = true; }
    if (who == "float" && (what == "rest" || what == "rest, aborted" || what == "given up")) data[2] = data[3] = data[10] = data[11] = 0xFFFF;   // (half a word is not the pattern)
    const unsigned long long limit = what == "rest, aborted" ? ~0ull >> 1 : 20;
    uint4 f[N];
    try {
        bool r;
        if (who == "few") {
            r = gave_up || probe_producers16(probe, true, &abort_word, limit);
            look16<N>(f, data, off);
            r = settle16<N>(f, data, off, r, &abort_word, limit);
        } else if (who == "float") {
            look16<N>(f, data, off);
            r = wait_written32<N>(f, [&]() { for (int q = 0; q < N; ++q) f[q] = ld_coh_16B(data + off(q)); }, gave_up, &abort_word, limit);
            printf("%d %u %llu %d\n", r, abort_word, loads, all_written32<N>(f));
            return 0;
        } else {
            look16<N>(f, data, off);
            r = wait_written<false, N>(f, [&]() { for (int q = 0; q < N; ++q) f[q] = ld_coh_16B(data + off(q)); }, gave_up, &abort_word, limit);
        }
        printf("%d %u %llu %d\n", r, abort_word, loads, all_written<N>(f));
    } catch (too_many_loads) { printf("unbounded\n"); }
}
