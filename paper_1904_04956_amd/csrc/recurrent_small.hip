// Persistent recurrent kernels (bf16) for few sequences: all T frames of one layer, both directions, in one launch.
//
// The kernels of recurrent.hip give a workgroup 32 units of 32 rows; with few batch tiles most CUs have none, and a frame
// is a chain of latencies whose length is the work of one workgroup.  Here a workgroup has 16 units of 16 rows (MFMA
// 16x16x32) and a tile of its own for the whole launch: a quarter of the products, the partial sums, the cells (one
// per thread) and, backward, half of the operand bytes a frame.  Used while the workgroups fit the device at once.
//
// Four wavefronts split the contraction (forward: a quarter of h each; backward: one gate's rows of dE/da each), their
// slices of U_h (U_h^T) stay in registers.  The slice is the first operand of the products, so that a lane has neighbouring
// units of one row: the partial sums go through LDS in 16-byte words (forward the four gates of a unit).
// Four more wavefronts move what is not the exchange: they bring the inputs of four frames ahead into LDS and store what the others leave
// there.  A wavefront's memory answers come back in the order it asked, so with these loads and stores in its own queue a computing
// wavefront spent 540 clocks a frame on asking, and its next look at the operand stood behind their answers.
// The look is timed: PAUSE clocks behind the wavefront's own stores.  A look that comes too early costs a whole one more (the operand of all
// workgroups through the XCD's L2, forward 16 KB each and backward 64), so that looking straight away and even a cheap probe of the producers
// first lose to it.  us a layer of 21 frames, probe (four computing wavefronts that do it all) / PAUSE of 600 / 700 / 800 / 900 / 1000,
// backward: 8 sequences of 512 cells 45.6 / 40.7 / 39.0 / 39.5 / 39.9 / 40.8, 30 of 512 43 / 46 / 39 / 39 / 40 / 41, 80 of 384 41.8 / 45 / 35.5 / 34.8 / 36.4 / 37.2,
// 8 of 256 38.1 / 32.7 / 32.1 / 32.2 / 32.8 / 32.9, 20 of 640 48 / 57 / 49 / 45 / 43 / 44, 30 of 1024 68 / 72 / 58.6 / 58.5 / 59 / 60; forward, straight / 400 / 500 / 600: 8 of 512 31.3 / 30.4 / 31.2 / 31.6, 8 of 256 28 / 25.9 / 26.0 / 27.1, 30 of 1024 47 / 42.6 / 41.7 / 42.0 (launches
// alone; in a model's pass 8 of 512 gains 0.3).
// Narrow layers (these figures and the next from events around the launch, which add about two us): backward, probe / 300 / 400 / 500 / 600 / 700, 200 of 128 31.7 / 47 / 40 / 33.1 / 32.2 / 32.0, 64 of
// 128 28.0 / 30.9 / 29.7 / 29.5 / 29.9 / 30.3, 100 of 64 30.0 / 31.0 / 30.7 / 30.6 / 30.6 / 30.9, 250 of 64 28.7 / 28.9 / 28.9 / 29.1 / 29.5 / 30.1, 200 of 32 28.3 / 29.0 / 28.9 / 29.2 / 29.7 / 30.1, which
// slices built for 64 cells instead of 128 take to 27.4; forward, straight (four wavefronts) / 200 / 250 / 300 / 400, 84 of 96 27.6 / 27.9 / 27.8 / 28.0 / 28.6, 336 of 96 28.3 / 30.7 / 29.5 /
// 29.5 / 29.8, 200 of 128 28.4 / 30.8 / 29.4 / 29.3 / 29.7, 200 of 32 27.0 / 28.0 / 28.0 / 28.0 / 28.4.  (Forward, many sequences of 33 to 128 cells stay 1 to 1.5 us above the
// four wavefronts that did it all, unless the L2 serves them.)
// Through the XCD's L2 (NEAR, see xcd.hpp), where the contiguous eighths of the grid are whole groups: forward, straight, 64 of 512 32.8 -> 29.7 (far 31.8), 50 of
// 320 28.5 -> 26.2, 128 of 256 27.4 -> 25.2; backward of 385 to 512 cells, 200 clocks behind the stores, 64 of 512 47.8 -> 40.3 (far 42.2), and of up to 128 cells, straight, where the far look loses
// to the probe: events, probe / far / near 64 of 128 28.0 / 29.2 / 26.0, 253 of 128 28.8 / 29.6 / 27.1, 256 of 64 28.6 / 29.6 / 24.8, 512 of 32 28.4 / 29.4 / 24.5.  Between these widths the far look
// gains by itself (50 of 320 43 / 38.3 / 34.7, 64 of 256 38.1 / 33.9 / 30.4, 64 of 384 45 / 37.6 / 35.1), and the L2 is not asked for.
//
// Exchange copies in the order of the fragments: [frame][direction][16-row
// tile]([gate])[32 columns][4][16 rows][8], a fragment load is one contiguous KB, a workgroup writes half of one.  The
// slices are whole pairs, so every block is written; units beyond H are zeros with zero weights, rows beyond the batch
// repeat its last row, and neither is stored row-major.  H a multiple of 8; protocol, bounded waits and failures as in
// recurrent.hip.  Saved activations are per-thread records: [frame][direction][tile][slice][thread].
#include "exchange.hpp"
#include "kernels.hpp"
#include "residency.hpp"
#include "xcd.hpp"

namespace blstm {
namespace {

constexpr int NWF = 4;                                   // wavefronts that compute, and as many that move what the exchange is not
constexpr int PAIR = 4 * 16 * 8;                         // elements of 32 columns of a tile (1 KB)
constexpr int SC1 = 16;                                  // cache policy of agent-scope accesses

// Workgroup -> (direction, tile, slice); each XCD (ids are dealt round-robin) takes a contiguous eighth of the sequence.
struct Spot { int d, tile, u, group; bool real; };
__device__ __forceinline__ Spot spot(int nu, int ntiles) {
    const int s = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
    Spot p;
    p.real = s < 2 * nu * ntiles;
    p.group = s / nu;
    p.u = s - p.group * nu; p.d = p.group / ntiles; p.tile = p.group - p.d * ntiles;
    return p;
}
__device__ __forceinline__ void st_exchange(bool write_back, bf16_t* p, const uint2& v) {
    if (write_back) *reinterpret_cast<uint2*>(p) = v; else st_coh_8B(p, v);
}
// f[q] = the 16 bytes at byte off(q) of a (frame, direction, tile) of the exchange copy, when every element is written: a look PAUSE clocks after
// `stored`, through the L2 (which then fetches a line once for all of its CUs) or, NEAR, past the L1, and again past the caches until
// nothing is missing.  Returns true if the wait was abandoned.
template <int PAUSE, bool NEAR, int N, typename F>
__device__ __forceinline__ bool operand(uint4 (&f)[N], const bf16_t* base, unsigned bytes, F off, unsigned long long stored, unsigned* abort_word, unsigned long long limit) {
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(base), 0, (int)bytes, 0x00020000);
    if constexpr (PAUSE > 0) while (__builtin_amdgcn_s_memtime() - stored < PAUSE) {}
#pragma unroll
    for (int q = 0; q < N; ++q) f[q] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off(q), 0, NEAR ? SC1 : 0));
    return wait_written<!NEAR, N>(f, [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < N; ++q) f[q] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off(q), 0, SC1));
    }, false, abort_word, limit);
}
// Four neighbouring lanes with four 16-bit values each, (a.lo, a.hi, b.lo, b.hi): lane k gets value k of each of them, in their order.
__device__ __forceinline__ uint2 quad_transpose(unsigned a, unsigned b) {
    const bool odd = threadIdx.x & 1, high = threadIdx.x & 2;
    const unsigned an = __builtin_amdgcn_update_dpp(0u, a, 0xB1, 0xF, 0xF, true), bn = __builtin_amdgcn_update_dpp(0u, b, 0xB1, 0xF, 0xF, true);   // quad_perm 1,0,3,2
    const unsigned p = odd ? __builtin_amdgcn_perm(a, an, 0x07060302u) : __builtin_amdgcn_perm(an, a, 0x05040100u);
    const unsigned q = odd ? __builtin_amdgcn_perm(b, bn, 0x07060302u) : __builtin_amdgcn_perm(bn, b, 0x05040100u);
    const unsigned x = __builtin_amdgcn_update_dpp(0u, high ? p : q, 0x4E, 0xF, 0xF, true);   // quad_perm 2,3,0,1
    return high ? make_uint2(x, q) : make_uint2(p, x);
}
// The value of four neighbouring lanes (units 4k .. 4k + 3 of one row) as four bf16, in the first of them.
__device__ __forceinline__ uint2 quad_pack(unsigned own) {
    const unsigned one = __builtin_amdgcn_update_dpp(0u, own, 0xB1, 0xF, 0xF, true);       // quad_perm 1,0,3,2
    const unsigned two = own | (one << 16);                                                // (in even lanes)
    return make_uint2(two, __builtin_amdgcn_update_dpp(0u, two, 0x4E, 0xF, 0xF, true));    // quad_perm 2,3,0,1
}

// ------------------------------------------------------------------------------ forward
// Width up to 128 NQ; each computing wavefront contracts 32 NQ columns.
constexpr int FROW = 17;                                 // float4 of a row of a partial tile: (i, f, g, o) of sixteen units, and one to turn the banks
template <int NQ, bool NEAR>
__global__ __launch_bounds__(128 * NWF) void rec_small_fwd_kernel(RecFwdArgs a) {
    __shared__ float4 part[2][NWF][16 * FROW], axs[2][64 * NWF];
    __shared__ uint4 out[2][64 * NWF];                   // gates, cell state, h of a cell
    const int T = a.T, B = a.B, H = a.H;
    const int blocks = (H + 31) / 32, nu = 2 * blocks, NT = (B + 15) / 16;
    const Spot sp = spot(nu, NT);
    const int tid = threadIdx.x & (64 * NWF - 1), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int d = sp.d, u = sp.u, tile = sp.tile, l16 = lane & 15;
    // this thread's cell: unit j, row r of the tile
    const int r = tid >> 4, j = u * 16 + l16;
    const bool junit = j < H;
    auto frame = [&](int n) { return d ? T - 1 - n : n; };
    if (wave >= NWF) {
        // this workgroup's share of the region to fill, some words every frame
        const unsigned long long share = a.fill ? (a.fill_words + gridDim.x - 1) / gridDim.x : 0ull;
        const unsigned long long first = min(a.fill_words, (unsigned long long)blockIdx.x * share);
        uint4* const fill = static_cast<uint4*>(a.fill) + first;
        const unsigned fill_end = (unsigned)(min(a.fill_words, first + share) - first);
        unsigned fill_pos = tid;
        const int fill_each = (int)((share + (unsigned long long)(256 * T) - 1) / (unsigned long long)(256 * T));
        auto fill_some = [&](int words) { for (int k = 0; k < words && fill_pos < fill_end; ++k, fill_pos += 256) fill[fill_pos] = make_uint4(~0u, ~0u, ~0u, ~0u); };
        if (!sp.real) { fill_some(1 << 30); return; }
        const int row = tile * 16 + r;
        const float* ax0 = a.ax + (size_t)min(row, B - 1) * 8 * H + d * 4 * H + min(j, H - 1);
        auto inputs = [&](int n, float4& v) __attribute__((always_inline)) {
            const float* p = ax0 + (size_t)frame(min(n, T - 1)) * B * 8 * H;
            v = make_float4(p[0], p[(size_t)H], p[2 * (size_t)H], p[3 * (size_t)H]);
        };
        auto save = [&](int n) __attribute__((always_inline)) {
            const uint4 v = out[n & 1][tid];
            const size_t rec = ((size_t)(frame(n) * 2 + d) * NT + tile) * nu + u;
            reinterpret_cast<uint2*>(a.gates)[rec * 256 + tid] = make_uint2(v.x, v.y);
            a.c[rec * 256 + tid] = __builtin_bit_cast(float, v.z);
            const uint2 hq = quad_pack(v.w);
            if ((tid & 3) == 0 && junit && row < B) {
                const size_t at = ((size_t)frame(n) * B + row) * 2 * H + d * H + j;
                *reinterpret_cast<uint2*>(a.y + at) = hq;
                if (a.z) *reinterpret_cast<uint2*>(a.z + at) = hq;
            }
        };
        float4 in[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) inputs(k, in[k]);
        for (int n0 = 0; n0 < T; n0 += 4) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int n = n0 + k;
                if (n >= T) break;
                axs[n & 1][tid] = in[k];
                lds_barrier();
                inputs(n + 4, in[k]);
                if (n > 0) save(n - 1);
                fill_some(fill_each);
            }
        }
        lds_barrier();
        save(T - 1);
        fill_some(1 << 30);
        return;
    }
    if (!sp.real) return;
    unsigned* const xcds = NEAR && a.xcd ? a.xcd + sp.group * nu : nullptr;
    tell_xcd(xcds, u);
    const int lq = lane >> 4;
    uint4 wf[4][NQ];
    {
        const int unit = u * 16 + l16;
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const int k = (wave * NQ + q) * 32 + 8 * lq;
                wf[g][q] = unit < H && k < H ? *reinterpret_cast<const uint4*>(a.uh[d] + (size_t)(g * H + unit) * H + k) : make_uint4(0u, 0u, 0u, 0u);
            }
    }
    auto off = [&](int q) { return (unsigned)(min(wave * NQ + q, blocks - 1) * PAIR + lane * 8) * 2; };
    const unsigned x_off = (unsigned)(u >> 1) * PAIR + ((2 * (u & 1) + (l16 >> 3)) * 16 + r) * 8 + (l16 & 7);
    float c = 0.0f;
    float poison = ld_coh_u32(a.abort_word) != 0 ? __builtin_nanf("") : 0.0f;
    bool lost;
    const bool near = one_xcd(xcds, nu, a.abort_word, a.limit_ticks, &lost);
    if (lost) poison = __builtin_nanf("");
    unsigned long long stored = 0;                       // when the last h went out
    for (int n = 0; n < T; ++n) {
        float4 sum = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (n > 0) {
            uint4 af[NQ];
            if (operand<NEAR ? 0 : NQ == 1 ? 300 : 400, NEAR, NQ>(af, a.hx + ((size_t)(frame(n - 1) * 2 + d) * NT + tile) * blocks * PAIR, blocks * PAIR * 2, off, stored, a.abort_word, a.limit_ticks)) poison = __builtin_nanf("");
            // rows of the products: the slice's units; columns: the tile's rows
            f32x4_t acc[4];
#pragma unroll
            for (int g = 0; g < 4; ++g)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[g][e] = 0.0f;
#pragma unroll
            for (int q = 0; q < NQ; ++q)
#pragma unroll
                for (int g = 0; g < 4; ++g) acc[g] = mfma16(wf[g][q], af[q], acc[g]);
#pragma unroll
            for (int e = 0; e < 4; ++e) part[n & 1][wave][l16 * FROW + 4 * lq + e] = make_float4(acc[0][e], acc[1][e], acc[2][e], acc[3][e]);
        }
        lds_barrier();                                   // one a frame: everything in LDS is there twice
        const float4 ax = axs[n & 1][tid];
        if (n > 0) {
            float4 v[NWF];
#pragma unroll
            for (int w = 0; w < NWF; ++w) v[w] = part[n & 1][w][r * FROW + l16];
#pragma unroll
            for (int w = 0; w < NWF; ++w) { sum.x += v[w].x; sum.y += v[w].y; sum.z += v[w].z; sum.w += v[w].w; }
        }
        const float gi = fast_sigmoid((junit ? ax.x : 0.0f) + sum.x), gf = fast_sigmoid((junit ? ax.y : 0.0f) + sum.y);
        const float gg = fast_tanh((junit ? ax.z : 0.0f) + sum.z), go = fast_sigmoid((junit ? ax.w : 0.0f) + sum.w);
        c = next_cell(gf, c, gi, gg);
        const unsigned h = coh_bf16(go * fast_tanh(c) + poison);
        const uint2 hq = quad_pack(h);
        if ((tid & 3) == 0) st_exchange(near, a.hx + ((size_t)(frame(n) * 2 + d) * NT + tile) * blocks * PAIR + x_off, hq);
        stored = __builtin_amdgcn_s_memtime();
        out[n & 1][tid] = make_uint4(pack_bf2(gi, gf), pack_bf2(gg, go), __builtin_bit_cast(unsigned, c), h);
    }
    lds_barrier();
}

// ------------------------------------------------------------------------------ backward
// Width up to 32 NQ; computing wavefront w contracts gate w's columns of dE/da.
// NEAR: whole groups an eighth of the grid, of up to 128 or 385 to 512 cells (see the head of this file); groups of at most 32 slices.
constexpr int BROW = 20;                                 // floats of a row of a partial tile
template <int NQ, bool NEAR>
__global__ __launch_bounds__(128 * NWF) void rec_small_bwd_kernel(RecBwdArgs a) {
    constexpr int PAUSE = NEAR ? (NQ <= 4 ? 0 : 200) : NQ <= 2 ? 400 : NQ <= 4 ? 550 : NQ <= 16 ? 800 : NQ <= 24 ? 900 : 700;   // (see the head of this file)
    __shared__ float part[2][NWF][16 * BROW];
    __shared__ uint4 in_s[2][64 * NWF];                  // gates, dy, the cell state before
    __shared__ uint2 out[2][64 * NWF];                   // dE/da: gate tid % 4 of four units
    const int T = a.T, B = a.B, H = a.H;
    const int blocks = (H + 31) / 32, nu = 2 * blocks, NT = (B + 15) / 16;
    const Spot sp = spot(nu, NT);
    if (!sp.real) return;
    const int d = sp.d, u = sp.u, tile = sp.tile;
    const int tid = threadIdx.x & (64 * NWF - 1), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, lq = lane >> 4;
    const int r = tid >> 4, j = u * 16 + l16;
    const bool junit = j < H;
    auto frame = [&](int k) { return d ? k : T - 1 - k; };   // (the last one visited forward comes first)
    auto record = [&](int t) { return (((size_t)(t * 2 + d) * NT + tile) * nu + u) * 256 + tid; };
    const float* const c_first = a.c + record(frame(0));
    if (wave >= NWF) {
        const int row = tile * 16 + r;
        const bf16_t* dy0 = a.dy + (size_t)min(row, B - 1) * 2 * H + d * H + min(j, H - 1);
        struct In { uint2 g; bf16_t dy; float cp; };
        auto inputs = [&](int k0, In& in) __attribute__((always_inline)) {
            const int k = min(k0, T - 1), t = frame(k);
            in.dy = dy0[(size_t)t * B * 2 * H];
            in.g = reinterpret_cast<const uint2*>(a.gates)[record(t)];
            in.cp = a.c[record(frame(min(k + 1, T - 1)))];
        };
        bf16_t* const da0 = a.da + (size_t)row * 8 * H + (size_t)d * 4 * H + (size_t)(tid & 3) * H + (j & ~3);
        auto save = [&](int k) __attribute__((always_inline)) {
            const uint2 v = out[k & 1][tid];
            if (junit && row < B) *reinterpret_cast<uint2*>(da0 + (size_t)frame(k) * B * 8 * H) = v;
        };
        In in[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) inputs(k, in[k]);
        for (int k0 = 0; k0 < T; k0 += 4) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int k = k0 + i;
                if (k >= T) break;
                // (the frame visited first forward has no cell state before it)
                in_s[k & 1][tid] = make_uint4(in[i].g.x, in[i].g.y, in[i].dy, k < T - 1 ? __builtin_bit_cast(unsigned, in[i].cp) : 0u);
                lds_barrier();
                inputs(k + 4, in[i]);
                if (k > 0) save(k - 1);
            }
        }
        lds_barrier();
        save(T - 1);
        return;
    }
    unsigned* const xcds = NEAR && a.xcd ? a.xcd + sp.group * nu : nullptr;
    tell_xcd(xcds, u);
    uint4 wf[NQ];
    {
        const int unit = u * 16 + l16;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int k = q * 32 + 8 * lq;
            wf[q] = unit < H && k < H ? *reinterpret_cast<const uint4*>(a.uht[d] + (size_t)unit * 4 * H + wave * H + k) : make_uint4(0u, 0u, 0u, 0u);
        }
    }
    auto off = [&](int q) { return (unsigned)((wave * blocks + min(q, blocks - 1)) * PAIR + lane * 8) * 2; };
    const size_t XT = (size_t)4 * blocks * PAIR;
    // (lane k of four has gate k of their four units)
    const unsigned x_off = ((unsigned)(tid & 3) * blocks + (u >> 1)) * PAIR + ((2 * (u & 1) + (l16 >> 3)) * 16 + r) * 8 + (l16 & 4);
    float c = *c_first, dcn = 0.0f;                      // this frame's cell state (then the one before's), carried dE/dc
    float poison = ld_coh_u32(a.abort_word) != 0 ? __builtin_nanf("") : 0.0f;
    bool lost;
    const bool near = one_xcd(xcds, nu, a.abort_word, a.limit_ticks, &lost);
    if (lost) poison = __builtin_nanf("");
    unsigned long long stored = 0;                       // when the last dE/da went out
    for (int k = 0; k < T; ++k) {
        float dh = 0.0f;
        if (k > 0) {
            const bf16_t* const base = a.dax + ((size_t)(frame(k - 1) * 2 + d) * NT + tile) * XT;
            f32x4_t acc[2];
#pragma unroll
            for (int e = 0; e < 4; ++e) { acc[0][e] = 0.0f; acc[1][e] = 0.0f; }
            if constexpr (NQ <= 24) {
                uint4 af[NQ];
                if (operand<PAUSE, NEAR, NQ>(af, base, (unsigned)XT * 2, off, stored, a.abort_word, a.limit_ticks)) poison = __builtin_nanf("");
#pragma unroll
                for (int q = 0; q < NQ; ++q) acc[q & 1] = mfma16(wf[q], af[q], acc[q & 1]);
            } else {                                     // (no registers for all of it: half by half)
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    uint4 af[NQ / 2];
                    if (operand<PAUSE, NEAR, NQ / 2>(af, base, (unsigned)XT * 2, [&](int q) { return off(s * (NQ / 2) + q); }, stored, a.abort_word, a.limit_ticks)) poison = __builtin_nanf("");
#pragma unroll
                    for (int q = 0; q < NQ / 2; ++q) acc[(s * (NQ / 2) + q) & 1] = mfma16(wf[s * (NQ / 2) + q], af[q], acc[(s * (NQ / 2) + q) & 1]);
                }
            }
            *reinterpret_cast<float4*>(&part[k & 1][wave][l16 * BROW + 4 * lq]) = make_float4(acc[0][0] + acc[1][0], acc[0][1] + acc[1][1], acc[0][2] + acc[1][2], acc[0][3] + acc[1][3]);
        }
        lds_barrier();
        const uint4 in = in_s[k & 1][tid];
        if (k > 0) {
            float v[NWF];
#pragma unroll
            for (int w = 0; w < NWF; ++w) v[w] = part[k & 1][w][r * BROW + l16];
#pragma unroll
            for (int w = 0; w < NWF; ++w) dh += v[w];
        }
        const float gi = bf2f((bf16_t)(in.x & 0xFFFFu)), gf = bf2f((bf16_t)(in.x >> 16));
        const float gg = bf2f((bf16_t)(in.y & 0xFFFFu)), go = bf2f((bf16_t)(in.y >> 16));
        const float cp = __builtin_bit_cast(float, in.w);
        const float dht = dh + (junit ? bf2f((bf16_t)in.z) : 0.0f) + poison;
        const float tc = fast_tanh(c);
        const float dc = dht * go * (1.0f - tc * tc) + dcn;
        const unsigned fi = (unsigned)coh_bf16(dc * gg * gi * (1.0f - gi)) | ((unsigned)coh_bf16(dc * cp * gf * (1.0f - gf)) << 16);
        const unsigned og = (unsigned)coh_bf16(dc * gi * (1.0f - gg * gg)) | ((unsigned)coh_bf16(dht * tc * go * (1.0f - go)) << 16);
        const uint2 da = quad_transpose(fi, og);
        st_exchange(near, a.dax + ((size_t)(frame(k) * 2 + d) * NT + tile) * XT + x_off, da);
        stored = __builtin_amdgcn_s_memtime();
        out[k & 1][tid] = da;
        dcn = dc * gf; c = cp;
    }
    lds_barrier();
}

template <auto KERNEL, typename A>
hipError_t run(const A& a, hipStream_t st, bool* launched) {
    const int real = 2 * 2 * ((a.H + 31) / 32) * ((a.B + 15) / 16);
    return launch_resident<KERNEL>(a, 128 * NWF, 0, (real + 7) & ~7, real, st, launched);
}
template <int NQ>
hipError_t run_fwd(const RecFwdArgs& a, hipStream_t st, bool* launched) {
    // (eighths of the grid that are whole groups: a direction's tiles are a multiple of four)
    return (a.B + 15) / 16 % 4 == 0 ? run<rec_small_fwd_kernel<NQ, true>>(a, st, launched) : run<rec_small_fwd_kernel<NQ, false>>(a, st, launched);
}
template <int NQ>
hipError_t run_bwd(const RecBwdArgs& a, hipStream_t st, bool* launched) {
    if constexpr (NQ <= 4 || NQ == 16) if ((a.B + 15) / 16 % 4 == 0) return run<rec_small_bwd_kernel<NQ, true>>(a, st, launched);
    return run<rec_small_bwd_kernel<NQ, false>>(a, st, launched);
}

}  // namespace

// Every workgroup on a CU of its own.  Measured, two layers, T = 21, forward / whole step in us, the kernels of
// recurrent.hip against these: H = 512, 32 sequences 177 / 578 against 93 / 286, 64 sequences 186 / 576 against 104 / 342
// (products included, which ran slower beside the former); H = 256, 128 sequences 147 / 339 against 93 / 275.  Two
// workgroups per CU lose it again, backward above all: H = 512, 128 sequences 198 / 496 against 204 / 661.
bool rec_small_supported(int B, int H) { return rec_supported(H) && 4 * ((H + 31) / 32) * ((B + 15) / 16) <= 256; }

hipError_t launch_rec_small_fwd(const RecFwdArgs& a, hipStream_t st, bool* launched) {
    *launched = false;
#define BLSTM_SMALL(NQ) if (a.H <= 128 * NQ) return run_fwd<NQ>(a, st, launched)
    BLSTM_SMALL(1); BLSTM_SMALL(2); BLSTM_SMALL(3); BLSTM_SMALL(4); BLSTM_SMALL(5); BLSTM_SMALL(6); BLSTM_SMALL(7); BLSTM_SMALL(8);
#undef BLSTM_SMALL
    return hipSuccess;
}
hipError_t launch_rec_small_bwd(const RecBwdArgs& a, hipStream_t st, bool* launched) {
    *launched = false;
#define BLSTM_SMALL(NQ) if (a.H <= 32 * NQ) return run_bwd<NQ>(a, st, launched)
    BLSTM_SMALL(2); BLSTM_SMALL(4); BLSTM_SMALL(8); BLSTM_SMALL(12); BLSTM_SMALL(16); BLSTM_SMALL(20); BLSTM_SMALL(24); BLSTM_SMALL(28); BLSTM_SMALL(32);
#undef BLSTM_SMALL
    return hipSuccess;
}

}  // namespace blstm
