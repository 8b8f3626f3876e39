// Persistent recurrent kernels (bf16) on 16-row batch tiles: all T frames of one layer, both directions, in one launch.
//
// A workgroup of four wavefronts has 16 NB units (32 or 64) of a 16-row tile.  Against 32 units of 32 rows
// (recurrent.hip) the slice of 64 units reads half of the operand bytes per cell (backward 64 KB a frame instead of 128 KB at
// 512 cells, the longest part of its frame), and half as many workgroups wait on each other.
//
// Forward: MFMA 16x16x32 with U_h as the first operand, its rows ordered so that a lane gets the four gates of NB
// neighbouring units of one batch row: the cell arithmetic follows the products in the same registers, without partial
// sums and without regrouping, and a_x, h and the records move in one access of NB values each.  Every wavefront needs the
// whole of h: each checks its quarter of the fragments, stages them in LDS, multiplies them from registers, and reads the
// other quarters behind the barrier.  Backward: the wavefronts split the contraction by the producing units, their partial
// sums meet in LDS in the same (unit, row) order, and an exchange between lane groups (v_permlane*_swap) leaves each
// lane with eight units of one gate: 16-byte stores.  The number of vector-memory instructions a frame is what the layout
// is made for: one costs a CU's memory pipeline about the same whatever its width.
//
// Exchange copies: [frame][direction][16-row tile]([gate])[8 columns][16 rows][8], a fragment of 32 columns is one contiguous
// KB.  A lane's units lie in one group of eight and H is a multiple of 8: they exist or not together, and what lies beyond H
// is neither written nor read (the last columns repeat there, against zero weights).  Rows beyond the batch repeat its last
// row and are not stored row-major.  Saved activations are per-lane records in the order of the units.
// Both protocols, bounded waits and failures as in recurrent.hip.
//
// The memory's answers come back to a wavefront in the order it asked, and a look at the exchanged operand that comes too early costs a round trip more.
// So the next frame's inputs (a_x; dy, gates, cell states) are asked for behind the operand's arrival and before h or dE/da goes
// out: they are back when the next look is due.  Row-major tensors move in whole lines, turned in LDS (see `turned`), the frame's h and
// dE/da a frame later behind the barrier that is there anyway; every lane issues every load and store (see recurrent_multi.hip).  Then
// the look is what comes too early: either the exchange goes through the XCD's L2 (NEAR, see xcd.hpp), twice as fast, or the look
// waits until PAUSE clocks after the wavefront's own stores.  us a layer, write-through, pause of 0 / 600 / 900 / 1200 / 1500 / 1800: 256 sequences of 512
// cells, backward 104 / 87 / 78 / 76 / 75 / 77, 128 70 / 52 / 54 / 56 / 58 / 61; forward 64 / 64 / 63 / 64 / 67 / 69 and 48 / 45 / 47 / 49 / 51 / 54; 64 of
// 1024 backward 94 / 73 / 76 / 78 / 80 / 82.  The other kernels, write-through, 0 / 600 / 900 / 1200, and through the L2: forward <2, 12> (128 of 384) 43 / 40 /
// 42 / 45, 37; <2, 20> (60 of 640) 48 / 45 / 47 / 49, 42; <2, 24> (64 of 768) 53 / 50 / 52 / 55, 48; <2, 28> (64 of 896) 58 / 54 / 56 / 59, 52; <4, 4> (1000 of 128) 55 / 52 / 52 / 52, 58;
// <4, 12> (300 of 384) 63 / 58 / 57 / 58, 60; backward <2, 12> 63 / 45 / 47 / 50, 42; <2, 20> 67 / 52 / 54 / 57, 49; <2, 24> 76 / 60 / 62 / 64, 57; <2, 28> 86 / 66 / 67 / 69, 70;
// <4, 8> (500 of 256) 103 / 95 / 91 / 86, 61; <4, 12> 94 / 82 / 75 / 71, 70.  Forward passes of four layers of 512 cells, 700 / 760 / 800: 256 sequences 467 / 463 / 462, 129 384 /
// 385 / 386.  What the L2 gains a layer a step can lose again (see near_fwd below).
//
// us a layer of 21 frames, forward / backward, before (a lane to a row, inputs behind the stores) and now: 512 cells, 128 sequences 49 / 55 and 45 / 52,
// 173 63 / 72 and 57 / 66, 256 71 / 79 and 63 / 76; 1024, 64 66 / 78 and 60 / 73; 320, 256 56 / 64 and 48 / 57; 128, 500 38 / 38 and 32 / 32; 64,
// 2000 53 / 62 and 46 / 50.  With several tiles a workgroup the kernels of recurrent_multi.hip run.
// What bounds a frame of 256 sequences (2.1 GHz, cycles): forward 950 products, 1100 cells (ten transcendentals each), 500 staging, 1500 to 2000 until
// the others' h is there, the rest what the memory takes (38 KB a workgroup and frame; without it 52 us a layer); backward 64 KB
// of operand, products and partial sums (63 us without what comes from memory).
#include "recurrent_tile.hpp"

namespace blstm {
namespace {

// Workgroup -> (direction, group of tiles, slice); ids are dealt round-robin to the eight XCDs, each of which gets whole groups.
struct Spot { int d, tile, u, group; };                         // (tile -1: a group that does not exist)
__device__ __forceinline__ Spot spot(int nu, int nbg) {
    const int slot = (int)blockIdx.x >> 3, group = (slot / nu) * 8 + ((int)blockIdx.x & 7);
    Spot p;
    p.u = slot % nu; p.d = group / nbg; p.group = group;
    p.tile = group < 2 * nbg ? group - p.d * nbg : -1;
    return p;
}

// ------------------------------------------------------------------------------ forward
// Width up to 32 KQ; a workgroup has one tile.  NEAR: a group on one XCD exchanges through its L2.
template <int NB, int KQ, bool SENTINEL, bool NEAR>
__global__ __launch_bounds__(64 * NW, fwd_per_cu(NB, KQ, false)) void tile_rec_fwd_kernel(RecFwdArgs a) {
    typedef typename Packs<NB>::F F;
    typedef typename Packs<NB>::W W;
    constexpr int FR = KQ / NW;                          // fragments a wavefront stages
    constexpr int PP = 4 * NB;                           // 16-byte pieces of a_x a row and gate
    constexpr int PAUSE = NEAR ? 0 : NB == 4 ? 760 : 600;   // clocks before the look (see the head of this file)
    extern __shared__ uint4 hs[];                        // [2][KQ][64], float4 [2][4][16][PP] a_x, W [2][16][16] h
    const int T = a.T, B = a.B, H = a.H;
    const int chunks = H / 8, nu = (H + 16 * NB - 1) / (16 * NB), NT = (B + 15) / 16;
    const Spot sp = spot(nu, a.nbg);
    const int d = sp.d, tile = sp.tile, row0 = tile * 16;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // this workgroup's share of the region to fill, NB / 2 words a thread and frame
    const unsigned long long share = a.fill ? (a.fill_words + gridDim.x - 1) / gridDim.x : 0ull;
    const unsigned long long first = min(a.fill_words, (unsigned long long)blockIdx.x * share);
    const unsigned fill_bytes = (unsigned)(min(a.fill_words, first + share) - first) * 16;
    const __amdgpu_buffer_rsrc_t fill = buffer(a.fill ? static_cast<uint4*>(a.fill) + first : a.fill, fill_bytes);
    unsigned fill_off = tid * 16;
    auto fill_word = [&]() { put<0>(fill, fill_off, make_uint4(~0u, ~0u, ~0u, ~0u)); fill_off += 64 * NW * 16; };
    if (tile < 0) { while (fill_off < fill_bytes) fill_word(); return; }
    float4* const axs = reinterpret_cast<float4*>(hs + 2 * KQ * 64);
    W* const ys = reinterpret_cast<W*>(axs + 2 * 4 * 16 * PP);
    unsigned* const xcds = SENTINEL && NEAR && nu > 1 && a.xcd ? a.xcd + sp.group * nu : nullptr;
    tell_xcd(xcds, sp.u);
    const int l16 = lane & 15, lq = lane >> 4;
    const int unit0 = (sp.u * NW + wave) * 4 * NB;       // this wavefront's units
    // row l16 of block b: gate l16 % 4 of unit NB (l16 / 4) + b; the wavefront's own fragments of h first
    uint4 wf[NB][KQ];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int q = 0; q < KQ; ++q) {
            const int unit = unit0 + NB * (l16 >> 2) + b, k = (q + wave * FR) % KQ * 32 + 8 * lq;
            wf[b][q] = unit < H && k < H ? *reinterpret_cast<const uint4*>(a.uh[d] + (size_t)((l16 & 3) * H + unit) * H + k) : make_uint4(0u, 0u, 0u, 0u);
        }
    park<KQ / 4>(wf);
    unsigned off[FR];                                    // bytes
#pragma unroll
    for (int i = 0; i < FR; ++i) off[i] = (unsigned)(min(4 * (wave * FR + i) + lq, chunks - 1) * CHUNK + l16 * 8) * 2;
    // this lane's cells: units j .. j + NB - 1 of row l16
    const int j = unit0 + NB * lq, jc = min(j, H - NB);
    const bool mine = j < H;
    const unsigned RT = (unsigned)(H / NB) * 16;         // lanes' records of a (frame, direction, tile)
    const unsigned rec0 = (unsigned)(jc / NB) * 16 + l16, XT = (unsigned)chunks * CHUNK;
    const unsigned x_off = mine ? (unsigned)((j >> 3) * CHUNK + l16 * 8 + (j & 7)) * 2 : DROP;
    const unsigned g_off = mine ? rec0 * 16 : DROP, c_off = mine ? rec0 * (unsigned)sizeof(F) : DROP;
    // what this lane moves of the row-major tensors: a_x, gate ax_g + k 4 / NB of row ax_row, piece ax_p; h, row y_row, word l16
    const int ax_g = lane / (16 * NB), ax_row = 4 * wave + lane % (16 * NB) / PP, ax_p = lane % PP, ax_slot = (ax_g * 16 + ax_row) * PP + (ax_p ^ (ax_row & (PP - 1)));
    const unsigned ax_off = (unsigned)(min(ax_row, B - 1 - row0) * 8 * H + ax_g * H + min(sp.u * 16 * NB + 4 * ax_p, H - 4)) * 4;
    const int y_row = 4 * wave + lq, y_unit = sp.u * 16 * NB + NB * l16;
    const unsigned y_off = y_unit < H ? (unsigned)(y_row * 2 * H + y_unit) * 2 : DROP, y_bytes = (unsigned)((min(B - row0, 16) - 1) * 2 * H + H) * 2;
    auto frame = [&](int n) { return d ? T - 1 - n : n; };
    float4 axr[NB];
    auto inputs = [&](int n) __attribute__((always_inline)) {
        const float* base = a.ax + ((size_t)frame(min(n, T - 1)) * B + row0) * 8 * H + d * 4 * H;
#pragma unroll
        for (int k = 0; k < NB; ++k) axr[k] = get<float4>(base + (size_t)(k * (4 / NB)) * H, ax_off);
    };
    auto store_y = [&](int n) __attribute__((always_inline)) {
        put<later(SENTINEL)>(buffer(a.y + ((size_t)frame(max(n, 0)) * B + row0) * 2 * H + d * H, n < 0 ? 0u : y_bytes), y_off, ys[(n & 1) * 256 + turned(y_row, l16)]);
    };
    inputs(0);
    float c[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) c[b] = 0.0f;
    float poison = ld_coh_u32(a.abort_word) != 0 ? __builtin_nanf("") : 0.0f;
    bool lost;
    const bool near = one_xcd(xcds, nu, a.abort_word, a.limit_ticks, &lost);
    if (lost) poison = __builtin_nanf("");
    unsigned long long stored = 0;                       // when the last h went out
    auto do_frame = [&](auto first_frame, const int n) __attribute__((always_inline)) {
        constexpr bool FIRST = decltype(first_frame)::value;
        const int t = frame(n);
        uint4* const hb = hs + (n & 1) * KQ * 64;
        float4* const ab = axs + (n & 1) * 4 * 16 * PP;
        f32x4_t acc[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[b][e] = 0.0f;
        uint4 f[FR];
        if constexpr (!FIRST) {
            bf16_t* const base = a.hx + ((size_t)(frame(n - 1) * 2 + d) * NT + tile) * XT;
            if constexpr (!SENTINEL) if (wait_counter(a.cnt + d * NT + tile, (unsigned)(nu * n), a.abort_word, a.limit_ticks)) poison = __builtin_nanf("");
            const __amdgpu_buffer_rsrc_t x = buffer(base, XT * 2);
            if constexpr (PAUSE > 0) while (__builtin_amdgcn_s_memtime() - stored < PAUSE) {}
            look_through<FR>(f, x, off);
#pragma unroll
            for (int k = 0; k < NB; ++k) ab[ax_slot + k * (4 / NB) * 16 * PP] = axr[k];
            if constexpr (SENTINEL) if (await<FR>(f, x, off, false, a.abort_word, a.limit_ticks)) poison = __builtin_nanf("");
#pragma unroll
            for (int i = 0; i < FR; ++i) hb[(wave * FR + i) * 64 + lane] = f[i];
#pragma unroll
            for (int q = 0; q < FR; ++q)
#pragma unroll
                for (int b = 0; b < NB; ++b) acc[b] = mfma16(wf[b][q], f[q], acc[b]);
            __builtin_amdgcn_sched_barrier(0);
        } else {
#pragma unroll
            for (int k = 0; k < NB; ++k) ab[ax_slot + k * (4 / NB) * 16 * PP] = axr[k];
        }
        lds_barrier();                                   // one a frame: the buffers are doubled
        inputs(n + 1);
        if constexpr (SENTINEL) store_y(n - 1);
        if constexpr (!FIRST) {
            // the others in groups of FR, a group read while the one before is multiplied
            uint4 h[2][FR];
            auto read = [&](int g, uint4 (&v)[FR]) __attribute__((always_inline)) {
                const int slot = (wave + g) % NW * FR;   // (uniform)
#pragma unroll
                for (int i = 0; i < FR; ++i) v[i] = hb[(slot + i) * 64 + lane];
            };
            read(1, h[1]);
#pragma unroll
            for (int g = 1; g < NW; ++g) {
                if (g + 1 < NW) read(g + 1, h[(g + 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < FR; ++i)
#pragma unroll
                    for (int b = 0; b < NB; ++b) acc[b] = mfma16(wf[b][g * FR + i], h[g & 1][i], acc[b]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        F ax[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            if constexpr (NB == 4) ax[g] = ab[(g * 16 + l16) * PP + ((4 * wave + lq) ^ l16)];
            else ax[g] = reinterpret_cast<const F*>(ab + (g * 16 + l16) * PP + ((2 * wave + (lq >> 1)) ^ (l16 & 7)))[lq & 1];
        }
        float gi[NB], gf[NB], gg[NB], go[NB];
        unsigned hw[NB / 2];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            gi[b] = fast_sigmoid(part(ax[0], b) + acc[b][0]);
            gf[b] = fast_sigmoid(part(ax[1], b) + acc[b][1]);
            gg[b] = fast_tanh(part(ax[2], b) + acc[b][2]);
            go[b] = fast_sigmoid(part(ax[3], b) + acc[b][3]);
            c[b] = next_cell(gf[b], c[b], gi[b], gg[b]);
            const unsigned h = coh_bf16(go[b] * fast_tanh(c[b]) + poison);
            hw[b >> 1] = b & 1 ? hw[b >> 1] | (h << 16) : h;
        }
        put_exchange(near, buffer(a.hx + ((size_t)(t * 2 + d) * NT + tile) * XT, XT * 2), x_off, pack(hw));
        if constexpr (PAUSE > 0) stored = __builtin_amdgcn_s_memtime();
        if constexpr (!SENTINEL) { signal_counter(a.cnt + d * NT + tile); store_y(n - 1); }
        // what follows is not on the frame-to-frame path
        const size_t rec = ((size_t)(t * 2 + d) * NT + tile) * RT;
        const __amdgpu_buffer_rsrc_t g4 = buffer(reinterpret_cast<uint4*>(a.gates) + rec * (NB / 2), RT * (NB / 2) * 16);
#pragma unroll
        for (int k = 0; k < NB / 2; ++k)
            put<later(SENTINEL)>(g4, g_off + k * RT * 16, make_uint4(pack_bf2(gi[2 * k], gf[2 * k]), pack_bf2(gg[2 * k], go[2 * k]), pack_bf2(gi[2 * k + 1], gf[2 * k + 1]), pack_bf2(gg[2 * k + 1], go[2 * k + 1])));
        put<later(SENTINEL)>(buffer(reinterpret_cast<F*>(a.c) + rec, RT * (unsigned)sizeof(F)), c_off, pack(c));
        ys[(n & 1) * 256 + turned(l16, 4 * wave + lq)] = pack(hw);
#pragma unroll
        for (int k = 0; k < NB / 2; ++k) fill_word();
    };
    do_frame(std::true_type{}, 0);
    for (int n = 1; n < T; ++n) do_frame(std::false_type{}, n);
    lds_barrier();
    store_y(T - 1);
    while (fill_off < fill_bytes) fill_word();           // (whatever rounding left over)
}

// ------------------------------------------------------------------------------ backward
// Each wavefront contracts KQ / 4 blocks of 32 columns of every gate, SL fragments of dE/da in flight ahead of the products.
template <int NB, int KQ, bool SENTINEL, bool NEAR>
__global__ __launch_bounds__(64 * NW, bwd_per_cu(NB, KQ, false)) void tile_rec_bwd_kernel(RecBwdArgs a) {
    typedef typename Packs<NB>::F F;
    typedef typename Packs<NB>::W W;
    constexpr int BW = KQ / 4;
    constexpr int SL = 4, NSL = KQ / SL;
    constexpr int AP = 2 * NB;                           // 16-byte pieces of dE/da a row and gate
    constexpr int PAUSE = NEAR ? 0 : NB == 4 ? 1200 : 600;
    extern __shared__ float4 ps[];                       // [2][NW][NB][64], uint4 [2][4][16][AP] dE/da, W [2][16][16] dy
    const int T = a.T, B = a.B, H = a.H;
    const int chunks = H / 8, nu = (H + 16 * NB - 1) / (16 * NB), NT = (B + 15) / 16;
    const Spot sp = spot(nu, a.nbg);
    const int d = sp.d, tile = sp.tile, row0 = tile * 16;
    if (tile < 0) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint4* const das = reinterpret_cast<uint4*>(ps + 2 * NW * NB * 64);
    W* const dys = reinterpret_cast<W*>(das + 2 * 4 * 16 * AP);
    unsigned* const xcds = SENTINEL && NEAR && nu > 1 && a.xcd ? a.xcd + sp.group * nu : nullptr;
    tell_xcd(xcds, sp.u);
    const int l16 = lane & 15, lq = lane >> 4;
    const int q0 = wave * BW;
    uint4 wf[NB][KQ];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int q = 0; q < KQ; ++q) {
            const int unit = sp.u * 16 * NB + b * 16 + l16, k = (q0 + q % BW) * 32 + 8 * lq;
            wf[b][q] = unit < H && k < H ? *reinterpret_cast<const uint4*>(a.uht[d] + (size_t)unit * 4 * H + (q / BW) * H + k) : make_uint4(0u, 0u, 0u, 0u);
        }
    // fragment q: gate q / BW, block q0 + q % BW of 32 columns
    unsigned offb[BW];                                   // bytes, within a gate
#pragma unroll
    for (int q = 0; q < BW; ++q) offb[q] = (unsigned)(min(4 * (q0 + q) + lq, chunks - 1) * CHUNK + l16 * 8) * 2;
    const int unit0 = (sp.u * NW + wave) * 4 * NB;       // this wavefront's units; the lane's: j .. j + NB - 1 of row l16
    const int j = unit0 + NB * lq, jc = min(j, H - NB);
    const unsigned RT = (unsigned)(H / NB) * 16, rec0 = (unsigned)(jc / NB) * 16 + l16;
    const unsigned XT = (unsigned)4 * chunks * CHUNK;    // exchange elements of a (frame, direction, tile)
    // eight units of one gate a lane (see below): where they go
    const int gate0 = NB == 2 ? lq : 2 * (lq & 1), u8 = NB == 2 ? unit0 : unit0 + 8 * (lq >> 1);
    const unsigned x_off = u8 < H ? (unsigned)((gate0 * chunks + (u8 >> 3)) * CHUNK + l16 * 8) * 2 : DROP;
    // what this lane moves of the row-major tensors: dy, row y_row, word l16; dE/da, gate `wave` of rows a_row + 8 k, piece a_p
    const int y_row = 4 * wave + lq, a_row = lane / AP, a_p = lane % AP, a_unit = sp.u * 16 * NB + 8 * a_p;
    const unsigned y_off = (unsigned)(min(y_row, B - 1 - row0) * 2 * H + min(sp.u * 16 * NB + NB * l16, H - NB)) * 2;
    const unsigned a_off = a_unit < H ? (unsigned)(a_row * 8 * H + wave * H + a_unit) * 2 : DROP, a_bytes = (unsigned)((min(B - row0, 16) - 1) * 8 * H + 4 * H) * 2;
    auto da_slot = [&](int gate, int row, int p) { return (gate * 16 + row) * AP + (p ^ (NB == 4 ? row >> 1 : row >> 2)); };
    auto frame = [&](int ni) { return d ? ni : T - 1 - ni; };   // (the last one visited forward comes first)
    auto record = [&](int t) { return ((size_t)(t * 2 + d) * NT + tile) * RT; };
    struct In { W dy; uint4 g[NB / 2]; F cp; };
    auto inputs = [&](int n, In& in) __attribute__((always_inline)) {
        const int ni = min(n, T - 1), t = frame(ni);
        in.dy = get<W>(a.dy + ((size_t)t * B + row0) * 2 * H + d * H, y_off);
#pragma unroll
        for (int k = 0; k < NB / 2; ++k) in.g[k] = get<uint4>(reinterpret_cast<const uint4*>(a.gates) + record(t) * (NB / 2) + (size_t)k * RT, rec0 * 16);
        in.cp = get<F>(reinterpret_cast<const F*>(a.c) + record(frame(min(ni + 1, T - 1))), rec0 * (unsigned)sizeof(F));
    };
    auto store_da = [&](int ni) __attribute__((always_inline)) {
        const __amdgpu_buffer_rsrc_t p = buffer(a.da + ((size_t)frame(max(ni, 0)) * B + row0) * 8 * H + d * 4 * H, ni < 0 ? 0u : a_bytes);
#pragma unroll
        for (int k = 0; k < NB / 2; ++k) put<later(SENTINEL)>(p, a_off + (unsigned)(k * 8 * 8 * H * 2), das[(ni & 1) * 4 * 16 * AP + da_slot(wave, a_row + 8 * k, a_p)]);
    };
    In in0, in1;
    inputs(0, in0);
    F c = get<F>(reinterpret_cast<const F*>(a.c) + record(frame(0)), rec0 * (unsigned)sizeof(F));   // this frame's cell state
    float dcn[NB];                                       // carried dE/dc
#pragma unroll
    for (int b = 0; b < NB; ++b) dcn[b] = 0.0f;
    float poison = ld_coh_u32(a.abort_word) != 0 ? __builtin_nanf("") : 0.0f;
    bool lost = false;
    // (a group of one workgroup is on one XCD: 2049 sequences of 24 cells 36 -> 31 us a layer, 4130 of 32 62 -> 58; but 3000 of 64 70 -> 72, and forward 4130 of 32 49 -> 58)
    const bool near = (SENTINEL && NEAR && NB == 2 && nu == 1 && a.xcd) || one_xcd(xcds, nu, a.abort_word, a.limit_ticks, &lost);
    if (lost) poison = __builtin_nanf("");
    unsigned long long stored = 0;                       // when the last dE/da went out
    auto do_frame = [&](auto first_frame, const int ni, const In& cur, In& nxt) __attribute__((always_inline)) {
        constexpr bool FIRST = decltype(first_frame)::value;
        const int t = frame(ni);
        float4* const pt = ps + (ni & 1) * NW * NB * 64;
        float dh[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) dh[b] = 0.0f;
        if constexpr (!FIRST) {
            bf16_t* const base = a.dax + ((size_t)(frame(ni - 1) * 2 + d) * NT + tile) * XT;
            uint4 f[2][SL];
            bool gu = false;
            if constexpr (!SENTINEL) gu = wait_counter(a.cnt + d * NT + tile, (unsigned)(nu * ni), a.abort_word, a.limit_ticks);
            const __amdgpu_buffer_rsrc_t x = buffer(base, XT * 2);
            auto off = [&](int s, unsigned (&o)[SL]) __attribute__((always_inline)) {
#pragma unroll
                for (int q = 0; q < SL; ++q) o[q] = (unsigned)((s * SL + q) / BW) * (unsigned)(chunks * CHUNK * 2) + offb[(s * SL + q) % BW];
            };
            unsigned o[2][SL];
            off(0, o[0]);
            if constexpr (PAUSE > 0) while (__builtin_amdgcn_s_memtime() - stored < PAUSE) {}
            look_through<SL>(f[0], x, o[0]);
            dys[(ni & 1) * 256 + turned(y_row, l16)] = cur.dy;
            f32x4_t acc[NB];
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[b][e] = 0.0f;
#pragma unroll
            for (int s = 0; s < NSL; ++s) {
                if (s + 1 < NSL) { off(s + 1, o[(s + 1) & 1]); look_through<SL>(f[(s + 1) & 1], x, o[(s + 1) & 1]); }
                if constexpr (SENTINEL) gu = await<SL>(f[s & 1], x, o[s & 1], gu, a.abort_word, a.limit_ticks);
#pragma unroll
                for (int q = 0; q < SL; ++q)
#pragma unroll
                    for (int b = 0; b < NB; ++b) acc[b] = mfma16(wf[b][s * SL + q], f[s & 1][q], acc[b]);
            }
            if (gu) poison = __builtin_nanf("");
#pragma unroll
            for (int b = 0; b < NB; ++b) pt[(wave * NB + b) * 64 + lane] = make_float4(acc[b][0], acc[b][1], acc[b][2], acc[b][3]);
        } else {
            dys[(ni & 1) * 256 + turned(y_row, l16)] = cur.dy;
        }
        lds_barrier();                                   // one a frame: the buffers are doubled
        inputs(ni + 1, nxt);
        if constexpr (SENTINEL) store_da(ni - 1);
        if constexpr (!FIRST) {
            // block b of the partial sums has units 16 b + 4 lq + e of row l16
            F v[NW];
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                if constexpr (NB == 4) v[w] = pt[(w * NB + wave) * 64 + lane];
                else v[w] = reinterpret_cast<const F*>(pt + (w * NB + (wave >> 1)) * 64)[(((wave & 1) * 2 + (lq >> 1)) * 16 + l16) * 2 + (lq & 1)];
            }
#pragma unroll
            for (int w = 0; w < NW; ++w)
#pragma unroll
                for (int b = 0; b < NB; ++b) dh[b] += part(v[w], b);
        }
        const W dy = dys[(ni & 1) * 256 + turned(l16, 4 * wave + lq)];
        const bool last = ni == T - 1;                   // (the frame visited first forward has no cell state before it)
        unsigned da[4][NB / 2];                          // a gate's units
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const uint4 g = cur.g[b >> 1];
            const unsigned gif = b & 1 ? g.z : g.x, ggo = b & 1 ? g.w : g.y, dyw = word(dy, b >> 1);
            const float gi = bf2f((bf16_t)(gif & 0xFFFFu)), gf = bf2f((bf16_t)(gif >> 16));
            const float gg = bf2f((bf16_t)(ggo & 0xFFFFu)), go = bf2f((bf16_t)(ggo >> 16));
            const float dht = dh[b] + bf2f((bf16_t)(b & 1 ? dyw >> 16 : dyw & 0xFFFFu)) + poison;
            const float tc = fast_tanh(part(c, b)), cp = last ? 0.0f : part(cur.cp, b);
            const float dc = dht * go * (1.0f - tc * tc) + dcn[b];
            const unsigned v[4] = {coh_bf16(dc * gg * gi * (1.0f - gi)), coh_bf16(dc * cp * gf * (1.0f - gf)),
                                   coh_bf16(dc * gi * (1.0f - gg * gg)), coh_bf16(dht * tc * go * (1.0f - go))};
#pragma unroll
            for (int k = 0; k < 4; ++k) da[k][b >> 1] = b & 1 ? da[k][b >> 1] | (v[k] << 16) : v[k];
            dcn[b] = dc * gf;
        }
        c = cur.cp;
        // Eight units of one gate a lane.  NB = 2: word g of lane group lq becomes word lq of lane group g (gate lq, the
        // wavefront's units).  NB = 4: neighbouring groups trade halves (gates 2 (lq % 2) and the next, units 8 (lq / 2) ..).
        uint4 o[NB / 2];
        if constexpr (NB == 2) {
            const auto s02 = __builtin_amdgcn_permlane32_swap(da[0][0], da[2][0], false, false), s13 = __builtin_amdgcn_permlane32_swap(da[1][0], da[3][0], false, false);
            const auto t01 = __builtin_amdgcn_permlane16_swap(s02[0], s13[0], false, false), t23 = __builtin_amdgcn_permlane16_swap(s02[1], s13[1], false, false);
            o[0] = make_uint4(t01[0], t01[1], t23[0], t23[1]);
        } else {
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const auto lo = __builtin_amdgcn_permlane16_swap(da[k][0], da[k + 2][0], false, false), hi = __builtin_amdgcn_permlane16_swap(da[k][1], da[k + 2][1], false, false);
                o[k] = make_uint4(lo[0], hi[0], lo[1], hi[1]);
            }
        }
        const __amdgpu_buffer_rsrc_t x = buffer(a.dax + ((size_t)(t * 2 + d) * NT + tile) * XT, XT * 2);
#pragma unroll
        for (int k = 0; k < NB / 2; ++k) put_exchange(near, x, x_off + (unsigned)(k * chunks * CHUNK * 2), o[k]);
        if constexpr (PAUSE > 0) stored = __builtin_amdgcn_s_memtime();
        if constexpr (!SENTINEL) { signal_counter(a.cnt + d * NT + tile); store_da(ni - 1); }
#pragma unroll
        for (int k = 0; k < NB / 2; ++k) das[(ni & 1) * 4 * 16 * AP + da_slot(gate0 + k, l16, (u8 >> 3) - sp.u * AP)] = o[k];
    };
    do_frame(std::true_type{}, 0, in0, in1);
    for (int ni = 1; ni < T; ni += 2) {
        do_frame(std::false_type{}, ni, in1, in0);
        if (ni + 1 < T) do_frame(std::false_type{}, ni + 1, in0, in1);
    }
    lds_barrier();
    store_da(T - 1);
}

// The groups of tiles a direction is cut into: as many as leave every XCD, which gets whole groups, per_cu workgroups a CU.
Cut cut(int B, int H, int units, int per_cu) {
    const int nu = (H + units - 1) / units, tiles = (B + 15) / 16, most = 4 * (32 * per_cu / nu);
    Cut c;
    c.per_group = (tiles + most - 1) / most;
    c.nbg = (tiles + c.per_group - 1) / c.per_group;
    c.grid = (2 * c.nbg + 7) / 8 * 8 * nu;
    c.real = 2 * c.nbg * nu;
    return c;
}
// More than one workgroup a CU only where that leaves each a tile of its own (and for layers of up to 32 units, whose workgroups
// have the least to do).  One layer of 21 frames, us, one a CU / as below, forward and backward: 64 units, 3000 sequences
// 158 + 181 / 124 + 160; 128, 1500 159 + 180 / 141 + 159; 256, 700 forward 160 / 144; 32, 8192 257 + 334 / 186 + 242.  Where two of
// three tiles were left, 128, 3000, it was 253 + 261 / 280 + 271.
Cut best_cut(int B, int H, int units, int most_per_cu) {
    for (int p = 1; p <= most_per_cu; ++p) {
        const Cut c = cut(B, H, units, p);
        if (c.per_group == 1) return c;
    }
    return cut(B, H, units, H <= 32 ? 2 : 1);
}

// Where the exchange goes through the XCD's L2 (else the look waits, see the head of this file): by the kernel, and wherever a CU has more than
// one workgroup, whose looks would come too early at any pause.  Whole steps of four layers, 21 frames, 8000 classes, us, pause / so: 500 sequences of 256 cells
// (backward <4, 8>) 1299 / 1190, 640 of 136 1215 / 1077; more than one workgroup a CU: 700 of 136 1385 / 1169, 512 of 200 1285 / 1082, 400 of 264 1584 / 1230,
// 1500 of 128 (forward <4, 4>) 2064 / 1996.  But 128 of 512 885 / 923, 1000 of 128 1393 / 1422 and 600 of 128 (forward) 976 / 998: the lines left dirty are written in the way of
// the products that follow.
constexpr bool near_fwd(int nb, int kq) { return kq == 8 || nb * kq == 8; }
constexpr bool near_bwd(int nb, int kq) { return kq == 4 || (nb == 4 && kq == 8); }
constexpr int ONE_A_CU = 256;

template <int NB, int KQ, bool S, bool NEAR>
hipError_t launch_one(const RecFwdArgs& a, const Cut& c, hipStream_t st, bool* launched) {
    return launch_resident<tile_rec_fwd_kernel<NB, KQ, S, NEAR>>(a, 64 * NW, (size_t)2 * (KQ * 64 * 16 + 4 * 16 * 4 * NB * 16 + 256 * NB * 2), c.grid, c.real, st, launched);
}
template <int NB, int KQ, bool S, bool NEAR>
hipError_t launch_one(const RecBwdArgs& a, const Cut& c, hipStream_t st, bool* launched) {
    return launch_resident<tile_rec_bwd_kernel<NB, KQ, S, NEAR>>(a, 64 * NW, (size_t)2 * (NW * NB * 64 * 16 + 4 * 16 * 2 * NB * 16 + 256 * NB * 2), c.grid, c.real, st, launched);
}
template <int NB, int KQ, bool S, typename A>
hipError_t run(const A& a, const Cut& c, hipStream_t st, bool* launched) {
    constexpr bool fwd = std::is_same_v<A, RecFwdArgs>, near = fwd ? near_fwd(NB, KQ) : near_bwd(NB, KQ);
    if constexpr (S && !near && (fwd ? fwd_per_cu(NB, KQ, false) : bwd_per_cu(NB, KQ, false)) > 1)
        if (c.real > ONE_A_CU) return launch_one<NB, KQ, S, true>(a, c, st, launched);
    return launch_one<NB, KQ, S, near>(a, c, st, launched);
}
template <int NB, int KQ, typename A>
hipError_t run_width(A a, bool sentinel, hipStream_t st, bool* launched) {
    const Cut c = best_cut(a.B, a.H, 16 * NB, std::is_same_v<A, RecFwdArgs> ? fwd_per_cu(NB, KQ, false) : bwd_per_cu(NB, KQ, false));
    a.nbg = c.nbg; a.tiles_per_group = c.per_group;
    if (c.per_group > 1) return launch_rec_multi(a, NB, KQ, sentinel, c.grid, c.real, st, launched);
    if (sentinel) return run<NB, KQ, true>(a, c, st, launched);
    if constexpr (KQ == 4 || KQ == 8 || KQ == 16 || KQ == 32) return run<NB, KQ, false>(a, c, st, launched);
    return hipSuccess;
}
template <typename A>
hipError_t launch(const A& a, bool sentinel, hipStream_t st, bool* launched) {
    *launched = false;
    const int units = rec_tile_units(a.B, a.H);
    if (units == 0 || !(sentinel || rec_fenced(a.H))) return hipSuccess;
#define BLSTM_TILE(NB, KQ) if (units == 16 * NB && a.H <= 32 * KQ) return run_width<NB, KQ>(a, sentinel, st, launched)
    BLSTM_TILE(2, 4); BLSTM_TILE(2, 8); BLSTM_TILE(2, 12); BLSTM_TILE(2, 16); BLSTM_TILE(2, 20); BLSTM_TILE(2, 24); BLSTM_TILE(2, 28); BLSTM_TILE(2, 32);
    BLSTM_TILE(4, 4); BLSTM_TILE(4, 8); BLSTM_TILE(4, 12); BLSTM_TILE(4, 16);
#undef BLSTM_TILE
    return hipSuccess;
}

}  // namespace

// Widths whose last slice of 64 units would be at most half full, and so many sequences that a workgroup would walk three or more
// tiles (four above 256 units): the slices of recurrent.hip have no empty part, and its forward kernel two workgroups a CU.  One layer of
// 21 frames, us, 16-row tiles / recurrent.hip, forward and backward: 96 units, 4096 sequences 360 + 358 / 282 + 315; 160, 2048 314 + 335 / 265 + 293;
// 200, 2048 397 + 394 / 328 + 406; 288, 2048 479 + 575 / 431 + 606.
bool rec_narrow(int B, int H) {
    return H > 64 && H <= 288 && H % 8 == 0 && H % 64 >= 1 && H % 64 <= 32 && cut(B, H, 64, 1).per_group > (H <= 256 ? 2 : 3);
}
// Slices of 32 units for a layer of one such slice, and while that leaves every workgroup a CU and a tile of its own; else of 64: half
// of the operand's bytes per cell, but their weights fit the registers up to 512 cells only.  (Of 32 with two workgroups a CU where the last slice
// of 64 would be at most half full and take two tiles a workgroup: 136 cells, 700 sequences 84 + 130 us against 127 + 159.)
// Learners that share a device: 65 to 128 sequences of 512 cells are 256 workgroups of 32 units, which no other learner's can run
// beside (residency.hip); of 64 units they would be 128.  Four layers, 72 sequences, 200 classes, us a step, one learner / two at
// once: 32 units 699 / 1384, 64 units 789 / 987.  Slices of 32 units, as one learner to a device is what this is for; not chosen by what else
// is running, because the slices' width shows in the last bits.
// Beyond 512 cells several tiles of 32 units a workgroup lose to recurrent.hip's 32 x 32 (1024 cells, 512 sequences 450 / 545 us a layer
// against 348 / 387; 128 sequences 121 / 145 against 96 / 115).
int rec_tile_units(int B, int H) {
    if (!rec_supported(H) || rec_narrow(B, H)) return 0;
    if (H <= 32 || cut(B, H, 32, 1).per_group == 1) return 32;
    const int last = H % 64;
    if (last >= 1 && last <= 32 && H <= 384 && cut(B, H, 64, 1).per_group > 1 && cut(B, H, 32, 2).per_group == 1) return 32;
    return H <= 512 ? 64 : 0;
}
hipError_t launch_rec_tile_fwd(const RecFwdArgs& a, bool sentinel, hipStream_t st, bool* launched) { return launch(a, sentinel, st, launched); }
hipError_t launch_rec_tile_bwd(const RecBwdArgs& a, bool sentinel, hipStream_t st, bool* launched) { return launch(a, sentinel, st, launched); }

}  // namespace blstm
