// Persistent recurrent kernels (bf16) on 16-row batch tiles, several of them a workgroup, walked one after the other in every frame.
//
// Layouts, products and protocols are those of recurrent_tile.hip.  What differs is what an item (a tile of a frame) may wait for: its
// operand was written a frame ago, so nothing here needs to be a chain of latencies.
//   - The inputs that come from memory (a_x; dy, gates, cell states) are asked for two items ahead, the operand one item ahead.
//   - An item is straight-line code.  Every lane issues every load and store (range-checked buffer stores drop what does not
//     exist; loads beyond the end repeat what does), so the compiler knows how many are in flight behind the one it waits for.  With a
//     branch round a store it does not, and waited for all of them in every item: the latency of a_x and the stores' acknowledgements.
//   - Row-major tensors are read and written in whole lines and turned in LDS (see `turned`).
//   - The carried state (c; dE/dc and the next item's c) stays in LDS (LOCAL) as long as the group's tiles fit there.
//   - The forward kernel's h goes through the XCD's L2 (xcd.hpp): 10 % of a layer.  The backward kernel's dE/da, four times as much, does not: 4 to
//     15 % slower (512 cells, 512 sequences 116 us a layer write-through, 135 through the L2).
// us a layer of 21 frames, forward / backward, before (inputs one item ahead, a lane to a row, waits for everything) and now, 512
// cells: 272 sequences 121 / 133 and 98 / 105, 512 153 / 154 and 122 / 116, 700 201 / 212 and 170 / 161, 2048 488 / 559 and 414 /
// 386; 320 cells, 3000 485 / 539 and 383 / 330; 256, 2048 235 / 253 and 199 / 170.  Bound by the memory: forward 1.85 GB a layer of 512
// cells and 2048 sequences (4.5 TB/s); without the marking of dE/da's copy an eighth less, without loading a_x a third; backward without its
// row-major stores 343, without its operand 346.  (The backward operand asked for under the products that free its registers,
// half an item earlier: 387 against 400 with eight tiles a workgroup, but 189 against 161 with three, whose looks then come too early.)
#include "recurrent_tile.hpp"

namespace blstm {
namespace {

// Workgroup -> (direction, group of tiles, slice), as in recurrent_tile.hip; the tiles are dealt evenly.  A group left with one tile
// takes a neighbour's as well (`pair`; both write the same bits): its look at the next operand, an item ahead, would always come too
// early (512 cells, 272 sequences backward 146 us a layer, 108 with the second tile).
struct Spot { int d, first, ntl, u, group; };
__device__ __forceinline__ Spot spot(int nu, int nbg, int ntiles, bool pair) {
    const int slot = (int)blockIdx.x >> 3, group = (slot / nu) * 8 + ((int)blockIdx.x & 7);
    Spot p;
    p.u = __builtin_amdgcn_readfirstlane(slot % nu); p.d = __builtin_amdgcn_readfirstlane(group / nbg); p.group = group;
    const int g = group - p.d * nbg;
    // (at most 256 groups a direction -- a slice of 32 units, two workgroups a CU --, so the products stay below 2^32 with 2^24 tiles)
    p.first = __builtin_amdgcn_readfirstlane((int)((unsigned)g * (unsigned)ntiles / (unsigned)nbg));
    p.ntl = group < 2 * nbg ? __builtin_amdgcn_readfirstlane((int)((unsigned)(g + 1) * (unsigned)ntiles / (unsigned)nbg)) - p.first : 0;
    if (pair && p.ntl == 1 && ntiles > 1) { p.first = max(p.first - 1, 0); p.ntl = 2; }
    return p;
}
// An item: the n-th visited frame of the group's i-th tile.
struct Item {
    int n, i;
    __device__ __forceinline__ void next(int ntl) { if (++i == ntl) { i = 0; ++n; } }
};
__device__ __forceinline__ void keep(const Item& p) { asm volatile("" :: "s"(p.n), "s"(p.i)); }

// ------------------------------------------------------------------------------ forward
template <int NB, int KQ, bool SENTINEL, bool LOCAL>
__global__ __launch_bounds__(64 * NW, fwd_per_cu(NB, KQ, true)) void multi_tile_rec_fwd_kernel(RecFwdArgs a) {
    typedef typename Packs<NB>::F F;
    typedef typename Packs<NB>::W W;
    constexpr int FR = KQ / NW;                          // fragments a wavefront stages
    constexpr int PP = 4 * NB;                           // 16-byte pieces of a_x a row and gate
    extern __shared__ uint4 hs[];                        // [2][KQ][64], float4 [2][4][16][PP] a_x, W [2][16][16] h, then (LOCAL) F [tiles][64 NW]
    const int T = a.T, B = a.B, H = a.H;
    const int chunks = H / 8, nu = (H + 16 * NB - 1) / (16 * NB), NT = (B + 15) / 16;
    const Spot sp = spot(nu, a.nbg, NT, SENTINEL);
    const int d = sp.d, ntl = sp.ntl;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // this workgroup's share of the region to fill, NB / 2 words a thread and item
    const unsigned long long share = a.fill ? (a.fill_words + gridDim.x - 1) / gridDim.x : 0ull;
    const unsigned long long first = min(a.fill_words, (unsigned long long)blockIdx.x * share);
    const unsigned fill_bytes = (unsigned)(min(a.fill_words, first + share) - first) * 16;
    const __amdgpu_buffer_rsrc_t fill = buffer(a.fill ? static_cast<uint4*>(a.fill) + first : a.fill, fill_bytes);
    unsigned fill_off = tid * 16;
    auto fill_word = [&]() { put<0>(fill, fill_off, make_uint4(~0u, ~0u, ~0u, ~0u)); fill_off += 64 * NW * 16; };
    if (ntl <= 0) { while (fill_off < fill_bytes) fill_word(); return; }
    float4* const axs = reinterpret_cast<float4*>(hs + 2 * KQ * 64);
    W* const ys = reinterpret_cast<W*>(axs + 2 * 4 * 16 * PP);
    F* const state = reinterpret_cast<F*>(ys + 2 * 256) + tid;
    unsigned* const xcds = SENTINEL && nu > 1 && a.xcd ? a.xcd + sp.group * nu : nullptr;
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
    const unsigned rec0 = (unsigned)(jc / NB) * 16 + l16;
    const unsigned x_off = mine ? (unsigned)((j >> 3) * CHUNK + l16 * 8 + (j & 7)) * 2 : DROP;
    const unsigned g_off = mine ? rec0 * 16 : DROP, c_off = mine ? rec0 * (unsigned)sizeof(F) : DROP;
    auto frame = [&](int n) { return d ? T - 1 - n : n; };
    auto record = [&](int t, int i) { return ((size_t)(t * 2 + d) * NT + sp.first + i) * RT; };
    // what this lane moves of the row-major tensors: a_x, gate ax_g + k 4 / NB of row ax_row, piece ax_p; h, row y_row, word y_p
    const int ax_g = lane / (16 * NB), ax_row = 4 * wave + lane % (16 * NB) / PP, ax_p = lane % PP, ax_slot = (ax_g * 16 + ax_row) * PP + (ax_p ^ (ax_row & (PP - 1)));
    const unsigned ax_off = (unsigned)(ax_g * H + min(sp.u * 16 * NB + 4 * ax_p, H - 4)) * 4;
    const int y_row = 4 * wave + lq, y_unit = sp.u * 16 * NB + NB * l16;
    const unsigned y_off = y_unit < H ? (unsigned)(y_row * 2 * H + y_unit) * 2 : DROP;
    struct In { float4 ax[NB]; F cp; };
    auto inputs = [&](const Item& p, In& in) __attribute__((always_inline)) {
        const int n = min(p.n, T - 1), t = frame(n), row0 = (sp.first + p.i) * 16;
        const float* base = a.ax + ((size_t)t * B + row0) * 8 * H + d * 4 * H;
        const unsigned o = (unsigned)(min(ax_row, B - 1 - row0) * 8 * H) * 4 + ax_off;
#pragma unroll
        for (int k = 0; k < NB; ++k) in.ax[k] = get<float4>(base + (size_t)(k * (4 / NB)) * H, o);
        if constexpr (!LOCAL) in.cp = get<F>(reinterpret_cast<const F*>(a.c) + record(frame(max(n - 1, 0)), p.i), rec0 * (unsigned)sizeof(F));
    };
    auto operand = [&](const Item& p) { return a.hx + ((size_t)(frame(p.n - 1) * 2 + d) * NT + sp.first + p.i) * chunks * CHUNK; };   // (behind the first frame)
    uint4 ahead[FR];
    auto look = [&](const Item& p) __attribute__((always_inline)) { look_through<FR>(ahead, buffer(operand(p), chunks * CHUNK * 2), off); };
    float poison = ld_coh_u32(a.abort_word) != 0 ? __builtin_nanf("") : 0.0f;
    bool lost;
    const bool near = one_xcd(xcds, nu, a.abort_word, a.limit_ticks, &lost);
    if (lost) poison = __builtin_nanf("");
    Item now{0, 0}, next{0, 0}, third{0, 0};             // this item and the two behind it
    next.next(ntl); third = next; third.next(ntl);
    int par = 0;                                         // of the item: which of the two buffers
    Item before{-1, 0};                                  // the item whose h waits in LDS for the other wavefronts
    auto store_y = [&]() __attribute__((always_inline)) {
        const int t = frame(max(before.n, 0)), row0 = (sp.first + before.i) * 16;
        const unsigned bytes = before.n < 0 ? 0u : (unsigned)((min(B - row0, 16) - 1) * 2 * H + H) * 2;
        put<later(SENTINEL)>(buffer(a.y + ((size_t)t * B + row0) * 2 * H + d * H, bytes), y_off, ys[(par ^ 1) * 256 + turned(y_row, l16)]);
    };
    auto do_item = [&](auto first_frame, const In& cur, In& nxt) __attribute__((always_inline)) {
        constexpr bool FIRST = decltype(first_frame)::value;
        const int t = frame(now.n);
        uint4* const hb = hs + par * KQ * 64;
        float4* const ab = axs + par * 4 * 16 * PP;
#pragma unroll
        for (int k = 0; k < NB; ++k) ab[ax_slot + k * (4 / NB) * 16 * PP] = cur.ax[k];
        F ax[4];
        auto read_ax = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                if constexpr (NB == 4) ax[g] = ab[(g * 16 + l16) * PP + ((4 * wave + lq) ^ l16)];
                else ax[g] = reinterpret_cast<const F*>(ab + (g * 16 + l16) * PP + ((2 * wave + (lq >> 1)) ^ (l16 & 7)))[lq & 1];
            }
        };
        f32x4_t acc[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[b][e] = 0.0f;
        F cp = F{};
        if constexpr (!FIRST) {
            const __amdgpu_buffer_rsrc_t x = buffer(operand(now), chunks * CHUNK * 2);
            uint4 f[FR];
            if constexpr (SENTINEL) {
#pragma unroll
                for (int i = 0; i < FR; ++i) f[i] = ahead[i];
                if (await<FR>(f, x, off, false, a.abort_word, a.limit_ticks)) poison = __builtin_nanf("");
            } else {
                if (wait_counter(a.cnt + d * NT + sp.first + now.i, (unsigned)(nu * now.n), a.abort_word, a.limit_ticks)) poison = __builtin_nanf("");
                look_through<FR>(f, x, off);
            }
#pragma unroll
            for (int i = 0; i < FR; ++i) hb[(wave * FR + i) * 64 + lane] = f[i];
#pragma unroll
            for (int q = 0; q < FR; ++q)
#pragma unroll
                for (int b = 0; b < NB; ++b) acc[b] = mfma16(wf[b][q], f[q], acc[b]);
            __builtin_amdgcn_sched_barrier(0);
            lds_barrier();                               // one an item: the buffers are doubled
            if constexpr (SENTINEL) look(next);          // (behind the last item: of the last frame, not used)
            store_y();
            if constexpr (LOCAL) cp = state[now.i * 64 * NW];
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
            if constexpr (!LOCAL) cp = cur.cp;
        } else {
            lds_barrier();
            store_y();
        }
        read_ax();
        float gi[NB], gf[NB], gg[NB], go[NB], c[NB];
        unsigned hw[NB / 2];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            gi[b] = fast_sigmoid(part(ax[0], b) + acc[b][0]);
            gf[b] = fast_sigmoid(part(ax[1], b) + acc[b][1]);
            gg[b] = fast_tanh(part(ax[2], b) + acc[b][2]);
            go[b] = fast_sigmoid(part(ax[3], b) + acc[b][3]);
            c[b] = next_cell(gf[b], part(cp, b), gi[b], gg[b]);
            const unsigned h = coh_bf16(go[b] * fast_tanh(c[b]) + poison);
            hw[b >> 1] = b & 1 ? hw[b >> 1] | (h << 16) : h;
        }
        put_exchange(near, buffer(a.hx + ((size_t)(t * 2 + d) * NT + sp.first + now.i) * chunks * CHUNK, (unsigned)chunks * CHUNK * 2), x_off, pack(hw));
        if constexpr (!SENTINEL) signal_counter(a.cnt + d * NT + sp.first + now.i);
        const size_t rec = record(t, now.i);
        if constexpr (LOCAL) state[now.i * 64 * NW] = pack(c);
        else put<later(SENTINEL)>(buffer(reinterpret_cast<F*>(a.c) + rec, RT * (unsigned)sizeof(F)), c_off, pack(c));   // (before the loads that may read it)
        inputs(third, nxt);
        const __amdgpu_buffer_rsrc_t g4 = buffer(reinterpret_cast<uint4*>(a.gates) + rec * (NB / 2), RT * (NB / 2) * 16);
#pragma unroll
        for (int k = 0; k < NB / 2; ++k)
            put<later(SENTINEL)>(g4, g_off + k * RT * 16, make_uint4(pack_bf2(gi[2 * k], gf[2 * k]), pack_bf2(gg[2 * k], go[2 * k]), pack_bf2(gi[2 * k + 1], gf[2 * k + 1]), pack_bf2(gg[2 * k + 1], go[2 * k + 1])));
        if constexpr (LOCAL) put<later(SENTINEL)>(buffer(reinterpret_cast<F*>(a.c) + rec, RT * (unsigned)sizeof(F)), c_off, pack(c));
        ys[par * 256 + turned(l16, 4 * wave + lq)] = pack(hw);
#pragma unroll
        for (int k = 0; k < NB / 2; ++k) fill_word();
        before = now; now = next; next = third; third.next(ntl);
        par ^= 1;
    };
    auto walk = [&](auto first_frame, int items) __attribute__((always_inline)) {
        In in0, in1, in2;
        inputs(now, in0);
        inputs(next, in1);
        __builtin_amdgcn_s_waitcnt(0x0F70);              // vmcnt(0): once, or the way in would count in every item's waits
        for (;;) {
            do_item(first_frame, in0, in2);
            if (--items == 0) break;
            do_item(first_frame, in1, in0);
            if (--items == 0) break;
            do_item(first_frame, in2, in1);
            if (--items == 0) break;
        }
        keep(now); keep(next); keep(third);
    };
    walk(std::true_type{}, ntl);
    if (T > 1) {
        if constexpr (SENTINEL) look(now);
        walk(std::false_type{}, (T - 1) * ntl);
    }
    lds_barrier();
    store_y();
    while (fill_off < fill_bytes) fill_word();           // (whatever rounding left over)
}

// ------------------------------------------------------------------------------ backward
// With two tiles a workgroup the next item's operand went out with the item before, and asked for straight behind the barrier it is still on its way: the look is
// timed, so many clocks behind the wavefront's own stores.  us a launch, straight / 2000 / 2500 / 3000 / 3500 clocks: 700 sequences of 256 cells 115.5 / 108 / 97 / 99 / 107, 700 of
// 200 120 / 112 / 104 / 102 / 106, 600 of 384 135 / 133 / 114 / 117 / 123, 520 of 320 108 / 106 / 101 / 107 / 113; 300 of 512, whose items take longer, 104 / 106 / 107 / 114 / 122
// (straight there); with more tiles the operand is older (1000 of 320 132 / 134 / 141 / 152 / 163).
constexpr unsigned bwd_pause(int kq) { return kq == 8 || kq == 12 ? 2500 : 0; }
template <int NB, int KQ, bool SENTINEL, bool LOCAL>
__global__ __launch_bounds__(64 * NW, bwd_per_cu(NB, KQ, true)) void multi_tile_rec_bwd_kernel(RecBwdArgs a) {
    typedef typename Packs<NB>::F F;
    typedef typename Packs<NB>::W W;
    constexpr int BW = KQ / 4, SL = 4;                   // fragments checked and asked for together
    constexpr int AP = 2 * NB;                           // 16-byte pieces of dE/da a row and gate
    extern __shared__ float4 ps[];                       // [2][NW][NB][64], uint4 [2][4][16][AP] dE/da, W [2][16][16] dy, then (LOCAL) F [tiles][2][64 NW]: c, dE/dc
    const int T = a.T, B = a.B, H = a.H;
    const int chunks = H / 8, nu = (H + 16 * NB - 1) / (16 * NB), NT = (B + 15) / 16;
    const Spot sp = spot(nu, a.nbg, NT, SENTINEL);
    const int d = sp.d, ntl = sp.ntl;
    if (ntl <= 0) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint4* const das = reinterpret_cast<uint4*>(ps + 2 * NW * NB * 64);
    W* const dys = reinterpret_cast<W*>(das + 2 * 4 * 16 * AP);
    F* const state = reinterpret_cast<F*>(dys + 2 * 256) + tid;
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
    park<0>(wf);
    // fragment q: gate q / BW, block q0 + q % BW of 32 columns
    unsigned offb[BW];                                   // bytes, within a gate
#pragma unroll
    for (int q = 0; q < BW; ++q) offb[q] = (unsigned)(min(4 * (q0 + q) + lq, chunks - 1) * CHUNK + l16 * 8) * 2;
    auto offsets = [&](int s, unsigned (&o)[SL]) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < SL; ++q) o[q] = (unsigned)((s * SL + q) / BW) * (unsigned)(chunks * CHUNK * 2) + offb[(s * SL + q) % BW];
    };
    const int unit0 = (sp.u * NW + wave) * 4 * NB;       // this wavefront's units; the lane's: j .. j + NB - 1 of row l16
    const int j = unit0 + NB * lq, jc = min(j, H - NB);
    const unsigned RT = (unsigned)(H / NB) * 16, rec0 = (unsigned)(jc / NB) * 16 + l16;
    const unsigned XT = (unsigned)4 * chunks * CHUNK;    // exchange elements of a (frame, direction, tile)
    // eight units of one gate a lane (see below): where they go
    const int gate0 = NB == 2 ? lq : 2 * (lq & 1), u8 = NB == 2 ? unit0 : unit0 + 8 * (lq >> 1);
    const unsigned x_off = u8 < H ? (unsigned)((gate0 * chunks + (u8 >> 3)) * CHUNK + l16 * 8) * 2 : DROP;
    // what this lane moves of the row-major tensors: dy, row y_row, word l16; dE/da, gate `wave` of rows a_row + 64 k / AP, piece a_p
    const int y_row = 4 * wave + lq, a_row = lane / AP, a_p = lane % AP, a_unit = sp.u * 16 * NB + 8 * a_p;
    const unsigned y_off = (unsigned)min(sp.u * 16 * NB + NB * l16, H - NB) * 2, a_off = a_unit < H ? (unsigned)(a_row * 8 * H + wave * H + a_unit) * 2 : DROP;
    auto da_slot = [&](int gate, int row, int p) { return (gate * 16 + row) * AP + (p ^ (NB == 4 ? row >> 1 : row >> 2)); };
    const unsigned dc_off = j < H ? rec0 * (unsigned)sizeof(F) : DROP;
    auto frame = [&](int ni) { return d ? ni : T - 1 - ni; };   // (the last one visited forward comes first)
    auto record = [&](int t, int i) { return ((size_t)(t * 2 + d) * NT + sp.first + i) * RT; };
    struct In { W dy; uint4 g[NB / 2]; F cp, c; };
    auto inputs = [&](auto first_frame, const Item& p, In& in) __attribute__((always_inline)) {
        const int ni = min(p.n, T - 1), t = frame(ni), row0 = (sp.first + p.i) * 16;
        in.dy = get<W>(a.dy + ((size_t)t * B + row0) * 2 * H + d * H, (unsigned)(min(y_row, B - 1 - row0) * 2 * H) * 2 + y_off);
        const size_t rec = record(t, p.i);
#pragma unroll
        for (int k = 0; k < NB / 2; ++k) in.g[k] = get<uint4>(reinterpret_cast<const uint4*>(a.gates) + rec * (NB / 2) + (size_t)k * RT, rec0 * 16);
        in.cp = get<F>(reinterpret_cast<const F*>(a.c) + record(frame(min(ni + 1, T - 1)), p.i), rec0 * (unsigned)sizeof(F));
        if constexpr (decltype(first_frame)::value) in.c = get<F>(reinterpret_cast<const F*>(a.c) + rec, rec0 * (unsigned)sizeof(F));
    };
    auto operand = [&](const Item& p) { return a.dax + ((size_t)(frame(p.n - 1) * 2 + d) * NT + sp.first + p.i) * XT; };   // (behind the first frame)
    uint4 f[KQ / SL][SL];
    auto look = [&](__amdgpu_buffer_rsrc_t x, int s) __attribute__((always_inline)) {
        unsigned o[SL];
        offsets(s, o);
        look_through<SL>(f[s], x, o);
    };
    float poison = ld_coh_u32(a.abort_word) != 0 ? __builtin_nanf("") : 0.0f;
    Item now{0, 0}, next{0, 0}, third{0, 0};
    next.next(ntl); third = next; third.next(ntl);
    int par = 0;                                         // of the item: which of the two buffers
    const bool timed = SENTINEL && bwd_pause(KQ) > 0 && ntl == 2;
    unsigned long long stored = 0;                       // when the last dE/da went out
    Item before{-1, 0};                                  // the item whose dE/da waits in LDS for the other wavefronts
    auto store_da = [&]() __attribute__((always_inline)) {
        const int t = frame(max(before.n, 0)), row0 = (sp.first + before.i) * 16;
        const unsigned bytes = before.n < 0 ? 0u : (unsigned)((min(B - row0, 16) - 1) * 8 * H + 4 * H) * 2;
        const __amdgpu_buffer_rsrc_t p = buffer(a.da + ((size_t)t * B + row0) * 8 * H + d * 4 * H, bytes);
#pragma unroll
        for (int k = 0; k < NB / 2; ++k) put<later(SENTINEL)>(p, a_off + (unsigned)(k * 8 * 8 * H * 2), das[(par ^ 1) * 4 * 16 * AP + da_slot(wave, a_row + 8 * k, a_p)]);
    };
    auto do_item = [&](auto first_frame, const In& cur, In& nxt) __attribute__((always_inline)) {
        constexpr bool FIRST = decltype(first_frame)::value;
        const int t = frame(now.n);
        float4* const pt = ps + par * NW * NB * 64;
        dys[par * 256 + turned(y_row, l16)] = cur.dy;
        float dh[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) dh[b] = 0.0f;
        const size_t carried = ((size_t)d * NT + sp.first + now.i) * RT;
        F c = cur.c, dcp = F{};
        if constexpr (!FIRST) {
            const __amdgpu_buffer_rsrc_t x = buffer(operand(now), XT * 2);
            if constexpr (!LOCAL) {
                c = get<F>(reinterpret_cast<const F*>(a.c) + record(t, now.i), rec0 * (unsigned)sizeof(F));
                dcp = get<F>(reinterpret_cast<const F*>(a.dc) + carried, rec0 * (unsigned)sizeof(F));
            }
            bool gu = false;
            if constexpr (!SENTINEL) {
                gu = wait_counter(a.cnt + d * NT + sp.first + now.i, (unsigned)(nu * now.n), a.abort_word, a.limit_ticks);
#pragma unroll
                for (int s = 0; s < KQ / SL; ++s) look(x, s);
            }
            f32x4_t acc[NB];
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[b][e] = 0.0f;
#pragma unroll
            for (int s = 0; s < KQ / SL; ++s) {
                if constexpr (SENTINEL) {
                    unsigned o[SL];
                    offsets(s, o);
                    gu = await<SL>(f[s], x, o, gu, a.abort_word, a.limit_ticks);
                }
#pragma unroll
                for (int q = 0; q < SL; ++q)
#pragma unroll
                    for (int b = 0; b < NB; ++b) acc[b] = mfma16(wf[b][s * SL + q], f[s][q], acc[b]);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (gu) poison = __builtin_nanf("");
            if constexpr (LOCAL) { c = state[now.i * 2 * 64 * NW]; dcp = state[(now.i * 2 + 1) * 64 * NW]; }
#pragma unroll
            for (int b = 0; b < NB; ++b) pt[(wave * NB + b) * 64 + lane] = make_float4(acc[b][0], acc[b][1], acc[b][2], acc[b][3]);
            lds_barrier();                               // one an item: the buffers are doubled
            if constexpr (SENTINEL) {                    // (behind the last item: of the last frame, not used)
                if (timed) while (__builtin_amdgcn_s_memtime() - stored < bwd_pause(KQ)) {}
#pragma unroll
                for (int s = 0; s < KQ / SL; ++s) look(buffer(operand(next), XT * 2), s);
            }
            store_da();
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
        } else {
            lds_barrier();
            store_da();
        }
        const W dy = dys[par * 256 + turned(l16, 4 * wave + lq)];
        const bool last = now.n == T - 1;                // (the frame visited first forward has no cell state before it)
        float dcn[NB];
        unsigned da[4][NB / 2];                          // a gate's units
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const uint4 g = cur.g[b >> 1];
            const unsigned gif = b & 1 ? g.z : g.x, ggo = b & 1 ? g.w : g.y, dyw = word(dy, b >> 1);
            const float gi = bf2f((bf16_t)(gif & 0xFFFFu)), gf = bf2f((bf16_t)(gif >> 16));
            const float gg = bf2f((bf16_t)(ggo & 0xFFFFu)), go = bf2f((bf16_t)(ggo >> 16));
            const float dht = dh[b] + bf2f((bf16_t)(b & 1 ? dyw >> 16 : dyw & 0xFFFFu)) + poison;
            const float tc = fast_tanh(part(c, b)), cp = last ? 0.0f : part(cur.cp, b);
            const float dc = dht * go * (1.0f - tc * tc) + part(dcp, b);
            const unsigned v[4] = {coh_bf16(dc * gg * gi * (1.0f - gi)), coh_bf16(dc * cp * gf * (1.0f - gf)),
                                   coh_bf16(dc * gi * (1.0f - gg * gg)), coh_bf16(dht * tc * go * (1.0f - go))};
#pragma unroll
            for (int k = 0; k < 4; ++k) da[k][b >> 1] = b & 1 ? da[k][b >> 1] | (v[k] << 16) : v[k];
            dcn[b] = dc * gf;
        }
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
        const __amdgpu_buffer_rsrc_t x = buffer(a.dax + ((size_t)(t * 2 + d) * NT + sp.first + now.i) * XT, XT * 2);
#pragma unroll
        for (int k = 0; k < NB / 2; ++k) put<SC1>(x, x_off + (unsigned)(k * chunks * CHUNK * 2), o[k]);
        if (timed) stored = __builtin_amdgcn_s_memtime();
        if constexpr (!SENTINEL) signal_counter(a.cnt + d * NT + sp.first + now.i);
        if constexpr (LOCAL) { state[now.i * 2 * 64 * NW] = cur.cp; state[(now.i * 2 + 1) * 64 * NW] = pack(dcn); }
        else put<later(SENTINEL)>(buffer(reinterpret_cast<F*>(a.dc) + carried, RT * (unsigned)sizeof(F)), dc_off, pack(dcn));
        inputs(first_frame, third, nxt);
#pragma unroll
        for (int k = 0; k < NB / 2; ++k) das[par * 4 * 16 * AP + da_slot(gate0 + k, l16, (u8 >> 3) - sp.u * AP)] = o[k];
        before = now;
        now = next; next = third; third.next(ntl);
        par ^= 1;
    };
    auto walk = [&](auto first_frame, int items) __attribute__((always_inline)) {
        In in0, in1, in2;
        inputs(first_frame, now, in0);
        inputs(first_frame, next, in1);
        __builtin_amdgcn_s_waitcnt(0x0F70);              // vmcnt(0), as in the forward kernel
        for (;;) {
            do_item(first_frame, in0, in2);
            if (--items == 0) break;
            do_item(first_frame, in1, in0);
            if (--items == 0) break;
            do_item(first_frame, in2, in1);
            if (--items == 0) break;
        }
        keep(now); keep(next); keep(third);
    };
    walk(std::true_type{}, ntl);
    if (T > 1) {
        if constexpr (SENTINEL) {
#pragma unroll
            for (int s = 0; s < KQ / SL; ++s) look(buffer(operand(now), XT * 2), s);
        }
        walk(std::false_type{}, (T - 1) * ntl);
    }
    lds_barrier();
    store_da();
}

template <int NB, int KQ, bool S, bool LOCAL>
hipError_t run(const RecFwdArgs& a, size_t lds, int grid, int real, hipStream_t st, bool* launched) {
    return launch_resident<multi_tile_rec_fwd_kernel<NB, KQ, S, LOCAL>>(a, 64 * NW, lds, grid, real, st, launched);
}
template <int NB, int KQ, bool S, bool LOCAL>
hipError_t run(const RecBwdArgs& a, size_t lds, int grid, int real, hipStream_t st, bool* launched) {
    return launch_resident<multi_tile_rec_bwd_kernel<NB, KQ, S, LOCAL>>(a, 64 * NW, lds, grid, real, st, launched);
}
template <int NB, int KQ, bool S, typename A>
hipError_t run_state(const A& a, int grid, int real, hipStream_t st, bool* launched) {
    constexpr bool fwd = std::is_same_v<A, RecFwdArgs>;
    // LDS: beside the carried state, and that of a tile
    constexpr size_t base = 2 * (fwd ? (size_t)KQ * 64 * 16 + 4 * 16 * 4 * NB * 16 + 256 * NB * 2 : (size_t)NW * NB * 64 * 16 + 4 * 16 * 2 * NB * 16 + 256 * NB * 2), tile = (size_t)(fwd ? 1 : 2) * 64 * NW * NB * 4;
    const size_t lds = base + tile * a.tiles_per_group;
    if (lds <= LDS_MOST / (fwd ? fwd_per_cu(NB, KQ, true) : bwd_per_cu(NB, KQ, true))) return run<NB, KQ, S, true>(a, lds, grid, real, st, launched);
    return run<NB, KQ, S, false>(a, base, grid, real, st, launched);
}
template <typename A>
hipError_t launch(const A& a, int nb, int kq, bool sentinel, int grid, int real, hipStream_t st, bool* launched) {
#define BLSTM_MULTI(NB, KQ) if (nb == NB && kq == KQ && sentinel) return run_state<NB, KQ, true>(a, grid, real, st, launched)
#define BLSTM_FENCED(NB, KQ) if (nb == NB && kq == KQ) return run_state<NB, KQ, false>(a, grid, real, st, launched)
    BLSTM_MULTI(2, 4); BLSTM_MULTI(4, 4); BLSTM_MULTI(4, 8); BLSTM_MULTI(4, 12); BLSTM_MULTI(4, 16);
    BLSTM_FENCED(4, 4); BLSTM_FENCED(4, 8); BLSTM_FENCED(4, 16);
#undef BLSTM_MULTI
#undef BLSTM_FENCED
    return hipSuccess;
}

}  // namespace

hipError_t launch_rec_multi(const RecFwdArgs& a, int nb, int kq, bool sentinel, int grid, int real, hipStream_t st, bool* launched) { return launch(a, nb, kq, sentinel, grid, real, st, launched); }
hipError_t launch_rec_multi(const RecBwdArgs& a, int nb, int kq, bool sentinel, int grid, int real, hipStream_t st, bool* launched) { return launch(a, nb, kq, sentinel, grid, real, st, launched); }

}  // namespace blstm
