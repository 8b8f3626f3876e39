// Persistent recurrent kernels: all T frames of one layer, both directions, in one launch.
//
// A workgroup owns 32 hidden units of one direction (all four gate rows of each) and a group
// of 32-row batch tiles.  Its slice of U_h stays in vector registers for the whole launch:
// NW wavefronts split the contraction index, each holding its part as MFMA B-fragments (64 to 256
// VGPRs per lane, by width).
// Per frame and batch tile a workgroup multiplies the previous h (forward) or the previous
// frame's gate gradients (backward) by its slice, reduces the NW partial accumulators through
// LDS, applies the cell arithmetic with all four gates of a unit in one lane, and writes its
// 32 columns.  The NU = H/32 workgroups that share a batch tile exchange these columns through
// global memory.  The exchanged tensor is a copy kept in the order the consumers' MFMA A-fragments
// want it, [frame][direction][32-row tile][16-column pair of chunks][chunk][row][8 columns]: a
// wavefront's load of one fragment is then one contiguous KB (row-major storage makes the same
// load touch 32 separate cache lines and runs three times slower), and a producer's 32 columns
// of a tile are one contiguous 2 KB block.  The row-major tensors the products outside these
// kernels read (h for the next layer, dE/da for the weight and input gradients) are written
// as well, off the frame-to-frame path.  Two protocols order the exchange:
//
//   SENTINEL  The exchanged tensor (h, or dE/da) is filled with the bf16 bit pattern 0xFFFF (a
//             NaN no finite value converts to) before the launch.  Producers store write-through
//             at agent scope, consumers load cache-bypassing at agent scope and take a chunk only
//             when none of its elements is the sentinel.  Each element is written once and is
//             its own ready flag: no counters, no fences, no barriers beyond the LDS reduction.
//   FENCED    Plain stores and loads ordered by a per-(group, tile) counter that is incremented
//             with agent-scope release semantics and polled with acquire semantics.
//
// Every wait is bounded by a wall-clock limit.  On expiry the wave raises a global abort word;
// every later wait returns at once when it sees the word, so all waves run to the end of the
// kernel.  A wave that abandoned a wait adds NaN to everything it writes from then on (h in the
// forward kernel, dE/da in the backward one), so the failure travels in-band into the loss, the
// gradient and the updated weights; blstm_device_status reports it as well.
#include "exchange.hpp"
#include "kernels.hpp"
#include "residency.hpp"

namespace blstm {
namespace {

__device__ __forceinline__ f32x16_t mfma_bf16(const uint4& a, const uint4& b, f32x16_t c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

// ---- SENTINEL protocol --------------------------------------------------------------------------
// Bounded wait of one wave.  `probe` points, for the lanes with probing set, at one element of each
// producer's block: a cheap first look before the full loads.  Returns true if the wait was
// abandoned (time limit, or the abort word raised by anyone).  Wave-uniform control flow.
__device__ __forceinline__ bool wait_probe(const bf16_t* probe, bool probing, unsigned* abort_word,
                                           unsigned long long limit_ticks) {
    const unsigned long long t0 = wall_clock64();
    unsigned it = 0;
    for (;;) {
        bool ready = true;
        if (probing) ready = __hip_atomic_load(probe, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != SENT16;
        if (__all(ready)) return false;
        __builtin_amdgcn_s_sleep(1);
        if ((++it & 31u) == 0) {
            if (ld_coh_u32(abort_word) != 0) return true;
            if (wall_clock64() - t0 > limit_ticks) {
                __hip_atomic_store(abort_word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                return true;
            }
        }
    }
}

constexpr int XPAIR = 2 * 32 * 8;                      // elements of one pair of 8-column chunks over 32 rows (1 KB)
// `last`: pairs beyond it (of a width padded to the kernel's) repeat that pair, against zero weights.
template <int NQ>
__device__ __forceinline__ void load_chunks(uint4 (&frag)[NQ], const bf16_t* p, int last) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) frag[q] = ld_coh_16B(p + min(q, last) * XPAIR);
}
// The chunks in frag were loaded once; reloads them until no element of any lane is the sentinel
// (or the wait is abandoned).  Normally the first check passes.
template <int NQ, bool APART = false>
__device__ __forceinline__ bool ensure_written(uint4 (&frag)[NQ], const bf16_t* p, int last, bool give_up,
                                               unsigned* abort_word, unsigned long long limit_ticks) {
    if (give_up || all_written<NQ, APART>(frag)) return give_up;
    const unsigned long long t0 = wall_clock64();
    unsigned it = 0;
    for (;;) {
        __builtin_amdgcn_s_sleep(1);
        load_chunks<NQ>(frag, p, last);
        if (all_written<NQ, APART>(frag)) return false;
        if ((++it & 31u) == 0) {
            if (ld_coh_u32(abort_word) != 0) return true;
            if (wall_clock64() - t0 > limit_ticks) {
                __hip_atomic_store(abort_word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                return true;
            }
        }
    }
}

// The same through a buffer, past the L1: a scalar offset per pair and one register of lanes' offsets, which leaves the registers to the
// weights.  `p`: the first pair (uniform).
template <int NQ>
__device__ __forceinline__ void load_pairs(uint4 (&frag)[NQ], const bf16_t* p, int last) {
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(p), 0, (min(NQ - 1, last) + 1) * XPAIR * 2, 0x00020000);
#pragma unroll
    for (int q = 0; q < NQ; ++q) frag[q] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)(threadIdx.x & 63) * 16, min(q, last) * XPAIR * 2, 16));
}
// ... and again until all of them are written.  Returns true if the wait was abandoned.
template <int NQ>
__device__ __forceinline__ bool await_pairs(uint4 (&frag)[NQ], const bf16_t* p, int last, unsigned* abort_word, unsigned long long limit_ticks) {
    return wait_written<false, NQ>(frag, [&]() __attribute__((always_inline)) { load_pairs<NQ>(frag, p, last); }, false, abort_word, limit_ticks);
}
// Keeps all of the weights in accumulation registers, which the products read as well as the others.
template <int NG, int NQ>
__device__ __forceinline__ void park_all(uint4 (&w)[NG][NQ]) {
    typedef unsigned u4 __attribute__((ext_vector_type(4)));
    __builtin_amdgcn_s_waitcnt(0x0F70);                  // vmcnt(0): one wait for all of them
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            u4 v = __builtin_bit_cast(u4, w[g][q]);
            asm volatile("" : "+a"(v));
            w[g][q] = __builtin_bit_cast(uint4, v);
        }
}

struct GroupMap { int d, u, bg, group; };

// Workgroups that exchange data sit on one XCD when ids are dealt round-robin over eight XCDs
// (a performance assumption only; correctness rests on the protocols above).  The grid holds a whole number of groups
// per XCD (grid_groups); the workgroups of the groups that do not exist have no batch tile and leave at once.
constexpr int grid_groups(int nbg) { return (2 * nbg + 7) & ~7; }
__device__ __forceinline__ GroupMap map_block(int NU, int nbg) {
    const int x = blockIdx.x;
    const int slot = x >> 3;
    const int group = (x & 7) + 8 * (slot / NU);
    GroupMap m;
    m.group = group; m.u = slot % NU; m.d = group / nbg; m.bg = group % nbg;
    return m;
}

// First attempt at the exchanged chunks: ordinary cached loads.  Every element is either the
// sentinel or its final value (it is written once, after the pre-fill), so whatever cache level
// answers, a chunk without sentinels is correct; anything else is re-read cache-bypassing by
// ensure_written.
template <int NQ>
__device__ __forceinline__ void load_chunks_cached(uint4 (&frag)[NQ], const bf16_t* p, int last) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) frag[q] = *reinterpret_cast<const uint4*>(p + min(q, last) * XPAIR);
}
// Element offset of column c (within a direction), row r of a tile, in the exchange order.
__device__ __forceinline__ unsigned xoff(int c, int r) { return (unsigned)((c >> 3) * 256 + r * 8 + (c & 7)); }

// Saved activations of the persistent kernels ("records"): the forward kernel's lane (workgroup of unit slice u, thread
// tid) owns four cells of a (frame, direction, batch tile) and the backward kernel's lane of the same ids owns the same
// four, so what one saves for the other is indexed [frame][direction][tile][unit slice][word][thread] in 16-byte
// words: a lane reads back exactly what it wrote, with one wide access per word instead of one per cell.
__device__ __forceinline__ size_t rec_index(int t, int d, int tile, int NT, int NU, int u) {
    return ((size_t)(t * 2 + d) * NT + tile) * NU + u;
}

// Number of 32-row batch tiles of this workgroup's group that lie inside the batch.
__device__ __forceinline__ int tiles_in_batch(int bg, int tiles_per_group, int B) {
    const int first = bg * tiles_per_group * 32;
    if (first >= B) return 0;
    const int n = (B - first + 31) / 32;
    return n < tiles_per_group ? n : tiles_per_group;
}

constexpr int NW = 4;                                    // wavefronts

// ------------------------------------------------------------------------------ forward
// KW = contraction elements per wavefront: H = NW * KW.
// FULL: B is a multiple of 32, so every row of every tile exists.  Otherwise the rows of the last tile beyond the batch
// repeat the batch's last row: their loads are clamped to it, they run through the recurrence and the exchange (whole
// tiles of both) like any other row, no row's result depends on another row's, and only the row-major stores leave them
// out.  No load is predicated: with one branch per loaded row a ragged batch took 119 us a layer where 256 whole rows
// took 76 (H = 512, 173 sequences; the backward kernel 104 against 83).
// MULTI: a workgroup owns several batch tiles (tiles_per_group > 1).
// PADDED: the layer is narrower than the kernel's NW * KW cells (any multiple of 8): U_h counts as zero beyond it, the
// exchange holds whole slices of 32 units, and the units beyond the layer come out as zeros that are not stored row-major.
// LEAN: few enough registers for two workgroups per CU, one of which computes while the other waits for its operand: one set of
// inputs, asked for behind the item's own operand, and half of the accumulators at a time.  Marks RecFwdArgs::fill on the side.
template <int KW, bool SENTINEL, bool FULL, bool MULTI, bool PADDED, bool LEAN>
__global__ __launch_bounds__(64 * NW, LEAN ? 2 : 1) void rec_fwd_kernel(RecFwdArgs a) {
    static_assert(!LEAN || (SENTINEL && MULTI && PADDED && KW < 128), "the forms that are used");
    // AHEAD (wide slices, several tiles): the next item's operand, written a frame ago, is asked for once the products have left its
    // registers, and every load and store is issued on every path, so that the waits,
    // which are counted, are for what is needed and not for what has just been asked for.  The weights stay in accumulation
    // registers.  The item's own inputs and what the item before stores for later launches, 23 vector-memory instructions a wavefront, go out one at a time
    // between the products: behind the cells they took 1500 to 1900 clocks of an item, the wavefront waiting to issue them.  The partial sums are in LDS
    // twice, so that one barrier an item is enough.  An item of 1024 units is 6900 clocks (8600 before): 320 looking its operand through, 2650
    // products and sums to LDS, 600 at the barrier, 600 + 700 reading the sums and asking for the next operand (the CU takes an instruction of 1 KB
    // every 25 to 35), 1100 cells, 300 h.  Asking for the next operand between the products too made the products wait (5500 clocks), and
    // a_x in 16-byte pieces turned in LDS was no faster (311 / 321).  A layer, 21 frames, us, forward, two sets of inputs and a probe of the producers / operand
    // ahead, inputs and stores behind the cells / so: 512 sequences of 1024 units - / 365 / 311, 256 of 1024
    // - / 172 / 147, 700 of 1024 - / 495 / 413, 384 - / 259 / 224, 300 of 768 - / 204 / 186, 1000 of 544 553 / 496 / 457, 512 of 640 - / 256 / 242, 150 of 640
    // - / 119 / 115 (on a card where the operand ahead took 365, others 343; the compiler spills 10 to 15 scalar registers in five of the six forms, which had none).
    // Backward, the first two: 512 of 1024 406 / 385, 256 of 1024 206 / 192, 600 of 768 449 / 399, 1000 of 640 653 / 569, 130 of 544 166 / 143; a second buffer of the sums, without the barrier
    // at an item's end, loses a tenth (426 / 466, on the slower card).  dE/da's copies are marked on the side (1024: 51 us a step less for two layers).
    // Taking the pairs of the operand in another order in each workgroup gave nothing, more slabs in flight backward lost 2 to 8 %.
    constexpr bool AHEAD = MULTI && SENTINEL && !LEAN;
    constexpr int EPT = 16 / NW;                         // accumulator registers (batch rows) per thread
    constexpr int KSTEPS = KW / 16;                      // MFMA steps per gate per wavefront
    extern __shared__ float lds[];                       // [AHEAD ? 2 : 1][NW][4][4][64][4] partial accumulators, [NW][128] regrouping of h
    const int H = PADDED ? a.H : NW * KW;                // (the launcher picks KW from a.H)
    const int B = a.B, T = a.T;
    const int NU = PADDED ? (H + 31) / 32 : NW * KW / 32;
    const GroupMap gm = map_block(NU, a.nbg);
    const int d = gm.d, u = gm.u;
    const int lane = threadIdx.x & 63, wave = PADDED || AHEAD ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : threadIdx.x >> 6;
    const int l32 = lane & 31, lh = lane >> 5;
    const int ntl = d < 2 ? tiles_in_batch(gm.bg, a.tiles_per_group, B) : 0;   // (d >= 2: a group that does not exist)
    // this workgroup's share of the region to fill, some words every item behind its stores (a share is far below 2^32 words)
    const unsigned long long share = (LEAN || AHEAD) && a.fill ? (a.fill_words + gridDim.x - 1) / gridDim.x : 0ull;
    const unsigned long long fill_first = min(a.fill_words, (unsigned long long)blockIdx.x * share);
    uint4* const fill = static_cast<uint4*>(a.fill) + fill_first;
    const unsigned fill_end = (unsigned)(min(a.fill_words, fill_first + share) - fill_first);
    unsigned fill_pos = threadIdx.x;
    auto fill_some = [&](int words) __attribute__((always_inline)) {
        if constexpr (LEAN || AHEAD) for (int k = 0; k < words && fill_pos < fill_end; ++k, fill_pos += 64 * NW) fill[fill_pos] = make_uint4(~0u, ~0u, ~0u, ~0u);
    };
    if (ntl == 0) { fill_some(1 << 30); return; }        // no batch tile of its own
    const int fill_each = (int)((share + (unsigned long long)(64 * NW) * (T * ntl) - 1) / ((unsigned long long)(64 * NW) * (T * ntl)));

    // this wavefront's slice of U_h as B-fragments: unit row l32 of each gate, 8 consecutive k per lane
    uint4 bfrag[4][KSTEPS];
    {
        const bf16_t* uh = a.uh[d];
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int q = 0; q < KSTEPS; ++q) {
                const int unit = u * 32 + l32, k = wave * KW + q * 16 + 8 * lh;
                const bool in = !PADDED || (unit < H && k < H);
                bfrag[g][q] = in ? *reinterpret_cast<const uint4*>(uh + (size_t)(g * H + unit) * H + k) : make_uint4(0, 0, 0, 0);
            }
    }
    if constexpr (AHEAD) park_all(bfrag);
    unsigned* cnt = a.cnt + (size_t)gm.group * a.tiles_per_group;
    const int j = u * 32 + l32;                          // this thread's hidden unit
    float4* l4 = reinterpret_cast<float4*>(lds);
    unsigned* const xs = reinterpret_cast<unsigned*>(lds) + (AHEAD ? 2 : 1) * NW * 4 * 4 * 64 * 4 + (threadIdx.x >> 6) * 128;

    // Addresses are a per-item uniform base (frame and tile origin) plus per-thread 32-bit element
    // offsets computed once: brow[e] is the batch row of accumulator register e within a tile.
    // Register e is batch row rb + re(e) of the tile: rb per thread, re(e) a compile-time constant.
    const int rb = 2 * EPT * wave + 4 * lh;
    auto re = [](int e) { return 8 * (e >> 2) + (e & 3); };
    const bool junit = !PADDED || j < H;                 // (a unit beyond the layer reads its last one's a_x and counts it as zero)
    const unsigned o8c = (unsigned)(d * 4 * H + (PADDED ? min(j, H - 1) : j));   // column in the row-major [.][8H] tensor (a_x)
    const unsigned o8b = (unsigned)(rb * 8 * H) + o8c;
    const int NT = (B + 31) / 32;                        // 32-row tiles of the batch
    const int XH = NU * 2 * XPAIR;                       // exchange elements per (frame, direction, tile)
    // this lane's 16 bytes of each chunk pair; the last pair that exists, counted from there
    const int firstp = PADDED ? min(wave * (KW / 16), NU * 2 - 1) : wave * (KW / 16), lastp = PADDED ? NU * 2 - 1 - firstp : KW;
    const unsigned ohp = (unsigned)(firstp * XPAIR + lane * 8);

    // Per-item inputs that do not depend on the exchange (a_x of the frame, previous cell state) are
    // loaded one item ahead, so that their HBM latency never sits on the frame-to-frame path.
    // Item = (visited frame n, batch tile i); this thread's EPT batch rows are accumulator
    // registers r = EPT*wave + e.
    auto issue_inputs = [&](int n, int i, float (&ax)[EPT][4], float (&cp)[EPT]) {
        const int t = d ? T - 1 - n : n;
        const int tp = d ? T - n : n - 1;
        const int b0 = (gm.bg * a.tiles_per_group + i) * 32;
        const float* axb = a.ax + ((size_t)t * B + b0) * 8 * H;
        // (a_x fetched as 16-byte pieces and transposed through LDS, a quarter of these loads, was measured: no gain with
        // one tile per workgroup, where the loads hide under the exchange wait, and slower with several)
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            const unsigned o = FULL ? o8b + (unsigned)(re(e) * 8 * H) : (unsigned)(min(rb + re(e), B - 1 - b0) * 8 * H) + o8c;
#pragma unroll
            for (int g = 0; g < 4; ++g) ax[e][g] = axb[o + (unsigned)(g * H)];
        }
        // the previous cell state of this lane's four cells is one 16-byte word of the saved records (one tile: c stays in registers)
        float4 c4 = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if constexpr (AHEAD) c4 = reinterpret_cast<const float4*>(a.c)[rec_index(n > 0 ? tp : t, d, b0 >> 5, NT, NU, u) * 256 + threadIdx.x];
        else if (n > 0 && ntl > 1) c4 = reinterpret_cast<const float4*>(a.c)[rec_index(tp, d, b0 >> 5, NT, NU, u) * 256 + threadIdx.x];
        cp[0] = c4.x; cp[1] = c4.y; cp[2] = c4.z; cp[3] = c4.w;
    };
    auto issue_item = [&](int item, float (&ax)[EPT][4], float (&cp)[EPT]) { const int n = item / ntl; issue_inputs(n, item - n * ntl, ax, cp); };

    const int nitems = T * ntl;
    // Two sets of input registers used in turn: an item computes from one while the next item's loads land
    // in the other, so nothing is copied (a copy would have to wait for loads issued a moment before).
    float ax0[EPT][4], cp0[EPT], ax1[EPT][4], cp1[EPT];
    if constexpr (!LEAN && !AHEAD) issue_inputs(0, 0, ax0, cp0);
    uint4 ahead[AHEAD ? KSTEPS : 1];                     // the operand of the item to come
    auto operand = [&](int n0, int i) {                  // this wavefront's part (the first frame, which has none: the second one's)
        const int n = max(n0, 1);
        return a.hx + ((size_t)((d ? T - n : n - 1) * 2 + d) * NT + gm.bg * a.tiles_per_group + i) * XH + firstp * XPAIR;
    };
    // Waited for here, once: the compiler places its waits for the worst path into the loop, and with these
    // loads still in flight on the way in, that path would make every item wait for its freshly issued loads.
    __builtin_amdgcn_s_waitcnt(0x0F70);                  // vmcnt(0) (expcnt and lgkmcnt left alone)
    float ccarry[EPT];                                   // one tile per workgroup: its cell state of the frame before
#pragma unroll
    for (int e = 0; e < EPT; ++e) ccarry[e] = 0.0f;
    // The row-major outputs of an item (c, the gates, h for the next layer) are not on the frame-to-frame path:
    // they wait in registers until the next item has issued its loads of the exchanged h, and go out behind them.
    struct Tail { int t, b0; bool have, xok; float cn[EPT]; uint2 g[EPT]; uint2 hq; } tail;
    tail.have = false; tail.t = 0; tail.b0 = 0;
    // NaN once this wave has abandoned a wait, or from the start if an earlier launch left the abort word raised:
    // added to every h it writes
    float poison = ld_coh_u32(a.abort_word) != 0 ? __builtin_nanf("") : 0.0f;
    auto flush_tail = [&]() __attribute__((always_inline)) {
        if (!tail.have) return;
        tail.have = false;
        bf16_t* yb = a.y + ((size_t)tail.t * B + tail.b0) * 2 * H;
        // What the backward kernel needs of this lane's four cells goes out as the lane's record: three 16-byte words
        // (gates of cells 0-1, gates of cells 2-3, the four cell states), each word array contiguous over the workgroup.
        {
            const size_t r = rec_index(tail.t, d, tail.b0 >> 5, NT, NU, u);
            uint4* g4 = reinterpret_cast<uint4*>(a.gates) + r * 2 * 256 + threadIdx.x;
            g4[0] = make_uint4(tail.g[0].x, tail.g[0].y, tail.g[1].x, tail.g[1].y);
            g4[256] = make_uint4(tail.g[2].x, tail.g[2].y, tail.g[3].x, tail.g[3].y);
            reinterpret_cast<float4*>(a.c)[r * 256 + threadIdx.x] = make_float4(tail.cn[0], tail.cn[1], tail.cn[2], tail.cn[3]);
        }
        const int lane_ = threadIdx.x & 63;
        const int xrow_ = 2 * EPT * (int)(threadIdx.x >> 6) + 4 * (lane_ >> 5) + ((lane_ >> 3) & 3);
        const unsigned xcol_ = (unsigned)(u * 32 + 8 * ((lane_ >> 1) & 3) + 4 * (lane_ & 1));
        if (tail.xok && (!PADDED || xcol_ < (unsigned)H)) *reinterpret_cast<uint2*>(yb + ((unsigned)xrow_ * (unsigned)(2 * H) + (unsigned)(d * H) + xcol_)) = tail.hq;
        fill_some(fill_each);
    };
    // AHEAD: every lane issues every store, what does not exist lies beyond the buffer
    const __amdgpu_buffer_rsrc_t fill_to = __builtin_amdgcn_make_buffer_rsrc(AHEAD && a.fill ? fill : nullptr, 0, AHEAD ? (int)(fill_end * 16) : 0, 0x00020000);
    // What an item stores for later launches, and its own inputs, one vector-memory instruction a step: they go out between the products, which the matrix
    // cores work through meanwhile.
    typedef unsigned u4 __attribute__((ext_vector_type(4)));
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    constexpr int SIDE = 6 + EPT * 4 + 1;
    auto side = [&](auto which, int n, int i, float (&ax)[EPT][4], float (&cp)[EPT]) __attribute__((always_inline)) {
        constexpr int k = decltype(which)::value;
        const size_t r = rec_index(tail.t, d, tail.b0 >> 5, NT, NU, u);
        if constexpr (k == 0) {                          // (c goes out first: where the group has one tile the inputs read it)
            const __amdgpu_buffer_rsrc_t c = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<float4*>(a.c) + r * 256, 0, tail.have ? 4096 : 0, 0x00020000);
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, make_float4(tail.cn[0], tail.cn[1], tail.cn[2], tail.cn[3])), c, (int)threadIdx.x * 16, 0, 0);
        } else if constexpr (k <= EPT * 4) {
            constexpr int e = (k - 1) / 4, g = (k - 1) % 4;
            const int t = d ? T - 1 - n : n, b0 = (gm.bg * a.tiles_per_group + i) * 32;
            const __amdgpu_buffer_rsrc_t x = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.ax) + ((size_t)t * B + b0) * 8 * H, 0, 32 * 8 * H * 4, 0x00020000);
            const int o = FULL ? (int)o8b * 4 : (int)((unsigned)(min(rb + re(e), B - 1 - b0) * 8 * H) + o8c) * 4;
            ax[e][g] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(x, o, ((FULL ? re(e) * 8 * H : 0) + g * H) * 4, 0));
        } else if constexpr (k == EPT * 4 + 1) {
            const float4 c4 = reinterpret_cast<const float4*>(a.c)[rec_index(n > 0 ? (d ? T - n : n - 1) : (d ? T - 1 - n : n), d, gm.bg * a.tiles_per_group + i, NT, NU, u) * 256 + threadIdx.x];
            cp[0] = c4.x; cp[1] = c4.y; cp[2] = c4.z; cp[3] = c4.w;
        } else if constexpr (k <= EPT * 4 + 3) {         // (not read again here: the L2 is left to the exchange copies, 1 to 2 %)
            constexpr int h = k - EPT * 4 - 2;
            const __amdgpu_buffer_rsrc_t g4 = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<u4*>(a.gates) + r * 2 * 256, 0, tail.have ? 8192 : 0, 0x00020000);
            __builtin_amdgcn_raw_buffer_store_b128(u4{tail.g[2 * h].x, tail.g[2 * h].y, tail.g[2 * h + 1].x, tail.g[2 * h + 1].y}, g4, (int)threadIdx.x * 16 + h * 4096, 0, 2);
        } else if constexpr (k == EPT * 4 + 4) {
            const int row = 2 * EPT * (int)(threadIdx.x >> 6) + 4 * (lane >> 5) + ((lane >> 3) & 3);
            const unsigned col = (unsigned)(u * 32 + 8 * ((lane >> 1) & 3) + 4 * (lane & 1));
            const __amdgpu_buffer_rsrc_t y = __builtin_amdgcn_make_buffer_rsrc(a.y + ((size_t)tail.t * B + tail.b0) * 2 * H + d * H, 0, tail.have ? ((min(B - tail.b0, 32) - 1) * 2 * H + H) * 2 : 0, 0x00020000);
            __builtin_amdgcn_raw_buffer_store_b64(u2{tail.hq.x, tail.hq.y}, y, col < (unsigned)H ? (int)((unsigned)row * 2 * H + col) * 2 : 0x7FFFFFF0, 0, 0);
        } else {
            __builtin_amdgcn_raw_buffer_store_b128(u4{~0u, ~0u, ~0u, ~0u}, fill_to, (int)(fill_pos * 16), 0, 2);   // (nontemporal too)
            fill_pos += 64 * NW;
        }
    };
    // (AHEAD: counted.  A division of an item's number costs 100 cycles where it stands; the forms that look at the operand when the item begins, too
    // early, gain by them: whole steps of two layers, us, without / with it: 128 sequences of 1024 cells 914 / 907, 100 853 / 851, 2048 of 160 1316 / 1312)
    int now_n = 0, now_i = 0;
    auto do_item = [&](const int item, const float (&ax)[EPT][4], const float (&cpl)[EPT], float (&axn)[EPT][4],
                       float (&cpn)[EPT]) __attribute__((always_inline)) {
        const int n = AHEAD ? now_n : item / ntl, i = AHEAD ? now_i : item - n * ntl;
        int next_n = 0, next_i = 0;                      // the next item (behind the last one: that one again, not used)
        if constexpr (AHEAD) {
            const bool over = item + 1 == nitems, wraps = i + 1 == ntl;
            next_n = !over && wraps ? n + 1 : n; next_i = over ? i : wraps ? 0 : i + 1;
            now_n = next_n; now_i = next_i;
        }
        const int t = d ? T - 1 - n : n;
        const int tp = d ? T - n : n - 1;
        const int b0 = (gm.bg * a.tiles_per_group + i) * 32;
        float sum[EPT][4];
#pragma unroll
        for (int e = 0; e < EPT; ++e)
#pragma unroll
            for (int g = 0; g < 4; ++g) sum[e][g] = 0.0f;
        if (n > 0) {
            // previous h of this batch tile: row l32, 8 consecutive k per lane
            const bf16_t* hb = a.hx + ((size_t)(tp * 2 + d) * NT + (b0 >> 5)) * XH;   // uniform: previous frame, this tile
            const bf16_t* hp = hb + ohp;
            uint4 afrag_own[AHEAD ? 1 : KSTEPS];
            auto& afrag = [&]() -> auto& { if constexpr (AHEAD) return ahead; else return afrag_own; }();
            if constexpr (AHEAD) {
                if (await_pairs<KSTEPS>(afrag, operand(n, i), lastp, a.abort_word, a.limit_ticks)) poison = __builtin_nanf("");
            } else if (SENTINEL) {
                // one probe per producing workgroup of this wavefront's k-range: its last unit, last row
                const bf16_t* probe = hb + xoff(PADDED ? min(wave * (KW / 32) + lane, NU - 1) * 32 + 31 : wave * KW + (lane & (KW / 32 - 1)) * 32 + 31, 31);
                bool gu = false;
                if constexpr (LEAN) {
                    // Straight for the data: the first look nearly always finds everything.  If not: the cheap probe, then cache-bypassing
                    // loads (the first ones may have left lines with sentinels in the L1).
                    load_chunks_cached<KSTEPS>(afrag, hp, lastp);
                    flush_tail();
                    if (!all_written<KSTEPS>(afrag)) {
                        gu = wait_probe(probe, lane < KW / 32, a.abort_word, a.limit_ticks);
                        asm volatile("" ::: "memory");
                        load_chunks<KSTEPS>(afrag, hp, lastp);
                    }
                } else {                                 // (no registers for two attempts: probe first, then the data)
                    gu = wait_probe(probe, lane < KW / 32, a.abort_word, a.limit_ticks);
                    asm volatile("" ::: "memory");
                    load_chunks_cached<KSTEPS>(afrag, hp, lastp);
                }
                if (ensure_written<KSTEPS>(afrag, hp, lastp, gu, a.abort_word, a.limit_ticks)) poison = __builtin_nanf("");
            } else {
                if (wait_counter(cnt + i, (unsigned)(NU * n), a.abort_word, a.limit_ticks)) poison = __builtin_nanf("");
#pragma unroll
                for (int q = 0; q < KSTEPS; ++q)
                    afrag[q] = *reinterpret_cast<const uint4*>(hp + min(q, lastp) * XPAIR);
            }
            if constexpr (LEAN) issue_item(item, axn, cpn);   // (in flight behind the products)
            constexpr int GP = LEAN || (AHEAD && KW > 224) ? 2 : 4;   // gates at a time
            each<0, 4 / GP>([&](auto pass) __attribute__((always_inline)) {
                constexpr int g0 = decltype(pass)::value * GP;
                f32x16_t acc[GP];
#pragma unroll
                for (int g = 0; g < GP; ++g)
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[g][e] = 0.0f;
                each<0, KSTEPS>([&](auto step) __attribute__((always_inline)) {
                    constexpr int q = decltype(step)::value, at = decltype(pass)::value * KSTEPS + q, all = KSTEPS * 4 / GP;
#pragma unroll
                    for (int g = 0; g < GP; ++g) acc[g] = mfma_bf16(afrag[q], bfrag[g0 + g][q], acc[g]);
                    if constexpr (AHEAD) {
                        each<at * SIDE / all, (at + 1) * SIDE / all>([&](auto which) __attribute__((always_inline)) { side(which, n, i, axn, cpn); });
                        __builtin_amdgcn_sched_barrier(0);
                    }
                });
                // partial accumulators -> LDS as [wave][gate][reg/4][lane][reg%4]
#pragma unroll
                for (int g = 0; g < GP; ++g)
#pragma unroll
                    for (int rq = 0; rq < 4; ++rq)
                        l4[((wave * 4 + g0 + g) * 4 + rq) * 64 + lane] =
                            make_float4(acc[g][4 * rq], acc[g][4 * rq + 1], acc[g][4 * rq + 2], acc[g][4 * rq + 3]);
            });
            if constexpr (!AHEAD) { if (SENTINEL) lds_barrier(); else __syncthreads(); }
        } else if constexpr (AHEAD) each<0, SIDE>([&](auto which) __attribute__((always_inline)) { side(which, n, i, axn, cpn); });
        // all partial sums of this thread's rows are read before any is added: the reads then
        // overlap instead of each waiting for its LDS round trip
        static_assert(EPT % 4 == 0, "rows per thread come in groups of four accumulator registers");
        float4 part[NW][4][EPT / 4];
        if constexpr (AHEAD) lds_barrier();
        if (n > 0) {
#pragma unroll
            for (int w2 = 0; w2 < NW; ++w2)
#pragma unroll
                for (int g = 0; g < 4; ++g)
#pragma unroll
                    for (int e4 = 0; e4 < EPT / 4; ++e4) part[w2][g][e4] = l4[((w2 * 4 + g) * 4 + (EPT / 4) * wave + e4) * 64 + lane];
        }
        if constexpr (AHEAD) load_pairs<KSTEPS>(ahead, operand(next_n, next_i), lastp);   // (on either way, so that the wait for the inputs below, which is counted, leaves these loads out)
        if (n > 0) {
#pragma unroll
            for (int w2 = 0; w2 < NW; ++w2)
#pragma unroll
                for (int g = 0; g < 4; ++g)
#pragma unroll
                    for (int e4 = 0; e4 < EPT / 4; ++e4) {
                        const float4 v = part[w2][g][e4];
                        sum[4 * e4][g] += v.x; sum[4 * e4 + 1][g] += v.y; sum[4 * e4 + 2][g] += v.z; sum[4 * e4 + 3][g] += v.w;
                    }
        }
        // (The next item's inputs come from HBM, and a CU's vector memory pipeline returns data in order: issued
        // before the barrier above they would sit in front of another wavefront's loads of the exchanged h and
        // add their latency to the frame-to-frame path.  They are issued below, once h has gone out.)
        if constexpr (!AHEAD) flush_tail();               // at the latest here: the loads issued below may read what it stores
        if constexpr (LEAN) if (n == 0) issue_item(item, axn, cpn);
        float cp[EPT];
#pragma unroll
        for (int e = 0; e < EPT; ++e) cp[e] = (ntl == 1) ? ccarry[e] : AHEAD && n == 0 ? 0.0f : cpl[e];
        if constexpr (!LEAN && !AHEAD) if (item + 1 < nitems) issue_item(item + 1, axn, cpn);   // (registers are short later on)
        // cell arithmetic; h goes out first because it is all the other workgroups wait for
        float gi[EPT], gf[EPT], gg[EPT], go[EPT], cn[EPT], hn[EPT];
        bf16_t* hxb = a.hx + ((size_t)(t * 2 + d) * NT + (b0 >> 5)) * XH;
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            gi[e] = fast_sigmoid((junit ? ax[e][0] : 0.0f) + sum[e][0]);
            gf[e] = fast_sigmoid((junit ? ax[e][1] : 0.0f) + sum[e][1]);
            gg[e] = fast_tanh((junit ? ax[e][2] : 0.0f) + sum[e][2]);
            go[e] = fast_sigmoid((junit ? ax[e][3] : 0.0f) + sum[e][3]);
            cn[e] = next_cell(gf[e], cp[e], gi[e], gg[e]);
            hn[e] = go[e] * fast_tanh(cn[e]) + poison;
        }
        // A lane holds four rows of one unit; both copies of h want the units of a row side by side.  Regrouped
        // through LDS inside the wavefront (as dE/da in the backward kernel), every lane stores four units of one
        // row: one 8-byte store per copy instead of four 2-byte ones.
        static_assert(EPT == 4, "the regrouping below is written for four rows per lane");
        xs[(lh * 2 + 0) * 32 + l32] = (unsigned)coh_bf16(hn[0]) | ((unsigned)coh_bf16(hn[1]) << 16);
        xs[(lh * 2 + 1) * 32 + l32] = (unsigned)coh_bf16(hn[2]) | ((unsigned)coh_bf16(hn[3]) << 16);
        const int xh = lane & 1, xk = (lane >> 1) & 3, xr = (lane >> 3) & 3, xl = lane >> 5;
        uint2 hq;                                         // units 8 xk + 4 xh .. + 3 of row xrow
        {
            const uint4 w = *reinterpret_cast<const uint4*>(xs + (xl * 2 + (xr >> 1)) * 32 + 8 * xk + 4 * xh);
            const unsigned sel = (xr & 1) ? 0x07060302u : 0x05040100u;
            hq = make_uint2(__builtin_amdgcn_perm(w.y, w.x, sel), __builtin_amdgcn_perm(w.w, w.z, sel));
        }
        const int xrow = 2 * EPT * wave + 4 * xl + xr;    // row of the tile
        const bool xok = FULL || b0 + xrow < B;
        const unsigned xcol = (unsigned)(u * 32 + 8 * xk + 4 * xh);
        {
            bf16_t* xp = hxb + ((xcol >> 3) * 256u + (unsigned)xrow * 8u + (xcol & 7u));
            if (SENTINEL) st_coh_8B(xp, hq); else *reinterpret_cast<uint2*>(xp) = hq;
        }
        if constexpr (AHEAD) l4 = reinterpret_cast<float4*>(lds) + (l4 == reinterpret_cast<float4*>(lds) ? NW * 4 * 4 * 64 : 0);   // (no barrier frees the buffer: there are two)
        else if (SENTINEL) lds_barrier();                // frees the LDS buffer for the next item
        else signal_counter(cnt + i);                    // barrier inside: same role
        // row-major outputs (h for the next layer, c and the gates for the backward pass): kept for flush_tail
        tail.t = t; tail.b0 = b0; tail.have = true; tail.xok = xok; tail.hq = hq;
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            tail.cn[e] = cn[e];
            tail.g[e] = make_uint2(pack_bf2(gi[e], gf[e]), pack_bf2(gg[e], go[e]));
        }
        // with one tile per workgroup the next item's previous cell state is the one just computed
#pragma unroll
        for (int e = 0; e < EPT; ++e) ccarry[e] = cn[e];
    };
    if constexpr (LEAN || AHEAD) {
        for (int item = 0; item < nitems; ++item) do_item(item, ax0, cp0, ax0, cp0);
    } else {
        // (the slice of U_h leaves no room for the loop body twice: one body, and a copy at its end)
        for (int item = 0; item < nitems; ++item) {
            do_item(item, ax0, cp0, ax1, cp1);
#pragma unroll
            for (int e = 0; e < EPT; ++e) {
#pragma unroll
                for (int g = 0; g < 4; ++g) ax0[e][g] = ax1[e][g];
                cp0[e] = cp1[e];
            }
        }
    }
    if constexpr (AHEAD) {
        auto last = [&](auto which) __attribute__((always_inline)) { side(which, 0, 0, ax0, cp0); };
        each<0, 1>(last);
        each<EPT * 4 + 2, SIDE>(last);
    } else flush_tail();
    fill_some(1 << 30);                                  // (whatever rounding left over)
}

// ------------------------------------------------------------------------------ backward
template <int KW, bool SENTINEL, bool FULL, bool MULTI, bool PADDED>
__global__ __launch_bounds__(64 * NW) void rec_bwd_kernel(RecBwdArgs a) {
    constexpr int EPT = 16 / NW;
    constexpr int KSTEPS = 4 * KW / 16;                  // the contraction runs over the 4H gate rows
    // The loop body twice, the sets of inputs in turn, and the next ones asked for once dE/da has gone out.  One layer, 4096
    // sequences, us, so / with one body: 288 units 1109 / 1131, 160 592 / 564, 96 336 / 315; wide slices leave no room for two.
    constexpr bool TWO = KW == 96;
    // AHEAD: two slabs of the operand in flight, across the items; one set of inputs, asked for behind the cells.
    constexpr bool AHEAD = MULTI && SENTINEL && KW > 128;
    constexpr int SLABS = KSTEPS / 8, DEEP = 2;
    constexpr bool APART = KW == 160;                    // (see all_written)
    extern __shared__ float lds[];                       // [NW][4][64][4]
    const int H = PADDED ? a.H : NW * KW;                // (the launcher picks KW from a.H)
    const int B = a.B, T = a.T;
    const int NU = PADDED ? (H + 31) / 32 : NW * KW / 32;
    const GroupMap gm = map_block(NU, a.nbg);
    const int d = gm.d, u = gm.u;
    const int lane = threadIdx.x & 63, wave = PADDED || AHEAD ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : threadIdx.x >> 6;
    const int l32 = lane & 31, lh = lane >> 5;
    static_assert(NW == 4, "a wavefront contracts one gate's rows");
    const int ntl = d < 2 ? tiles_in_batch(gm.bg, a.tiles_per_group, B) : 0;   // (d >= 2: a group that does not exist)
    if (ntl == 0) return;

    // U_h^T slice: output unit l32, 8 consecutive gate rows per lane
    uint4 bfrags[1][KSTEPS];
    auto& bfrag = bfrags[0];
    {
        const bf16_t* uht = a.uht[d];
#pragma unroll
        for (int q = 0; q < KSTEPS; ++q) {
            const int unit = u * 32 + l32, k = q * 16 + 8 * lh;
            const bool in = !PADDED || (unit < H && k < H);
            bfrag[q] = in ? *reinterpret_cast<const uint4*>(uht + (size_t)unit * 4 * H + wave * H + k) : make_uint4(0, 0, 0, 0);
        }
    }
    if constexpr (AHEAD) park_all(bfrags);
    unsigned* cnt = a.cnt + (size_t)gm.group * a.tiles_per_group;
    const int j = u * 32 + l32;
    float4* l4 = reinterpret_cast<float4*>(lds);

    // per-thread 32-bit element offsets, added to per-item uniform bases (as in the forward kernel)
    const int rb = 2 * EPT * wave + 4 * lh;              // register e is batch row rb + re(e) of the tile
    auto re = [](int e) { return 8 * (e >> 2) + (e & 3); };
    const bool junit = !PADDED || j < H;
    const unsigned o2c = (unsigned)(d * H + (PADDED ? min(j, H - 1) : j));   // column in the row-major [.][2H] tensor (dy)
    const unsigned o2b = (unsigned)(rb * 2 * H) + o2c;
    const int NT = (B + 31) / 32;
    const int HX = NU * 32;                              // columns of a gate in the exchange copy
    const int XA = 4 * HX / 16 * XPAIR;                  // exchange elements per (frame, direction, tile)
    const int lastp = PADDED ? NU * 2 - 1 : KSTEPS;      // a gate's last pair of chunks
    const unsigned oap = (unsigned)(wave * (HX / 16) * XPAIR + lane * 8);   // this lane's 16 bytes of each chunk pair

    // Saved activations of an item, loaded one item ahead (raw bf16 for the gates and dy).
    // dy of a wavefront's cells is eight rows of 32 units: 512 contiguous-by-row bytes.  With one tile per workgroup
    // 32 lanes fetch it as one 16-byte piece each (dyr) and the wavefront spreads it through LDS at the start of the item
    // (one vector-memory instruction instead of four); with several tiles each lane loads its four values (see the
    // forward kernel's a_x for why).
    constexpr bool WIDE_DY = !MULTI;
    struct Inputs { uint4 g01, g23; bf16_t dy[EPT]; uint4 dyr; float4 c, cp, dcr; };   // g01, g23: (i, f), (g, o) of two cells each as bf16 pairs
    auto issue_inputs = [&](int ni, int i, Inputs& in) {
        const int n = T - 1 - ni;
        const int t = d ? T - 1 - n : n;
        const int tp = d ? T - n : n - 1;
        const int b0 = (gm.bg * a.tiles_per_group + i) * 32;
        const size_t m0 = (size_t)t * B + b0;
        const bf16_t* dyb = a.dy + m0 * 2 * H;
        // the lane's records (see rec_index): gates of its four cells, their cell states, those of the frame visited before
        const size_t r = rec_index(t, d, b0 >> 5, NT, NU, u);
        const uint4* g4 = reinterpret_cast<const uint4*>(a.gates) + r * 2 * 256 + threadIdx.x;
        const uint4 g01 = g4[0], g23 = g4[256];
        float4 c4 = make_float4(0.0f, 0.0f, 0.0f, 0.0f), cp4 = c4, dc4 = c4;
        if constexpr (MULTI) c4 = reinterpret_cast<const float4*>(a.c)[r * 256 + threadIdx.x];   // (one tile: the c of this frame was the item before's c_prev)
        if (AHEAD || n > 0) cp4 = reinterpret_cast<const float4*>(a.c)[rec_index(AHEAD && n == 0 ? t : tp, d, b0 >> 5, NT, NU, u) * 256 + threadIdx.x];
        if (AHEAD || (MULTI && n < T - 1 && ntl > 1)) dc4 = reinterpret_cast<const float4*>(a.dc)[((size_t)(d * NT + (b0 >> 5)) * NU + u) * 256 + threadIdx.x];   // (one tile: carried in registers)
        if constexpr (WIDE_DY) {                         // piece lane % 32: row (lane % 32) / 4 of the wavefront's eight, units 8 (lane % 4) .. + 7
            const int row0 = 2 * EPT * wave + (l32 >> 2), row = FULL ? row0 : min(row0, B - 1 - b0);
            const int col = u * 32 + (l32 & 3) * 8;
            in.dyr = *reinterpret_cast<const uint4*>(dyb + (size_t)row * 2 * H + d * H + (PADDED ? min(col, H - 8) : col));
        }
        static_assert(EPT == 4, "a record holds four cells");
        in.g01 = g01; in.g23 = g23; in.c = c4; in.cp = cp4; in.dcr = dc4;
        if constexpr (!WIDE_DY) {
#pragma unroll
            for (int e = 0; e < EPT; ++e) in.dy[e] = dyb[FULL ? o2b + (unsigned)(re(e) * 2 * H) : (unsigned)(min(rb + re(e), B - 1 - b0) * 2 * H) + o2c];
        }
    };
    auto issue_item = [&](int item, Inputs& in) { const int ni = item / ntl; issue_inputs(ni, item - ni * ntl, in); };

    static_assert(EPT <= 8, "two sets of inputs (this item's and the next one's) must fit in registers");
    const int nitems = T * ntl;
    uint4 ahead[DEEP][8];                                // AHEAD: slabs of the operand on their way
    auto ask = [&](int n0, int i, int sl, uint4 (&to)[8]) __attribute__((always_inline)) {   // slab sl (of the first frame, which has none: of the second)
        const int ni = max(n0, 1);
        const bf16_t* p = a.dax + ((size_t)((d ? ni - 1 : T - ni) * 2 + d) * NT + gm.bg * a.tiles_per_group + i) * XA + wave * (HX / 16) * XPAIR;
        if constexpr (PADDED) load_pairs<8>(to, p + min(sl * 8, lastp) * XPAIR, max(lastp - sl * 8, 0));
        else load_pairs<8>(to, p + sl * 8 * XPAIR, 8);
    };
    Inputs in0, in1;                                     // two sets used in turn, as in the forward kernel
    issue_inputs(0, 0, in0);
    float4 cfirst = make_float4(0.0f, 0.0f, 0.0f, 0.0f);  // (one tile) the c of the first item, later ones are carried
    if constexpr (!MULTI) cfirst = reinterpret_cast<const float4*>(a.c)[rec_index(d ? 0 : T - 1, d, gm.bg, NT, NU, u) * 256 + threadIdx.x];
    __builtin_amdgcn_s_waitcnt(0x0F70);                  // vmcnt(0): see the forward kernel
    // One tile per workgroup: dE/dc of the frame visited before and that frame's c_prev (this frame's c) stay in
    // registers; a wavefront can have 63 vector-memory operations in flight, and an item of this kernel issues about 50.
    float dccarry[EPT], ccarry[EPT];
#pragma unroll
    for (int e = 0; e < EPT; ++e) dccarry[e] = 0.0f;
    ccarry[0] = cfirst.x; ccarry[1] = cfirst.y; ccarry[2] = cfirst.z; ccarry[3] = cfirst.w;
    // NaN once this wave has abandoned a wait, or from the start if the abort word is already raised: added to
    // every dE/da it writes
    float poison = ld_coh_u32(a.abort_word) != 0 ? __builtin_nanf("") : 0.0f;
    int now_n = 0, now_i = 0;                            // frames from the last one, tile of the item
    auto do_item = [&](const int item, const Inputs& cur, Inputs& nxt) __attribute__((always_inline)) {
        const int ni = AHEAD ? now_n : item / ntl, i = AHEAD ? now_i : item - ni * ntl;
        int next_n = 0, next_i = 0;                      // the next item (behind the last one: that one again, not used)
        if constexpr (AHEAD) {
            const bool over = item + 1 == nitems, wraps = i + 1 == ntl;
            next_n = !over && wraps ? ni + 1 : ni; next_i = over ? i : wraps ? 0 : i + 1;
            now_n = next_n; now_i = next_i;
        }
        const int n = T - 1 - ni;
        const int t = d ? T - 1 - n : n;
        const int tn = d ? T - 2 - n : n + 1;            // frame visited after t (its da feeds dh)
        const int b0 = (gm.bg * a.tiles_per_group + i) * 32;
        float dh[EPT];
#pragma unroll
        for (int e = 0; e < EPT; ++e) dh[e] = 0.0f;
        bf16_t dyv[EPT];
        if constexpr (WIDE_DY) {
            bf16_t* dys = reinterpret_cast<bf16_t*>(lds + NW * 4 * 64 * 4 + NW * 512) + wave * 256;   // 512 bytes per wavefront: [row][unit]
            const uint4 dyr = cur.dyr;                    // (read before the branch: read inside it, the compiler keeps both sets of inputs in scratch memory)
            if (lane < 32) reinterpret_cast<uint4*>(dys)[lane] = dyr;
#pragma unroll
            for (int e = 0; e < EPT; ++e) dyv[e] = dys[(4 * lh + e) * 32 + l32];
        } else {
#pragma unroll
            for (int e = 0; e < EPT; ++e) dyv[e] = cur.dy[e];
        }
        if (n < T - 1) {
            const bf16_t* ab = a.dax + ((size_t)(tn * 2 + d) * NT + (b0 >> 5)) * XA;   // uniform: the frame visited before, this tile
            const bf16_t* ap = ab + oap;
            f32x16_t acc;
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[e] = 0.0f;
            if constexpr (AHEAD) {
                bool gu = false;
#pragma unroll
                for (int sl = 0; sl < SLABS; ++sl) {
                    // (spelt out: through wait_written another 2 % of a layer of 768 units)
                    if (!gu && !all_written<8, true>(ahead[sl % DEEP])) gu = look_again<false, 8>(ahead[sl % DEEP], [&]() __attribute__((always_inline)) { ask(ni, i, sl, ahead[sl % DEEP]); }, a.abort_word, a.limit_ticks);
#pragma unroll
                    for (int q = 0; q < 8; ++q) acc = mfma_bf16(ahead[sl % DEEP][q], bfrag[sl * 8 + q], acc);
                    if (sl + DEEP < SLABS) ask(ni, i, sl + DEEP, ahead[sl % DEEP]);
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (gu) poison = __builtin_nanf("");
            } else if (SENTINEL) {
                // the gate rows of this wavefront come from the NU producers: probe each one's last unit,
                // then stream the slabs of 128 gate rows with the next slab's loads in flight
                const bf16_t* probe = ab + xoff(wave * HX + (PADDED ? min(lane, NU - 1) : lane & (4 * KW / 32 - 1)) * 32 + 31, 31);
                uint4 afrag[2][8];
                // first pair of a slab (a slab beyond the layer repeats the last pair), and the last pair counted from it
                auto slab = [&](int sl) { return (PADDED ? min(sl * 8, lastp) : sl * 8) * XPAIR; };
                auto left = [&](int sl) { return PADDED ? max(lastp - sl * 8, 0) : 8; };
                bool gu = false;
                // (straight for the data, the probe only if the first look fails)
                load_chunks_cached<8>(afrag[0], ap, lastp);
                if (!all_written<8, APART>(afrag[0])) {
                    gu = wait_probe(probe, lane < 4 * KW / 32, a.abort_word, a.limit_ticks);
                    asm volatile("" ::: "memory");
                    load_chunks<8>(afrag[0], ap, lastp);
                }
#pragma unroll
                for (int sl = 0; sl < KSTEPS / 8; ++sl) {
                    if (sl + 1 < KSTEPS / 8) load_chunks_cached<8>(afrag[(sl + 1) & 1], ap + slab(sl + 1), left(sl + 1));
                    gu = ensure_written<8, APART>(afrag[sl & 1], ap + slab(sl), left(sl), gu, a.abort_word, a.limit_ticks);
#pragma unroll
                    for (int q = 0; q < 8; ++q) acc = mfma_bf16(afrag[sl & 1][q], bfrag[sl * 8 + q], acc);
                }
                if (gu) poison = __builtin_nanf("");
            } else {
                if (wait_counter(cnt + i, (unsigned)(NU * (T - 1 - n)), a.abort_word, a.limit_ticks)) poison = __builtin_nanf("");
#pragma unroll
                for (int q0 = 0; q0 < KSTEPS; q0 += 8) {
                    uint4 afrag[8];
#pragma unroll
                    for (int q = 0; q < 8; ++q)
                        afrag[q] = *reinterpret_cast<const uint4*>(ap + min(q0 + q, lastp) * XPAIR);
#pragma unroll
                    for (int q = 0; q < 8; ++q) acc = mfma_bf16(afrag[q], bfrag[q0 + q], acc);
                }
            }
#pragma unroll
            for (int rq = 0; rq < 4; ++rq)
                l4[(wave * 4 + rq) * 64 + lane] = make_float4(acc[4 * rq], acc[4 * rq + 1], acc[4 * rq + 2], acc[4 * rq + 3]);
            if constexpr (!AHEAD) { if (SENTINEL) lds_barrier(); else __syncthreads(); }
        }
        if constexpr (AHEAD) {                           // (on either way: see the forward kernel)
            lds_barrier();
#pragma unroll
            for (int sl = 0; sl < DEEP; ++sl) ask(next_n, next_i, sl, ahead[sl]);
        }
        if (n < T - 1) {
            // this thread's rows are EPT/4 whole float4 of each wavefront's partial tile; all are read
            // before any is added so that the LDS round trips overlap
            static_assert(EPT % 4 == 0, "rows per thread come in groups of four accumulator registers");
            float4 part[NW][EPT / 4];
#pragma unroll
            for (int w2 = 0; w2 < NW; ++w2)
#pragma unroll
                for (int e4 = 0; e4 < EPT / 4; ++e4) part[w2][e4] = l4[(w2 * 4 + (EPT / 4) * wave + e4) * 64 + lane];
#pragma unroll
            for (int w2 = 0; w2 < NW; ++w2)
#pragma unroll
                for (int e4 = 0; e4 < EPT / 4; ++e4) {
                    const float4 v = part[w2][e4];
                    dh[4 * e4] += v.x; dh[4 * e4 + 1] += v.y; dh[4 * e4 + 2] += v.z; dh[4 * e4 + 3] += v.w;
                }
        }
        const float curdcr[EPT] = {cur.dcr.x, cur.dcr.y, cur.dcr.z, cur.dcr.w}, curc[EPT] = {cur.c.x, cur.c.y, cur.c.z, cur.c.w};
        const bool none = AHEAD && n == 0;               // (no frame before it)
        const float curcp[EPT] = {none ? 0.0f : cur.cp.x, none ? 0.0f : cur.cp.y, none ? 0.0f : cur.cp.z, none ? 0.0f : cur.cp.w};
        const uint2 curg[EPT] = {make_uint2(cur.g01.x, cur.g01.y), make_uint2(cur.g01.z, cur.g01.w), make_uint2(cur.g23.x, cur.g23.y), make_uint2(cur.g23.z, cur.g23.w)};
        float dcr[EPT];
#pragma unroll
        for (int e = 0; e < EPT; ++e) dcr[e] = (!MULTI || ntl == 1) ? dccarry[e] : AHEAD && n == T - 1 ? 0.0f : curdcr[e];
        float cthis[EPT];
#pragma unroll
        for (int e = 0; e < EPT; ++e) cthis[e] = !MULTI ? ccarry[e] : curc[e];
        if (!TWO && !AHEAD && item + 1 < nitems) issue_item(item + 1, nxt);   // (wide slices: registers are short later on)
        float dcf[EPT];
        unsigned dav[EPT][2];                             // (i, f) and (g, o) as bf16 pairs: kept for the row-major copy below
        bf16_t* dxb = a.dax + ((size_t)(t * 2 + d) * NT + (b0 >> 5)) * XA;
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            const float gi = bf2f((bf16_t)(curg[e].x & 0xFFFFu)), gf = bf2f((bf16_t)(curg[e].x >> 16));
            const float gg = bf2f((bf16_t)(curg[e].y & 0xFFFFu)), go = bf2f((bf16_t)(curg[e].y >> 16));
            const float dht = dh[e] + (junit ? bf2f(dyv[e]) : 0.0f) + poison;
            const float tc = fast_tanh(cthis[e]);
            const float dc = dht * go * (1.0f - tc * tc) + dcr[e];
            const float da_o = dht * tc * go * (1.0f - go);
            const float da_i = dc * gg * gi * (1.0f - gi);
            const float da_f = dc * curcp[e] * gf * (1.0f - gf);
            const float da_g = dc * gi * (1.0f - gg * gg);
            dcf[e] = dc * gf;
            dav[e][0] = (unsigned)coh_bf16(da_i) | ((unsigned)coh_bf16(da_f) << 16);
            dav[e][1] = (unsigned)coh_bf16(da_g) | ((unsigned)coh_bf16(da_o) << 16);
        }
        // A lane holds four rows of one unit; a 16-byte word of either copy of dE/da is eight units of one row.
        // Regrouped through LDS inside the wavefront (its LDS operations execute in order), every lane ends up with
        // the eight units of one (row, pair of gates): two 16-byte stores per copy instead of sixteen 2-byte ones
        // (the memory pipeline takes about as long for a 2-byte store of a wavefront as for a 16-byte one).
        static_assert(EPT == 4, "the regrouping below is written for four rows per lane");
        unsigned* xs = reinterpret_cast<unsigned*>(lds) + NW * 4 * 64 * 4 + wave * 512;
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            xs[((lh * 4 + e) * 2 + 0) * 32 + l32] = dav[e][0];
            xs[((lh * 4 + e) * 2 + 1) * 32 + l32] = dav[e][1];
        }
        const int xk = lane & 3, xq = (lane >> 2) & 1, xr = (lane >> 3) & 3, xl = lane >> 5;
        uint4 cga, cgb;                                   // gate 2 xq and gate 2 xq + 1, units 8 xk .. 8 xk + 7, row xrow
        {
            const uint4* src = reinterpret_cast<const uint4*>(xs + ((xl * 4 + xr) * 2 + xq) * 32 + 8 * xk);
            const uint4 w0 = src[0], w1 = src[1];
            cga = make_uint4(__builtin_amdgcn_perm(w0.y, w0.x, 0x05040100u), __builtin_amdgcn_perm(w0.w, w0.z, 0x05040100u),
                             __builtin_amdgcn_perm(w1.y, w1.x, 0x05040100u), __builtin_amdgcn_perm(w1.w, w1.z, 0x05040100u));
            cgb = make_uint4(__builtin_amdgcn_perm(w0.y, w0.x, 0x07060302u), __builtin_amdgcn_perm(w0.w, w0.z, 0x07060302u),
                             __builtin_amdgcn_perm(w1.y, w1.x, 0x07060302u), __builtin_amdgcn_perm(w1.w, w1.z, 0x07060302u));
        }
        const int xrow = 2 * EPT * wave + 4 * xl + xr;    // row of the tile
        const bool xok = FULL || b0 + xrow < B;
        const unsigned ucol = (unsigned)(u * 32 + 8 * xk);   // first unit; a gate has HX columns in the exchange copy and H row-major
        {
            const unsigned xc = 2 * xq * (unsigned)HX + ucol;
            bf16_t* pa = dxb + ((xc >> 3) * 256u + (unsigned)xrow * 8u);
            bf16_t* pb = dxb + (((xc + (unsigned)HX) >> 3) * 256u + (unsigned)xrow * 8u);
            if (SENTINEL) { st_coh_16B(pa, cga); st_coh_16B(pb, cgb); }
            else { *reinterpret_cast<uint4*>(pa) = cga; *reinterpret_cast<uint4*>(pb) = cgb; }
        }
        if constexpr (AHEAD) {
            asm volatile("" ::: "memory");
            issue_inputs(next_n, next_i, nxt);
        }
        if (TWO && item + 1 < nitems) issue_item(item + 1, nxt);
        if (SENTINEL) lds_barrier();
        else signal_counter(cnt + i);
        // row-major dE/da for the weight- and input-gradient products, and the carried dE/dc
        bf16_t* dab = a.da + ((size_t)t * B + b0) * 8 * H;
        if constexpr (AHEAD) {                           // (every lane issues the stores: see the forward kernel)
            typedef unsigned u4 __attribute__((ext_vector_type(4)));
            const __amdgpu_buffer_rsrc_t p = __builtin_amdgcn_make_buffer_rsrc(dab + d * 4 * H, 0, ((min(B - b0, 32) - 1) * 8 * H + 4 * H) * 2, 0x00020000);
            const int o = !PADDED || ucol < (unsigned)H ? (int)((unsigned)xrow * (unsigned)(8 * H) + (unsigned)(2 * xq * H) + ucol) * 2 : 0x7FFF0000;
            __builtin_amdgcn_raw_buffer_store_b128(u4{cga.x, cga.y, cga.z, cga.w}, p, o, 0, 0);
            __builtin_amdgcn_raw_buffer_store_b128(u4{cgb.x, cgb.y, cgb.z, cgb.w}, p, o + 2 * H, 0, 0);
        } else if (xok && (!PADDED || ucol < (unsigned)H)) {
            bf16_t* pr = dab + ((unsigned)xrow * (unsigned)(8 * H) + (unsigned)(d * 4 * H + 2 * xq * H) + ucol);
            *reinterpret_cast<uint4*>(pr) = cga;
            *reinterpret_cast<uint4*>(pr + H) = cgb;
        }
        if (AHEAD || ntl > 1)                             // carried dE/dc of the lane's four cells: one 16-byte word
            reinterpret_cast<float4*>(a.dc)[((size_t)(d * NT + (b0 >> 5)) * NU + u) * 256 + threadIdx.x] = make_float4(dcf[0], dcf[1], dcf[2], dcf[3]);
        // next item's inputs; with one tile per workgroup its carried dE/dc is the one just computed
#pragma unroll
        for (int e = 0; e < EPT; ++e) { dccarry[e] = dcf[e]; ccarry[e] = curcp[e]; }
    };
    if constexpr (TWO) {
        for (int item = 0; item < nitems; item += 2) {
            do_item(item, in0, in1);
            if (item + 1 < nitems) do_item(item + 1, in1, in0);
        }
    } else {
        for (int item = 0; item < nitems; ++item) {
            do_item(item, in0, AHEAD ? in0 : in1);
            if constexpr (!AHEAD) in0 = in1;
        }
    }
}

// U_h [4H][H] -> U_h^T [H][4H]; blockIdx.z = 2 * layer + direction.
// A wavefront per 64 x 64 elements, a lane per 8 x 8 (H is a multiple of 8): eight 16-byte loads, the 8 x 8 transposed in
// registers, eight 16-byte stores, both sides in whole 128-byte
// pieces.  Bound by the memory; 32 x 32 tiles through LDS in 2-byte accesses took 17.4 us where this takes 9.4 (8 matrices of 512
// cells) and 84 against 38 (12 of 1024).
__global__ __launch_bounds__(256) void transpose_uh_kernel(TransposeUhArgs a, int H) {
    const bf16_t* src = a.src[blockIdx.z];
    bf16_t* dst = a.dst + (size_t)blockIdx.z * 4 * H * H;
    const int lane = threadIdx.x & 63;
    const int r0 = ((int)blockIdx.y * 4 + (int)(threadIdx.x >> 6)) * 64 + (lane >> 3) * 8, c0 = (int)blockIdx.x * 64 + (lane & 7) * 8;
    if (r0 >= 4 * H || c0 >= H) return;                   // rows of U_h (4H), columns (H)
    unsigned x[8][4];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const uint4 v = *reinterpret_cast<const uint4*>(src + (size_t)(r0 + i) * H + c0);
        x[i][0] = v.x; x[i][1] = v.y; x[i][2] = v.z; x[i][3] = v.w;
    }
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        unsigned w[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) w[k] = __builtin_amdgcn_perm(x[2 * k + 1][c >> 1], x[2 * k][c >> 1], c & 1 ? 0x07060302u : 0x05040100u);
        *reinterpret_cast<uint4*>(dst + (size_t)(c0 + c) * 4 * H + r0) = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

// dst[r][0..cols_p) = src[r][0..cols) followed by zeros: one thread per 8-column chunk, grid-stride; and, by all threads, the marking of the
// exchange copies of h.  Two launches of a few us each were mostly their start and end; large ones are bound by the stores.  Apart /
// in one, us: 4 x 512 cells, 8 sequences 9.8 / 5.2, 128 11.5 / 8.7, 2048 67 / 64, 6 x 1024, 512 sequences 48 / 48.
__global__ __launch_bounds__(256) void pad_cols_kernel(PadColsArgs a) {
    const int k = blockIdx.y;
    const unsigned short* src = a.src[k];
    unsigned short* dst = a.dst[k];
    const long long ld = a.ld[k];
    const int cpr = a.cols_p >> 3;
    const long long n = (long long)a.rows[k] * cpr;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
        const long long r = i / cpr;
        const int c = (int)(i - r * cpr) * 8;
        uint4 out;
        const unsigned short* p = src + r * ld + c;
        if (c + 8 <= a.cols && (reinterpret_cast<uintptr_t>(p) & 7) == 0) {      // whole chunk, 8-byte aligned: two loads
            const uint2 lo = *reinterpret_cast<const uint2*>(p), hi = *reinterpret_cast<const uint2*>(p + 4);
            out = make_uint4(lo.x, lo.y, hi.x, hi.y);
        } else {
            unsigned short v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = (c + e < a.cols) ? p[e] : (unsigned short)0;
            out = make_uint4(v[0] | ((unsigned)v[1] << 16), v[2] | ((unsigned)v[3] << 16), v[4] | ((unsigned)v[5] << 16), v[6] | ((unsigned)v[7] << 16));
        }
        *reinterpret_cast<uint4*>(dst + r * a.cols_p + c) = out;
    }
    const size_t stride = (size_t)gridDim.x * gridDim.y * blockDim.x;
    for (size_t i = ((size_t)k * gridDim.x + blockIdx.x) * blockDim.x + threadIdx.x; i < a.fill_words; i += stride) static_cast<uint4*>(a.fill)[i] = make_uint4(~0u, ~0u, ~0u, ~0u);
}

// p[0..n) = v for 16-byte words, grid-stride.
__global__ __launch_bounds__(256) void fill_u128_kernel(uint4* p, size_t n, unsigned v) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    const uint4 w = make_uint4(v, v, v, v);
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = w;
}
__global__ void fill_u32_kernel(unsigned* p, int n, unsigned v) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

template <int KW, bool S, bool FULL, bool MULTI, bool PADDED, bool LEAN = false>
hipError_t run_one(const RecFwdArgs& a, int grid, hipStream_t st, bool* launched) {
    const size_t lds = (size_t)(MULTI && S && !LEAN ? 2 : 1) * NW * 4 * 4 * 64 * 16 + (size_t)NW * 512;   // partial sums; regrouping of h, 512 bytes per wavefront
    return launch_resident<rec_fwd_kernel<KW, S, FULL, MULTI, PADDED, LEAN>>(a, 64 * NW, lds, grid, grid, st, launched);
}
template <int KW, bool S, bool FULL, bool MULTI, bool PADDED>
hipError_t run_one(const RecBwdArgs& a, int grid, hipStream_t st, bool* launched) {
    const size_t lds = (size_t)NW * 4 * 64 * 16 + (size_t)NW * 2048 + (size_t)NW * 512;   // partial sums; regrouping of dE/da, 2 KB per wavefront; spreading dy, 512 bytes per wavefront
    return launch_resident<rec_bwd_kernel<KW, S, FULL, MULTI, PADDED>>(a, 64 * NW, lds, grid, grid, st, launched);
}
template <int KW, bool S, bool FULL, bool PADDED, typename A>
hipError_t run_multi(const A& a, int grid, hipStream_t st, bool* launched) {
    return a.tiles_per_group == 1 ? run_one<KW, S, FULL, false, PADDED>(a, grid, st, launched) : run_one<KW, S, FULL, true, PADDED>(a, grid, st, launched);
}
// Narrow layers of many sequences (see rec_tile_units): the forward kernel with two workgroups per CU.  The backward kernel, whose time
// is the traffic of its operand, gains nothing by that.
template <int KW>
hipError_t run_narrow(const RecFwdArgs& a, hipStream_t st, bool* launched) {
    const int nu = (a.H + 31) / 32, tiles = (a.B + 31) / 32;
    RecFwdArgs b = a;
    b.nbg = rec_groups(a.H, tiles, 2);
    b.tiles_per_group = (tiles + b.nbg - 1) / b.nbg;
    return run_one<KW, true, false, true, true, true>(b, grid_groups(b.nbg) * nu, st, launched);
}
template <int KW>
hipError_t run_narrow(const RecBwdArgs& a, hipStream_t st, bool* launched) {
    return run_one<KW, true, false, true, true>(a, grid_groups(a.nbg) * ((a.H + 31) / 32), st, launched);
}
template <typename A>
hipError_t run_width(const A& a, bool sentinel, hipStream_t st, bool* launched) {
    *launched = false;
    const int grid = grid_groups(a.nbg) * ((a.H + 31) / 32);
    if (a.H == 1024) {
        if (sentinel) return a.B % 32 == 0 ? run_multi<256, true, true, false>(a, grid, st, launched) : run_multi<256, true, false, false>(a, grid, st, launched);
        return a.B % 32 == 0 ? run_multi<256, false, true, false>(a, grid, st, launched) : run_multi<256, false, false, false>(a, grid, st, launched);
    }
    if (!sentinel || !rec_supported(a.H) || (a.H <= 512 && !rec_narrow(a.B, a.H))) return hipSuccess;   // (padded widths: sentinel protocol only)
#define BLSTM_NARROW(KW) if (a.H <= 4 * KW) return run_narrow<KW>(a, st, launched)
    BLSTM_NARROW(32); BLSTM_NARROW(64); BLSTM_NARROW(96);
#undef BLSTM_NARROW
#define BLSTM_PADDED(KW) if (a.H <= 4 * KW) return run_multi<KW, true, false, true>(a, grid, st, launched)
    BLSTM_PADDED(160); BLSTM_PADDED(192); BLSTM_PADDED(224); BLSTM_PADDED(256);
#undef BLSTM_PADDED
    return hipSuccess;
}

}  // namespace

// Supported widths: multiples of 8 up to 1024.  The kernels of this file run those above 512 cells with more sequences than
// recurrent_tile.hip takes there, and some narrow ones (rec_narrow), on four wavefronts that split the contraction (four batch rows per thread in every variant).
// 1024 has kernels of its own; the others run padded to the next multiple of 128 (H = 320, 50 sequences, when these kernels ran
// it: 61 us a layer forward and 66 backward, where launches per frame took 617 and 386).
// Padded widths above 512 only up to 3072 sequences (tests/test_dispatch_cpu.py holds the line there).  One layer, 21 frames, both
// passes' recurrences, us, persistent / launches per frame: H = 576, B = 2048 2104 / 3159, 3072 3193 / 3756, 4096 4488 / 4990, 6144
// 7132 / 6836; H = 768, 3072 3950 / 5215, 4096 5639 / 6222; H = 896, 3072 4445 / 6012: the two cross between 4096 and 6144
// sequences of 576 units by now, and 8 to 16 % is left between 3072 and there.  And not for a single frame, which has no
// recurrence (H = 320, B = 512, two layers forward 46 us against 32).
bool rec_supported(int H) { return H % 8 == 0 && H >= 8 && H <= 1024; }
bool rec_takes(int T, int B, int H) { return rec_supported(H) && (rec_fenced(H) || (T > 1 && (H <= 512 || B <= 3072))); }
bool rec_fenced(int H) { return H == 128 || H == 256 || H == 512 || H == 1024; }
// Batch groups per direction: as many as leave each of the eight XCDs, which get whole groups (map_block), no more than
// per_cu workgroups per CU (of 32).
int rec_groups(int H, int tiles, int per_cu) {
    const int most = 4 * (32 * per_cu / ((H + 31) / 32));
    return tiles < most ? tiles : most;
}
hipError_t launch_fill_u32(unsigned* p, int n, unsigned v, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_u32_kernel, dim3((n + 255) / 256), dim3(256), 0, st, p, n, v);
    return hipGetLastError();
}

hipError_t launch_fill_bytes16(void* p, size_t bytes, unsigned v, hipStream_t st) {
    const size_t n = bytes / 16;
    if (n == 0) return hipSuccess;
    size_t blocks = (n + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(fill_u128_kernel, dim3((unsigned)blocks), dim3(256), 0, st, static_cast<uint4*>(p), n, v);
    return hipGetLastError();
}

hipError_t launch_pad_cols(const PadColsArgs& a, hipStream_t st) {
    if (a.count <= 0) return hipSuccess;
    long long most = 0;
    for (int k = 0; k < a.count; ++k) { const long long n = (long long)a.rows[k] * (a.cols_p / 8); if (n > most) most = n; }
    if (most == 0 && a.fill_words == 0) return hipSuccess;
    const long long fills = (long long)((a.fill_words + 256ull * a.count - 1) / (256ull * a.count));
    long long blocks = (most + 255) / 256 > fills ? (most + 255) / 256 : fills;
    if (blocks > 2048) blocks = 2048;
    hipLaunchKernelGGL(pad_cols_kernel, dim3((unsigned)blocks, (unsigned)a.count), dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_transpose_uh(const TransposeUhArgs& a, int H, hipStream_t st) {
    if (a.count <= 0) return hipSuccess;
    hipLaunchKernelGGL(transpose_uh_kernel, dim3((H + 63) / 64, (4 * H + 255) / 256, a.count), dim3(256), 0, st, a, H);
    return hipGetLastError();
}

hipError_t launch_rec_fwd(const RecFwdArgs& a, bool sentinel, hipStream_t st, bool* launched) { return run_width(a, sentinel, st, launched); }
hipError_t launch_rec_bwd(const RecBwdArgs& a, bool sentinel, hipStream_t st, bool* launched) { return run_width(a, sentinel, st, launched); }

}  // namespace blstm
