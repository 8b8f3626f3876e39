// Persistent recurrent kernels (bf16) for few sequences: all T frames of one layer, both directions, in one launch.
//
// The kernels of recurrent.hip give a workgroup 32 units of 32 rows; with few batch tiles most CUs have none, and a frame
// is a chain of latencies whose length is the work of one workgroup.  Here a workgroup has 16 units of 16 rows (MFMA
// 16x16x32) and a tile of its own for the whole launch: a quarter of the products, the partial sums, the cells (one
// per thread) and, backward, half of the operand bytes a frame.  Used while the workgroups fit the device at once.
//
// Four wavefronts split the contraction (forward: a quarter of h each; backward: one gate's rows of dE/da each), their
// slices of U_h (U_h^T) stay in registers.  Exchange copies in the order of the fragments: [frame][direction][16-row
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

constexpr int NWF = 4;
constexpr int PAIR = 4 * 16 * 8;                         // elements of 32 columns of a tile (1 KB)
constexpr int PS = 20;                                   // floats per row of a partial tile

// Lane 2 q + i probes the last two elements that slice i of block q writes.
constexpr int LAST_OF_SLICE = 128 + 15 * 8 + 6;

// The value of four neighbouring lanes (units 4k .. 4k + 3 of one row) as four bf16, in the first of them.
__device__ __forceinline__ uint2 quad_bf16(float v) {
    const unsigned own = coh_bf16(v);
    const unsigned one = __builtin_amdgcn_update_dpp(0u, own, 0xB1, 0xF, 0xF, true);       // quad_perm 1,0,3,2
    const unsigned two = own | (one << 16);                                                // (in even lanes)
    return make_uint2(two, __builtin_amdgcn_update_dpp(0u, two, 0x4E, 0xF, 0xF, true));    // quad_perm 2,3,0,1
}

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

// ------------------------------------------------------------------------------ forward
// Width up to 128 NQ; each wavefront contracts 32 NQ columns.
template <int NQ>
__global__ __launch_bounds__(64 * NWF, 2) void rec_small_fwd_kernel(RecFwdArgs a) {
    __shared__ float part[2][NWF][4][16 * PS];
    const int T = a.T, B = a.B, H = a.H;
    const int blocks = (H + 31) / 32, nu = 2 * blocks, NT = (B + 15) / 16;
    // this workgroup's share of the region to fill, some words every frame behind its stores
    const unsigned long long share = a.fill ? (a.fill_words + gridDim.x - 1) / gridDim.x : 0ull;
    const unsigned long long first = min(a.fill_words, (unsigned long long)blockIdx.x * share);
    uint4* const fill = static_cast<uint4*>(a.fill) + first;
    const unsigned fill_end = (unsigned)(min(a.fill_words, first + share) - first);
    unsigned fill_pos = threadIdx.x;
    const int fill_each = (int)((share + (unsigned long long)(256 * T) - 1) / (unsigned long long)(256 * T));
    auto fill_some = [&](int words) { for (int k = 0; k < words && fill_pos < fill_end; ++k, fill_pos += 256) fill[fill_pos] = make_uint4(~0u, ~0u, ~0u, ~0u); };
    const Spot sp = spot(nu, NT);
    if (!sp.real) { fill_some(1 << 30); return; }
    const int d = sp.d, u = sp.u, tile = sp.tile;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, lq = lane >> 4;
    uint4 bf[4][NQ];
    {
        const int unit = u * 16 + l16;
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const int k = (wave * NQ + q) * 32 + 8 * lq;
                bf[g][q] = unit < H && k < H ? *reinterpret_cast<const uint4*>(a.uh[d] + (size_t)(g * H + unit) * H + k) : make_uint4(0u, 0u, 0u, 0u);
            }
    }
    auto off = [&](int q) { return min(wave * NQ + q, blocks - 1) * PAIR + lane * 8; };
    // this thread's cell: unit j, row r of the tile
    const int r = tid >> 4, j = u * 16 + l16;
    const bool junit = j < H;
    const int row = tile * 16 + r, rc = min(row, B - 1);
    const float* ax0 = a.ax + (size_t)rc * 8 * H + d * 4 * H + min(j, H - 1);
    const size_t axt = (size_t)B * 8 * H;
    float ax[4], axn[4];
    auto inputs = [&](int n, float (&v)[4]) {
        const float* p = ax0 + (size_t)(d ? T - 1 - n : n) * axt;
#pragma unroll
        for (int g = 0; g < 4; ++g) v[g] = p[(size_t)g * H];
    };
    inputs(0, ax);
    float c = 0.0f;
    float poison = ld_coh_u32(a.abort_word) != 0 ? __builtin_nanf("") : 0.0f;
    auto frame = [&](const int n, const float (&ax)[4], float (&axn)[4], float (&pt)[NWF][4][16 * PS]) __attribute__((always_inline)) {
        const int t = d ? T - 1 - n : n, tp = d ? T - n : n - 1;
        float sum[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if (n > 0) {
            const bf16_t* base = a.hx + ((size_t)(tp * 2 + d) * NT + tile) * blocks * PAIR;
            uint4 af[NQ];
            bool gu = false;
            if constexpr (NQ >= PROBE_FROM) {
                gu = probe_producers16(base + min(wave * NQ + (lane >> 1), blocks - 1) * PAIR + (lane & 1) * 256 + LAST_OF_SLICE, lane < 2 * NQ, a.abort_word, a.limit_ticks);
                asm volatile("" ::: "memory");
            }
            look16<NQ>(af, base, off);
            if (settle16<NQ>(af, base, off, gu, a.abort_word, a.limit_ticks)) poison = __builtin_nanf("");
            f32x4_t acc[4];
#pragma unroll
            for (int g = 0; g < 4; ++g)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[g][e] = 0.0f;
#pragma unroll
            for (int q = 0; q < NQ; ++q)
#pragma unroll
                for (int g = 0; g < 4; ++g) acc[g] = mfma16(af[q], bf[g][q], acc[g]);
#pragma unroll
            for (int g = 0; g < 4; ++g)
#pragma unroll
                for (int e = 0; e < 4; ++e) pt[wave][g][(4 * lq + e) * PS + l16] = acc[g][e];
            lds_barrier();                               // one a frame: the partial tiles are double-buffered
            float v[NWF][4];
#pragma unroll
            for (int w = 0; w < NWF; ++w)
#pragma unroll
                for (int g = 0; g < 4; ++g) v[w][g] = pt[w][g][r * PS + l16];
#pragma unroll
            for (int w = 0; w < NWF; ++w)
#pragma unroll
                for (int g = 0; g < 4; ++g) sum[g] += v[w][g];
        }
        const float gi = fast_sigmoid((junit ? ax[0] : 0.0f) + sum[0]), gf = fast_sigmoid((junit ? ax[1] : 0.0f) + sum[1]);
        const float gg = fast_tanh((junit ? ax[2] : 0.0f) + sum[2]), go = fast_sigmoid((junit ? ax[3] : 0.0f) + sum[3]);
        c = next_cell(gf, c, gi, gg);
        const float h = go * fast_tanh(c) + poison;
        const uint2 hq = quad_bf16(h);
        const size_t rec = ((size_t)(t * 2 + d) * NT + tile) * nu + u;
        if ((tid & 3) == 0)
            st_coh_8B(a.hx + (((size_t)(t * 2 + d) * NT + tile) * blocks + (u >> 1)) * PAIR + ((2 * (u & 1) + (l16 >> 3)) * 16 + r) * 8 + (l16 & 7), hq);
        if (n + 1 < T) inputs(n + 1, axn);
        reinterpret_cast<uint2*>(a.gates)[rec * 256 + tid] = make_uint2(pack_bf2(gi, gf), pack_bf2(gg, go));
        a.c[rec * 256 + tid] = c;
        if ((tid & 3) == 0 && junit && row < B) *reinterpret_cast<uint2*>(a.y + ((size_t)t * B + row) * 2 * H + d * H + j) = hq;
        fill_some(fill_each);
    };
    for (int n = 0; n < T; n += 2) {
        frame(n, ax, axn, part[0]);
        if (n + 1 < T) frame(n + 1, axn, ax, part[1]);
    }
    fill_some(1 << 30);
}

// ------------------------------------------------------------------------------ backward
// Width up to 32 NQ; wavefront w contracts gate w's columns of dE/da.
// NEAR: groups found on one XCD exchange through its L2 (xcd.hpp).  They can be where the contiguous eighths are whole groups: eight groups
// of at most 32 slices, 385 to 512 cells and 49 to 64 sequences (64 of 512 cells 53.5 -> 49.5 us a layer; 50 of 320 43.0 -> 44.0, so not there).
// Elsewhere the answer would be no, and the question takes half a microsecond.
// Else, from 385 cells on, the probe of the producers right behind the wavefront's own stores comes too early: it waits PAUSE x 64 clocks.  us a layer,
// PAUSE 0 / 1 / 2 / 3: 8 sequences of 512 cells 48 / 48 / 47 / 47, 32 46 / 46 / 46 / 46, 33 53 / 51 / 48 / 47; 0 / 2 / 4 / 6: 15 of 1024 71 / 69 / 67 / 67, 30 78 / 76 / 72 / 69,
// 20 of 640 56 / 53 / 51 / 51, 1 of 768 59 / 57 / 55 / 56.
template <int NQ, bool NEAR>
__global__ __launch_bounds__(64 * NWF, NQ <= 16 ? 2 : 1) void rec_small_bwd_kernel(RecBwdArgs a) {
    __shared__ float part[2][NWF][16 * PS];
    const int T = a.T, B = a.B, H = a.H;
    const int blocks = (H + 31) / 32, nu = 2 * blocks, NT = (B + 15) / 16;
    const Spot sp = spot(nu, NT);
    if (!sp.real) return;
    const int d = sp.d, u = sp.u, tile = sp.tile;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int PAUSE = NEAR || NQ < 16 ? 0 : NQ == 16 ? 2 : 4;
    unsigned* const xcds = NEAR && a.xcd ? a.xcd + sp.group * nu : nullptr;
    tell_xcd(xcds, u);
    const int l16 = lane & 15, lq = lane >> 4;
    uint4 bf[NQ];
    {
        const int unit = u * 16 + l16;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int k = q * 32 + 8 * lq;
            bf[q] = unit < H && k < H ? *reinterpret_cast<const uint4*>(a.uht[d] + (size_t)unit * 4 * H + wave * H + k) : make_uint4(0u, 0u, 0u, 0u);
        }
    }
    auto off = [&](int q) { return (wave * blocks + min(q, blocks - 1)) * PAIR + lane * 8; };
    const int r = tid >> 4, j = u * 16 + l16;
    const bool junit = j < H;
    const int row = tile * 16 + r, rc = min(row, B - 1);
    const bf16_t* dy0 = a.dy + (size_t)rc * 2 * H + d * H + min(j, H - 1);
    struct In { bf16_t dy; uint2 g; float cp; };
    auto record = [&](int t) { return (((size_t)(t * 2 + d) * NT + tile) * nu + u) * 256 + tid; };
    auto inputs = [&](int n, In& in) {                   // n = visited frame
        const int t = d ? T - 1 - n : n, tp = d ? T - n : n - 1;
        in.dy = dy0[(size_t)t * B * 2 * H];
        in.g = reinterpret_cast<const uint2*>(a.gates)[record(t)];
        in.cp = 0.0f;
        if (n > 0) in.cp = a.c[record(tp)];
    };
    In in0, in1;
    inputs(T - 1, in0);
    float c = a.c[record(d ? 0 : T - 1)], dcn = 0.0f;    // this frame's cell state (then the one before's), carried dE/dc
    float poison = ld_coh_u32(a.abort_word) != 0 ? __builtin_nanf("") : 0.0f;
    bool lost;
    const bool near = one_xcd(xcds, nu, a.abort_word, a.limit_ticks, &lost);
    if (lost) poison = __builtin_nanf("");
    const size_t XT = (size_t)4 * blocks * PAIR;
    auto frame = [&](const int n, const In& cur, In& nxt, float (&pt)[NWF][16 * PS]) __attribute__((always_inline)) {
        const int t = d ? T - 1 - n : n, tn = d ? T - 2 - n : n + 1;
        float dh = 0.0f;
        if (n < T - 1) {
            const bf16_t* base = a.dax + ((size_t)(tn * 2 + d) * NT + tile) * XT;
            uint4 af[NQ];
            bool gu = false;
            if constexpr (PAUSE > 0) __builtin_amdgcn_s_sleep(PAUSE);
            if constexpr (NQ >= PROBE_FROM) {
                gu = probe_producers16(base + (wave * blocks + min(lane >> 1, blocks - 1)) * PAIR + (lane & 1) * 256 + LAST_OF_SLICE, lane < 2 * NQ, a.abort_word, a.limit_ticks);
                asm volatile("" ::: "memory");
            }
            look16<NQ>(af, base, off);
            if (settle16<NQ>(af, base, off, gu, a.abort_word, a.limit_ticks)) poison = __builtin_nanf("");
            f32x4_t acc[2];
#pragma unroll
            for (int e = 0; e < 4; ++e) { acc[0][e] = 0.0f; acc[1][e] = 0.0f; }
#pragma unroll
            for (int q = 0; q < NQ; ++q) acc[q & 1] = mfma16(af[q], bf[q], acc[q & 1]);
#pragma unroll
            for (int e = 0; e < 4; ++e) pt[wave][(4 * lq + e) * PS + l16] = acc[0][e] + acc[1][e];
            lds_barrier();
#pragma unroll
            for (int w = 0; w < NWF; ++w) dh += pt[w][r * PS + l16];
        }
        const float gi = bf2f((bf16_t)(cur.g.x & 0xFFFFu)), gf = bf2f((bf16_t)(cur.g.x >> 16));
        const float gg = bf2f((bf16_t)(cur.g.y & 0xFFFFu)), go = bf2f((bf16_t)(cur.g.y >> 16));
        const float dht = dh + (junit ? bf2f(cur.dy) : 0.0f) + poison;
        const float tc = fast_tanh(c);
        const float dc = dht * go * (1.0f - tc * tc) + dcn;
        const uint2 qi = quad_bf16(dc * gg * gi * (1.0f - gi)), qf = quad_bf16(dc * cur.cp * gf * (1.0f - gf));
        const uint2 qg = quad_bf16(dc * gi * (1.0f - gg * gg)), qo = quad_bf16(dht * tc * go * (1.0f - go));
        if ((tid & 3) == 0) {
            bf16_t* x = a.dax + ((size_t)(t * 2 + d) * NT + tile) * XT + (size_t)(u >> 1) * PAIR + ((2 * (u & 1) + (l16 >> 3)) * 16 + r) * 8 + (l16 & 7);
            const size_t gs = (size_t)blocks * PAIR;
            st_exchange(near, x, qi); st_exchange(near, x + gs, qf); st_exchange(near, x + 2 * gs, qg); st_exchange(near, x + 3 * gs, qo);
        }
        if (n > 0) inputs(n - 1, nxt);
        dcn = dc * gf; c = cur.cp;
        if ((tid & 3) == 0 && junit && row < B) {
            bf16_t* o = a.da + ((size_t)t * B + row) * 8 * H + (size_t)d * 4 * H + j;
            *reinterpret_cast<uint2*>(o) = qi; *reinterpret_cast<uint2*>(o + H) = qf;
            *reinterpret_cast<uint2*>(o + 2 * (size_t)H) = qg; *reinterpret_cast<uint2*>(o + 3 * (size_t)H) = qo;
        }
    };
    for (int n = T - 1; n >= 0; n -= 2) {
        frame(n, in0, in1, part[0]);
        if (n > 0) frame(n - 1, in1, in0, part[1]);
    }
}

template <auto KERNEL, typename A>
hipError_t run(const A& a, hipStream_t st, bool* launched) {
    const int real = 2 * 2 * ((a.H + 31) / 32) * ((a.B + 15) / 16);
    return launch_resident<KERNEL>(a, 64 * NWF, 0, (real + 7) & ~7, real, st, launched);
}
template <int NQ>
hipError_t run_bwd(const RecBwdArgs& a, hipStream_t st, bool* launched) {
    if constexpr (NQ == 16) if ((a.B + 15) / 16 == 4) return run<rec_small_bwd_kernel<NQ, true>>(a, st, launched);   // (eight groups)
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
#define BLSTM_SMALL(NQ) if (a.H <= 128 * NQ) return run<rec_small_fwd_kernel<NQ>>(a, st, launched)
    BLSTM_SMALL(1); BLSTM_SMALL(2); BLSTM_SMALL(3); BLSTM_SMALL(4); BLSTM_SMALL(5); BLSTM_SMALL(6); BLSTM_SMALL(7); BLSTM_SMALL(8);
#undef BLSTM_SMALL
    return hipSuccess;
}
hipError_t launch_rec_small_bwd(const RecBwdArgs& a, hipStream_t st, bool* launched) {
    *launched = false;
#define BLSTM_SMALL(NQ) if (a.H <= 32 * NQ) return run_bwd<NQ>(a, st, launched)
    BLSTM_SMALL(4); BLSTM_SMALL(8); BLSTM_SMALL(12); BLSTM_SMALL(16); BLSTM_SMALL(20); BLSTM_SMALL(24); BLSTM_SMALL(28); BLSTM_SMALL(32);
#undef BLSTM_SMALL
    return hipSuccess;
}

}  // namespace blstm
