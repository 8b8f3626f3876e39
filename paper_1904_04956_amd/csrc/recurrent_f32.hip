// Persistent recurrent kernels in float: all T frames of one layer, both directions, in one launch.
//
// As the bf16 kernels (recurrent.hip), with the split that the float matrix rate asks for: a CU multiplies 32 x 32 x 512
// in 1.9 us, so a workgroup owns only 8 hidden units forward (their 32 gate rows against 32 batch rows, MFMA 32x32x2) and
// 16 units backward (against 16 batch rows, MFMA 16x16x4): 64 sequences of 512 cells are 256 workgroups a frame, one per
// CU.  The workgroup's slice of U_h stays in registers for the whole launch (H/8 and H/4 registers a lane), its four
// wavefronts split the contraction and add their parts through LDS, each thread then does one cell.
// The workgroups of a batch tile exchange h (dE/da) through a copy in the order of the consumers' MFMA fragments, 16
// bytes a lane: [frame][direction][tile][8 columns][2][32 rows][4] forward and [frame][direction][tile][gate][16
// columns][4][16 rows][4] backward, so that a wavefront's load is one contiguous KB and a workgroup's columns of a tile
// are one contiguous KB (a gate).  Protocol: the copy is filled with 0xFFFFFFFF (a NaN that no arithmetic here gives: a
// NaN result is stored as 0x7FC00000) before the launch; producers store write-through at agent scope; consumers load and
// take a word once it is not the pattern.  Each word is written once, so any other value is final.  Waits are bounded and
// failures travel in-band exactly as in the bf16 kernels.
//
// Any H up to 1024: H' = H rounded up to the next built width; weights beyond H are zero, the columns beyond the last
// workgroup's repeat its block (against those zero weights).  Rows of the last tile beyond the batch repeat the batch's
// last row and are never stored row-major.  All global accesses but the exchange are single floats, so no alignment
// is asked of H.  Saved activations are in the row-major layout of the per-frame path (cell.hip).
#include "common.hpp"
#include "kernels.hpp"
#include "residency.hpp"
#include <initializer_list>

namespace blstm {
namespace {

constexpr unsigned SENT32 = 0xFFFFFFFFu;
constexpr int NWF = 4;                                   // wavefronts, splitting the contraction

__device__ __forceinline__ unsigned ld_agent(const unsigned* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void st_exchange(float* p, float v) {
    const unsigned b = __builtin_bit_cast(unsigned, v);
    __hip_atomic_store(reinterpret_cast<unsigned*>(p), b == SENT32 ? 0x7FC00000u : b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint4 ld_exchange(const float* p) {
    const unsigned long long* q = reinterpret_cast<const unsigned long long*>(p);
    const unsigned long long lo = __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned long long hi = __hip_atomic_load(q + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return make_uint4((unsigned)lo, (unsigned)(lo >> 32), (unsigned)hi, (unsigned)(hi >> 32));
}
template <int N>
__device__ __forceinline__ bool written(const uint4 (&f)[N]) {
    unsigned m = 0;
#pragma unroll
    for (int q = 0; q < N; ++q) m = max(max(m, max(f[q].x, f[q].y)), max(f[q].z, f[q].w));
    return __all(m != SENT32);
}
__device__ __forceinline__ void lds_only_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Fragments f[q] = the 16 bytes at base + off(q) floats, first by ordinary loads (whatever cache answers, a word that
// is not the pattern is final).  settle: reloads them past the caches until all are written, or the wait is abandoned.
template <int N, typename F>
__device__ __forceinline__ void fetch(uint4 (&f)[N], const float* base, F off) {
#pragma unroll
    for (int q = 0; q < N; ++q) f[q] = *reinterpret_cast<const uint4*>(base + off(q));
}
template <int N, typename F>
__device__ __forceinline__ bool settle(uint4 (&f)[N], const float* base, F off, bool gave_up, unsigned* abort_word, unsigned long long limit) {
    if (gave_up || written<N>(f)) return gave_up;
    const unsigned long long t0 = wall_clock64();
    for (unsigned it = 1;; ++it) {
        __builtin_amdgcn_s_sleep(1);
#pragma unroll
        for (int q = 0; q < N; ++q) f[q] = ld_exchange(base + off(q));
        if (written<N>(f)) return false;
        if ((it & 31u) == 0) {
            if (ld_agent(abort_word) != 0) return true;
            if (wall_clock64() - t0 > limit) {
                __hip_atomic_store(abort_word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                return true;
            }
        }
    }
}

// Waits until the word at p, one per producing workgroup and lane with `mine` set, is written, before any data is looked at
// (see recurrent_small.hip: with eight or more fragments a wavefront, early looks cost more than the probe).
constexpr int PROBE_FROM = 8;
__device__ __forceinline__ bool probe_producers(const float* p, bool mine, unsigned* abort_word, unsigned long long limit) {
    const unsigned long long t0 = wall_clock64();
    for (unsigned it = 1;; ++it) {
        const unsigned v = mine ? ld_agent(reinterpret_cast<const unsigned*>(p)) : 0u;
        if (__all(v != SENT32)) return false;
        if ((it & 31u) == 0) {
            if (ld_agent(abort_word) != 0) return true;
            if (wall_clock64() - t0 > limit) {
                __hip_atomic_store(abort_word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                return true;
            }
        }
    }
}

// Workgroup -> (direction, group of batch tiles, unit slice).  Ids are dealt round-robin to the eight XCDs; each XCD takes
// a contiguous eighth of the sequence, so that the slices of a group sit on as few XCDs as they fill.
struct Place { int d, bg, u; bool real; };
__device__ __forceinline__ Place place(int nu, int nbg) {
    const int s = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
    Place p;
    p.real = s < 2 * nu * nbg;
    const int group = s / nu;
    p.u = s - group * nu; p.d = group / nbg; p.bg = group - p.d * nbg;
    return p;
}
__device__ __forceinline__ int tiles_of(int bg, int per_group, int rows, int B) {
    const int nt = (B + rows - 1) / rows - bg * per_group;
    return nt < 0 ? 0 : nt < per_group ? nt : per_group;
}

// ------------------------------------------------------------------------------ forward
// H' = 32 NQ; each wavefront contracts 8 NQ columns.  H = 512, 64 sequences: 91 us for 21 frames, 4.3 a frame (with a
// product and a cell launch a frame 65).
template <int NQ>
__global__ __launch_bounds__(64 * NWF, 1) void rec32_fwd_kernel(Rec32FwdArgs a) {
    constexpr int PS = 36;                               // floats per row of the partial tiles
    __shared__ float part[2][NWF][32 * PS];
    const int T = a.T, B = a.B, H = a.H, nu = a.nu;
    const Place pl = place(nu, a.nbg);
    if (!pl.real) return;
    const int d = pl.d, u = pl.u;
    const int ntl = tiles_of(pl.bg, a.tiles_per_group, 32, B);
    if (ntl == 0) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, lh = lane >> 5;

    // column l32 of the slice: gate l32 & 3 of unit l32 >> 2
    float bf[NQ][4];
    {
        const int unit = u * 8 + (l32 >> 2);
        const float* row = a.uh[d] + ((size_t)(l32 & 3) * H + min(unit, H - 1)) * H;
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int k = (wave * NQ + q) * 8 + 4 * lh + e;
                const float v = row[min(k, H - 1)];
                bf[q][e] = unit < H && k < H ? v : 0.0f;
            }
    }
    const int NT = (B + 31) / 32;
    auto off = [&](int q) { return min(wave * NQ + q, nu - 1) * 256 + lane * 4; };
    // this thread's cell: unit j, row r of the tile
    const int r = tid >> 3, j = u * 8 + (tid & 7), jc = min(j, H - 1);
    const bool junit = j < H;
    struct In { float ax[4], cp; };
    auto issue = [&](int item, In& in) {
        const int n = item / ntl, i = item - n * ntl;
        const int t = d ? T - 1 - n : n, tp = d ? T - n : n - 1;
        const int row = (pl.bg * a.tiles_per_group + i) * 32 + r, rc = min(row, B - 1);
        const float* ax = a.ax + ((size_t)t * B + rc) * 8 * H + d * 4 * H + jc;
#pragma unroll
        for (int g = 0; g < 4; ++g) in.ax[g] = ax[(size_t)g * H];
        in.cp = 0.0f;
        if (ntl > 1 && n > 0 && row < B) in.cp = a.c[((size_t)tp * B + row) * 2 * H + d * H + jc];
    };
    const int nitems = T * ntl;
    In in0, in1;                                         // used in turn: an item's inputs load while the one before computes
    issue(0, in0);
    float ccarry = 0.0f;
    float poison = ld_agent(a.abort_word) != 0 ? __builtin_nanf("") : 0.0f;
    auto do_item = [&](const int item, const In& cur, In& nxt, float (&pt)[NWF][32 * PS]) __attribute__((always_inline)) {
        const int n = item / ntl, i = item - n * ntl;
        const int t = d ? T - 1 - n : n, tp = d ? T - n : n - 1;
        const int tile = pl.bg * a.tiles_per_group + i;
        float4 sum = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (n > 0) {
            const float* base = a.hx + ((size_t)(tp * 2 + d) * NT + tile) * nu * 256;
            uint4 af[NQ];
            bool gu = false;
            if constexpr (NQ >= PROBE_FROM) {            // lane q: the last word of the wavefront's pair q
                if (ntl == 1) gu = probe_producers(base + min(wave * NQ + lane, nu - 1) * 256 + 255, lane < NQ, a.abort_word, a.limit_ticks);
                asm volatile("" ::: "memory");
            }
            fetch<NQ>(af, base, off);
            if (settle<NQ>(af, base, off, gu, a.abort_word, a.limit_ticks)) poison = __builtin_nanf("");
            f32x16_t acc;
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[e] = 0.0f;
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__builtin_bit_cast(float, af[q].x), bf[q][0], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__builtin_bit_cast(float, af[q].y), bf[q][1], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__builtin_bit_cast(float, af[q].z), bf[q][2], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__builtin_bit_cast(float, af[q].w), bf[q][3], acc, 0, 0, 0);
            }
#pragma unroll
            for (int e = 0; e < 16; ++e) pt[wave][(8 * (e >> 2) + 4 * lh + (e & 3)) * PS + l32] = acc[e];
            // one barrier an item: the partial tiles are double-buffered, and every wavefront has read an item's before it
            // reaches the next item's barrier
            lds_only_barrier();
#pragma unroll
            for (int w = 0; w < NWF; ++w) {
                const float4 v = *reinterpret_cast<const float4*>(&pt[w][r * PS + 4 * (tid & 7)]);
                sum.x += v.x; sum.y += v.y; sum.z += v.z; sum.w += v.w;
            }
        }
        const float cp = ntl == 1 ? ccarry : cur.cp;
        const float gi = sigmoidf_((junit ? cur.ax[0] : 0.0f) + sum.x), gf = sigmoidf_((junit ? cur.ax[1] : 0.0f) + sum.y);
        const float gg = tanhf_((junit ? cur.ax[2] : 0.0f) + sum.z), go = sigmoidf_((junit ? cur.ax[3] : 0.0f) + sum.w);
        const float c = junit ? gf * cp + gi * gg : 0.0f;
        const float h = go * tanhf_(c) + poison;
        st_exchange(a.hx + (((size_t)(t * 2 + d) * NT + tile) * nu + u) * 256 + ((tid >> 2) & 1) * 128 + r * 4 + (tid & 3), h);
        if (item + 1 < nitems) issue(item + 1, nxt);
        ccarry = c;
        const int row = tile * 32 + r;
        if (junit && row < B) {
            const size_t m = (size_t)t * B + row;
            a.y[m * 2 * H + d * H + j] = h;
            a.c[m * 2 * H + d * H + j] = c;
            float* g = a.gates + m * 8 * H + (size_t)d * 4 * H + j;
            g[0] = gi; g[H] = gf; g[2 * (size_t)H] = gg; g[3 * (size_t)H] = go;
        }
    };
    for (int item = 0; item < nitems; item += 2) {
        do_item(item, in0, in1, part[0]);
        if (item + 1 < nitems) do_item(item + 1, in1, in0, part[1]);
    }
}

// ------------------------------------------------------------------------------ backward
// H' = 16 NQ; wavefront w contracts gate w's H columns of dE/da.  H = 512, 64 sequences: 160 us for 21 frames, 7.6 a
// frame (with a product and a cell launch a frame 23).
template <int NQ>
__global__ __launch_bounds__(64 * NWF, 1) void rec32_bwd_kernel(Rec32BwdArgs a) {
    constexpr int PS = 20;
    constexpr int SL = NQ < 16 ? NQ : NQ >= 64 ? 4 : NQ % 16 == 0 && NQ < 48 ? 16 : 8, NSL = NQ / SL; // fragments a slab; two slabs in flight (the widest slices leave registers for eight or four each)
    static_assert(NQ % SL == 0, "whole slabs");
    __shared__ float part[2][NWF][16 * PS];
    const int T = a.T, B = a.B, H = a.H, nu = a.nu;
    const Place pl = place(nu, a.nbg);
    if (!pl.real) return;
    const int d = pl.d, u = pl.u;
    const int ntl = tiles_of(pl.bg, a.tiles_per_group, 16, B);
    if (ntl == 0) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, lq = lane >> 4;

    // column l16 of U_h's rows of gate `wave`
    float bf[NQ][4];
    {
        const int unit = u * 16 + l16;
        const float* col = a.uh[d] + (size_t)wave * H * H + min(unit, H - 1);
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int k = q * 16 + 4 * lq + e;
                const float v = col[(size_t)min(k, H - 1) * H];
                bf[q][e] = unit < H && k < H ? v : 0.0f;
            }
    }
    const int NT = (B + 15) / 16;
    const size_t XT = (size_t)4 * nu * 256;              // exchange floats of a (frame, direction, tile)
    auto off = [&](int q) { return (wave * nu + min(q, nu - 1)) * 256 + lane * 4; };
    const int r = tid >> 4, j = u * 16 + l16, jc = min(j, H - 1);
    const bool junit = j < H;
    struct In { float dy, g[4], c, cp, dc; };
    auto issue = [&](int item, In& in) {
        const int ni = item / ntl, i = item - ni * ntl;
        const int n = T - 1 - ni;
        const int t = d ? T - 1 - n : n, tp = d ? T - n : n - 1;
        const int row = (pl.bg * a.tiles_per_group + i) * 16 + r, rc = min(row, B - 1);
        const size_t m = (size_t)t * B + rc;
        in.dy = a.dy[m * 2 * H + d * H + jc];
        const float* g = a.gates + m * 8 * H + (size_t)d * 4 * H + jc;
#pragma unroll
        for (int k = 0; k < 4; ++k) in.g[k] = g[(size_t)k * H];
        in.c = a.c[m * 2 * H + d * H + jc];
        in.cp = 0.0f;
        if (n > 0) in.cp = a.c[((size_t)tp * B + rc) * 2 * H + d * H + jc];
        in.dc = 0.0f;
        if (ntl > 1 && ni > 0 && row < B) in.dc = a.dc[((size_t)d * B + row) * H + jc];
    };
    const int nitems = T * ntl;
    In in0, in1;
    issue(0, in0);
    float dccarry = 0.0f;
    float poison = ld_agent(a.abort_word) != 0 ? __builtin_nanf("") : 0.0f;
    auto do_item = [&](const int item, const In& cur, In& nxt, float (&pt)[NWF][16 * PS]) __attribute__((always_inline)) {
        const int ni = item / ntl, i = item - ni * ntl;
        const int n = T - 1 - ni;
        const int t = d ? T - 1 - n : n, tn = d ? T - 2 - n : n + 1;
        const int tile = pl.bg * a.tiles_per_group + i;
        float dh = 0.0f;
        if (ni > 0) {
            const float* base = a.dax + ((size_t)(tn * 2 + d) * NT + tile) * XT;
            uint4 af[2][SL];
            bool gu = false;
            if constexpr (NQ >= PROBE_FROM) {            // lane q: the last word of the gate's block q
                if (ntl == 1) gu = probe_producers(base + (wave * nu + min(lane, nu - 1)) * 256 + 255, lane < NQ, a.abort_word, a.limit_ticks);
                asm volatile("" ::: "memory");
            }
            fetch<SL>(af[0], base, off);
            f32x4_t acc[2];
#pragma unroll
            for (int e = 0; e < 4; ++e) { acc[0][e] = 0.0f; acc[1][e] = 0.0f; }
#pragma unroll
            for (int s = 0; s < NSL; ++s) {
                if (s + 1 < NSL) fetch<SL>(af[(s + 1) & 1], base, [&](int q) { return off((s + 1) * SL + q); });
                gu = settle<SL>(af[s & 1], base, [&](int q) { return off(s * SL + q); }, gu, a.abort_word, a.limit_ticks);
#pragma unroll
                for (int q = 0; q < SL; ++q) {
                    const uint4 v = af[s & 1][q];
                    acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(float, v.x), bf[s * SL + q][0], acc[0], 0, 0, 0);
                    acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(float, v.y), bf[s * SL + q][1], acc[1], 0, 0, 0);
                    acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(float, v.z), bf[s * SL + q][2], acc[0], 0, 0, 0);
                    acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(float, v.w), bf[s * SL + q][3], acc[1], 0, 0, 0);
                }
            }
            if (gu) poison = __builtin_nanf("");
#pragma unroll
            for (int e = 0; e < 4; ++e) pt[wave][(4 * lq + e) * PS + l16] = acc[0][e] + acc[1][e];
            lds_only_barrier();                          // (one an item: see the forward kernel)
#pragma unroll
            for (int w = 0; w < NWF; ++w) dh += pt[w][r * PS + l16];
        }
        const float gi = cur.g[0], gf = cur.g[1], gg = cur.g[2], go = cur.g[3];
        const float dht = cur.dy + dh + poison;
        const float tc = tanhf_(cur.c);
        const float dc = dht * go * (1.0f - tc * tc) + (ntl == 1 ? dccarry : cur.dc);
        float da[4];
        da[0] = dc * gg * gi * (1.0f - gi);
        da[1] = dc * cur.cp * gf * (1.0f - gf);
        da[2] = dc * gi * (1.0f - gg * gg);
        da[3] = dht * tc * go * (1.0f - go);
        float* x = a.dax + ((size_t)(t * 2 + d) * NT + tile) * XT + (size_t)u * 256 + (l16 >> 2) * 64 + r * 4 + (l16 & 3);
#pragma unroll
        for (int g = 0; g < 4; ++g) st_exchange(x + (size_t)g * nu * 256, junit ? da[g] : 0.0f);
        if (item + 1 < nitems) issue(item + 1, nxt);
        dccarry = dc * gf;
        const int row = tile * 16 + r;
        if (junit && row < B) {
            float* o = a.da + ((size_t)t * B + row) * 8 * H + (size_t)d * 4 * H + j;
#pragma unroll
            for (int g = 0; g < 4; ++g) o[(size_t)g * H] = da[g];
            if (ntl > 1) a.dc[((size_t)d * B + row) * H + j] = dccarry;
        }
    };
    for (int item = 0; item < nitems; item += 2) {
        do_item(item, in0, in1, part[0]);
        if (item + 1 < nitems) do_item(item + 1, in1, in0, part[1]);
    }
}

// (the workgroups that pad the grid to whole rounds of the eight XCDs leave at once)
template <auto KERNEL, typename A>
hipError_t run(const A& a, hipStream_t st, bool* launched) {
    const int real = 2 * a.nu * a.nbg;
    return launch_resident<KERNEL>(a, 64 * NWF, 0, (real + 7) & ~7, real, st, launched);
}

// Unit slices of `units` for H, and the batch groups that leave every XCD no more than one workgroup per CU.
template <typename A>
void split(A& a, int units, int rows) {
    a.nu = (a.H + units - 1) / units;
    const int tiles = (a.B + rows - 1) / rows, most = 256 / (2 * a.nu);
    a.nbg = tiles < most ? tiles : most;
    a.tiles_per_group = (tiles + a.nbg - 1) / a.nbg;
}

}  // namespace

// Which of the two paths is the faster, by estimates of what a frame takes (us).  Persistent: the tiles a workgroup walks one
// after the other, each a chain whose length goes with the width the kernel is built for (measured, us a tile and frame,
// forward / backward: 2.0 / 1.9 at 64 cells, 2.7 / 2.9 at 256, 3.8 / 4.8 at 512, 5.2 / 6.2 at 768, 6.9 / 7.6 at 1024).  One
// launch per frame: forward the chain of one round of 128x128 tiles, the cells, and the further rounds of tiles; backward
// the launches, the cells, and the product, which is split along K.  Of 194 shapes of 64 to 1024 cells and 96 to 8192
// sequences the estimates pick the slower path by more than 6 % in two forward (worst 12 %) and in six backward (12 %).
// (A line at B H^2 = 650e6 and 180e6 did so in 15 and 28, worst 55 and 34 %: 1408 sequences of 576 cells forward
// 4266 us persistent, 3063 with launches per frame.)
namespace {
int tiles_a_workgroup(int B, int H, int units, int rows) {
    Rec32FwdArgs a{};
    a.B = B; a.H = H;
    split(a, units, rows);
    return a.tiles_per_group;
}
// The built width for H (see launch_rec32_*): `unit` times the least of the built NQ.
int built_width(int H, int unit, std::initializer_list<int> nqs) {
    for (int nq : nqs) if (H <= unit * nq) return unit * nq;
    return 0;
}
}  // namespace
bool rec32_fwd_supported(int B, int H) {
    if (H > 1024) return false;
    const double persistent = tiles_a_workgroup(B, H, 8, 32) * (1.5 + 0.0049 * built_width(H, 32, {1, 2, 4, 8, 12, 16, 20, 24, 32}));
    const long long tiles = 2LL * ((B + 127) / 128) * ((4 * H + 127) / 128);
    const double per_frame = 32 + 0.0645 * H + 5e-5 * (double)B * H + 0.055 * H * (double)((tiles + 255) / 256 - 1);
    return persistent <= per_frame;
}
bool rec32_bwd_supported(int B, int H) {
    if (!rec32_fwd_supported(B, H)) return false;        // (its workspace is part of the forward kernel's)
    const double persistent = tiles_a_workgroup(B, H, 16, 16) * (1.4 + 0.0063 * built_width(H, 16, {2, 4, 8, 16, 24, 32, 40, 48, 64}));
    const double cells = (double)B * H, per_frame = 20 + 15e-6 * cells + 0.115e-6 * cells * H;
    return persistent <= per_frame;
}
size_t rec32_hx_bytes(int T, int B, int H) { return (size_t)T * 2 * ((B + 31) / 32) * ((H + 7) / 8) * 1024; }
size_t rec32_dax_bytes(int T, int B, int H) { return (size_t)T * 2 * ((B + 15) / 16) * ((H + 15) / 16) * 4096; }

hipError_t launch_rec32_fwd(Rec32FwdArgs a, hipStream_t st, bool* launched) {
    *launched = false;
    split(a, 8, 32);
#define BLSTM_R32(NQ) if (a.H <= 32 * NQ) return run<rec32_fwd_kernel<NQ>>(a, st, launched)
    BLSTM_R32(1); BLSTM_R32(2); BLSTM_R32(4); BLSTM_R32(8); BLSTM_R32(12); BLSTM_R32(16); BLSTM_R32(20); BLSTM_R32(24); BLSTM_R32(32);
#undef BLSTM_R32
    return hipSuccess;
}
hipError_t launch_rec32_bwd(Rec32BwdArgs a, hipStream_t st, bool* launched) {
    *launched = false;
    split(a, 16, 16);
#define BLSTM_R32(NQ) if (a.H <= 16 * NQ) return run<rec32_bwd_kernel<NQ>>(a, st, launched)
    BLSTM_R32(2); BLSTM_R32(4); BLSTM_R32(8); BLSTM_R32(16); BLSTM_R32(24); BLSTM_R32(32); BLSTM_R32(40); BLSTM_R32(48); BLSTM_R32(64);
#undef BLSTM_R32
    return hipSuccess;
}

}  // namespace blstm
