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
// last row and are never stored row-major.  No alignment is asked of H: beside the exchange, the rows of U_h and dE/da's row-major stores go in 16-byte pieces where H and
// the weights' address allow it, all else in single floats.  Saved activations are in the row-major layout of the per-frame path (cell.hip).
#include "exchange.hpp"
#include "kernels.hpp"
#include "residency.hpp"
#include <initializer_list>

namespace blstm {
namespace {

constexpr int NWF = 4;                                   // wavefronts, splitting the contraction

constexpr int SC1 = 16;                                  // cache policy of agent-scope accesses

__device__ __forceinline__ unsigned exchange_bits(float v) {
    const unsigned b = __builtin_bit_cast(unsigned, v);
    return b == SENT32 ? 0x7FC00000u : b;
}
__device__ __forceinline__ void st_exchange(float* p, float v) {
    __hip_atomic_store(reinterpret_cast<unsigned*>(p), exchange_bits(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer(const float* p, size_t floats) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), 0, (int)(floats * 4), 0x00020000); }

// Fragments f[q] = the 16 bytes at byte off(q) of a tile of the exchange copy, by ordinary loads (whatever cache answers, a word that
// is not the pattern is final) or past the caches.
template <int AUX, int N, typename F>
__device__ __forceinline__ void look(uint4 (&f)[N], __amdgpu_buffer_rsrc_t r, F off) {
#pragma unroll
    for (int q = 0; q < N; ++q) f[q] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off(q), 0, AUX));
}
// Behind a first look: past the caches until all of it is written.  Returns true if the wait was abandoned.
template <int N, typename F>
__device__ __forceinline__ bool settle(uint4 (&f)[N], __amdgpu_buffer_rsrc_t r, F off, bool gave_up, unsigned* abort_word, unsigned long long limit) {
    return wait_written32<N>(f, [&]() __attribute__((always_inline)) { look<SC1, N>(f, r, off); }, gave_up, abort_word, limit);
}
// With one tile a workgroup the look is timed, so many clocks behind the wavefront's own stores (as in recurrent_small.hip).
__device__ __forceinline__ void pause_until(unsigned long long stored, unsigned clocks) { while (__builtin_amdgcn_s_memtime() - stored < clocks) {} }

template <int CTRL> __device__ __forceinline__ float lane_of_quad(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
// Four neighbouring lanes with four values each: lane k gets value k of each of them, in their order.
__device__ __forceinline__ float4 quad_transpose(const float (&v)[4]) {
    const bool odd = threadIdx.x & 1, high = threadIdx.x & 2;
    const float a = lane_of_quad<0xB1>(odd ? v[0] : v[1]), b = lane_of_quad<0xB1>(odd ? v[2] : v[3]);   // quad_perm 1,0,3,2
    const float p0 = odd ? a : v[0], p1 = odd ? v[1] : a, q0 = odd ? b : v[2], q1 = odd ? v[3] : b;
    const float x = lane_of_quad<0x4E>(high ? p0 : q0), y = lane_of_quad<0x4E>(high ? p1 : q1);          // quad_perm 2,3,0,1
    return high ? make_float4(x, y, q0, q1) : make_float4(p0, p1, x, y);
}

// The slice of U_h.  Forward: row l32 is gate l32 % 4 of unit u8 + l32 / 4, columns 8 q0 + 4 lh and on; four neighbouring ones in a load where they are
// aligned (64 sequences of 512 cells: one by one 7 us a launch longer).  Backward: column `unit` of the rows of a gate, through a buffer, so that the
// addresses are 32-bit sums (by pointers, which the compiler formed one after the other, 34 us a launch longer).
template <int NQ>
__device__ __forceinline__ void load_rows(float (&wf)[NQ][4], const float* uh, int H, int unit, int l32, int lh, int q0) {
    const float* row = uh + ((size_t)(l32 & 3) * H + min(unit, H - 1)) * H;
    if ((H & 3) == 0 && (reinterpret_cast<uintptr_t>(uh) & 15) == 0) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int k = (q0 + q) * 8 + 4 * lh;
            const float4 v = *reinterpret_cast<const float4*>(row + min(k, H - 4));
            const bool in = unit < H && k < H;
            wf[q][0] = in ? v.x : 0.0f; wf[q][1] = in ? v.y : 0.0f; wf[q][2] = in ? v.z : 0.0f; wf[q][3] = in ? v.w : 0.0f;
        }
        return;
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int k = (q0 + q) * 8 + 4 * lh + e;
            const float v = row[min(k, H - 1)];
            wf[q][e] = unit < H && k < H ? v : 0.0f;
        }
}
template <int NQ>
__device__ __forceinline__ void load_columns(float (&wf)[NQ][4], const float* gate, int H, int unit, int lq) {
    const __amdgpu_buffer_rsrc_t rows = buffer(gate, (size_t)H * H);   // (what lies beyond reads as zero)
    const int first = unit < H ? (4 * lq * H + unit) * 4 : 0x70000000;
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) wf[q][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rows, first + (q * 16 + e) * H * 4, 0, 0));
}

// us a launch of 21 frames, a probe of the producers first (the kernels for several tiles, then used for one) / a pause of 300 / 500 / 700 / 900 / 1100
// clocks, forward: 64 sequences of 512 cells 98 / 98 / 90 / 91 / 92 / 94, 20 of 128 41 / 39.8 / 40.8 / 41 / 44 / 44, 20 of 700 134 / 131 / 130 / 126 / 122 / 124;
// backward, 300 / 600 / 800 / 1000 / 1200: 64 of 512 144 / 109 / 87.1 / 87.2 / 87.6 / 89.5, 60 of 256 77 / 73 / 55 / 56 / 58 / 60, 40 of 320 98 / 90 / 70 / 67 / 69 / 70, 20 of
// 128 51 / 41 / 39 / 40 / 41 / 43.
// The more workgroups, the later the operand is there (events, which add about two us, 300 / 400 / 500 / 600, forward: 250 of 128 49.4 / 44.7 / 43.4 / 43.8, 200 of 128 46.2 / 43.1 / 43.5 / 44.1, 8 of 128
// 41.2 / 41.3 / 41.9 / 42.6, 250 of 64 35.9 / 36.4 / 37.3 / 38.0, which leaves 128 cells 400; backward, 500 / 600 / 700 / 800: 250 of 128 58.6 / 44.7 / 44.0 / 44.7, 120 of 32 31.0 / 31.1 / 31.5 / 32.3, 250 of 16
// 30.5 / 30.4 / 30.7 / 31.5, which leaves up to 32 cells 600).
constexpr unsigned fwd_pause(int nq) { return nq <= 2 ? 300 : nq <= 4 ? 400 : nq <= 16 ? 500 : 900; }
constexpr unsigned bwd_pause(int nq) { return nq <= 2 ? 600 : 700; }
constexpr int ONE_MOST = 24;                             // the widest NQ of rec32_fwd_one_kernel

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
// Several tiles a workgroup, and wide layers.  H' = 32 NQ; each wavefront contracts 8 NQ columns.  30 sequences of 1024 cells: 176 us for 21 frames before the
// look was timed and the weights came in 16-byte pieces, 146 so.
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
    load_rows<NQ>(bf, a.uh[d], H, u * 8 + (l32 >> 2), l32, lh, wave * NQ);
    const int NT = (B + 31) / 32;
    auto off = [&](int q) { return (unsigned)(min(wave * NQ + q, nu - 1) * 256 + lane * 4) * 4; };
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
    float poison = ld_coh_u32(a.abort_word) != 0 ? __builtin_nanf("") : 0.0f;
    unsigned long long stored = 0;                       // when the last exchange store went out
    auto do_item = [&](const int item, const In& cur, In& nxt, float (&pt)[NWF][32 * PS]) __attribute__((always_inline)) {
        const int n = item / ntl, i = item - n * ntl;
        const int t = d ? T - 1 - n : n, tp = d ? T - n : n - 1;
        const int tile = pl.bg * a.tiles_per_group + i;
        float4 sum = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (n > 0) {
            const __amdgpu_buffer_rsrc_t x = buffer(a.hx + ((size_t)(tp * 2 + d) * NT + tile) * nu * 256, (size_t)nu * 256);
            uint4 af[NQ];
            if (ntl == 1) pause_until(stored, fwd_pause(NQ));
            look<0, NQ>(af, x, off);
            if (settle<NQ>(af, x, off, false, a.abort_word, a.limit_ticks)) poison = __builtin_nanf("");
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
            lds_barrier();
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
        stored = __builtin_amdgcn_s_memtime();
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
// H' = 16 NQ; wavefront w contracts gate w's H columns of dE/da.  30 sequences of 1024 cells: 236 us for 21 frames with a probe of the producers, 154 so; 150 of 512 (two tiles
// a workgroup) 318 -> 279, which is the loading of the weights.
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
    load_columns<NQ>(bf, a.uh[d] + (size_t)wave * H * H, H, u * 16 + l16, lq);
    const int NT = (B + 15) / 16;
    const size_t XT = (size_t)4 * nu * 256;              // exchange floats of a (frame, direction, tile)
    auto off = [&](int q) { return (unsigned)((wave * nu + min(q, nu - 1)) * 256 + lane * 4) * 4; };
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
    float poison = ld_coh_u32(a.abort_word) != 0 ? __builtin_nanf("") : 0.0f;
    unsigned long long stored = 0;                       // when the last exchange store went out
    auto do_item = [&](const int item, const In& cur, In& nxt, float (&pt)[NWF][16 * PS]) __attribute__((always_inline)) {
        const int ni = item / ntl, i = item - ni * ntl;
        const int n = T - 1 - ni;
        const int t = d ? T - 1 - n : n, tn = d ? T - 2 - n : n + 1;
        const int tile = pl.bg * a.tiles_per_group + i;
        float dh = 0.0f;
        if (ni > 0) {
            const __amdgpu_buffer_rsrc_t x = buffer(a.dax + ((size_t)(tn * 2 + d) * NT + tile) * XT, XT);
            uint4 af[2][SL];
            bool gu = false;
            if (ntl == 1) pause_until(stored, bwd_pause(NQ));
            look<0, SL>(af[0], x, off);
            f32x4_t acc[2];
#pragma unroll
            for (int e = 0; e < 4; ++e) { acc[0][e] = 0.0f; acc[1][e] = 0.0f; }
#pragma unroll
            for (int s = 0; s < NSL; ++s) {
                if (s + 1 < NSL) look<0, SL>(af[(s + 1) & 1], x, [&](int q) { return off((s + 1) * SL + q); });
                gu = settle<SL>(af[s & 1], x, [&](int q) { return off(s * SL + q); }, gu, a.abort_word, a.limit_ticks);
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
            lds_barrier();                          // (one an item: see the forward kernel)
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
        float* xo = a.dax + ((size_t)(t * 2 + d) * NT + tile) * XT + (size_t)u * 256 + (l16 >> 2) * 64 + r * 4 + (l16 & 3);
#pragma unroll
        for (int g = 0; g < 4; ++g) st_exchange(xo + (size_t)g * nu * 256, junit ? da[g] : 0.0f);
        stored = __builtin_amdgcn_s_memtime();
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

// ------------------------------------------------------------------------------ one tile a workgroup
// Layers of up to 768 cells forward and 512 backward (what leaves a wavefront the registers of half a SIMD): four wavefronts compute, four more bring the inputs of four
// frames ahead into LDS and store what the others leave there, so that neither stands in the queue of a computing wavefront (see recurrent_small.hip).  The slice
// is the first operand of the products: a lane has the four gates of a unit, or four units, and the partial sums go through LDS in 16-byte words;
// dE/da leaves in one 16-byte store.  us a launch of 21 frames, forward / backward, with the kernels above as they were and so: 64 sequences of 512 cells
// 98 / 144 and 84 / 87 (3.8 and 3.8 a frame, of which the products are 1.8), 60 of 256 64 / 77 and 52 / 56, 8 of 32 31.4 / 28.8 and 30.4 / 28.4, 20 of 700 forward 136 and 100.
// (With a product and a cell launch a frame 65 and 23 a frame.)
template <int NQ>
__global__ __launch_bounds__(128 * NWF) void rec32_fwd_one_kernel(Rec32FwdArgs a) {
    constexpr int PR = 9;                                // float4 of a row of a partial tile: (i, f, g, o) of eight units, and one to turn the banks
    __shared__ float4 part[2][NWF][32 * PR], axs[2][64 * NWF], gates[2][64 * NWF];
    __shared__ float2 state[2][64 * NWF];                // c, h
    const int T = a.T, B = a.B, H = a.H, nu = a.nu;
    const Place pl = place(nu, a.nbg);
    const int d = pl.d, u = pl.u, tile = pl.bg;
    const int tid = threadIdx.x & (64 * NWF - 1), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // this thread's cell: unit j, row r of the tile
    const int r = tid >> 3, j = u * 8 + (tid & 7);
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
        if (!pl.real) { fill_some(1 << 30); return; }
        const int row = tile * 32 + r;
        const float* ax0 = a.ax + (size_t)min(row, B - 1) * 8 * H + d * 4 * H + min(j, H - 1);
        auto inputs = [&](int n, float4& v) __attribute__((always_inline)) {
            const float* p = ax0 + (size_t)frame(min(n, T - 1)) * B * 8 * H;
            v = make_float4(p[0], p[(size_t)H], p[2 * (size_t)H], p[3 * (size_t)H]);
        };
        auto save = [&](int n) __attribute__((always_inline)) {
            const float4 g4 = gates[n & 1][tid];
            const float2 ch = state[n & 1][tid];
            if (junit && row < B) {
                const size_t m = (size_t)frame(n) * B + row;
                a.y[m * 2 * H + d * H + j] = ch.y;
                if (a.z) a.z[m * 2 * H + d * H + j] = ch.y;
                a.c[m * 2 * H + d * H + j] = ch.x;
                float* g = a.gates + m * 8 * H + (size_t)d * 4 * H + j;
                g[0] = g4.x; g[H] = g4.y; g[2 * (size_t)H] = g4.z; g[3 * (size_t)H] = g4.w;
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
    if (!pl.real) return;
    const int l32 = lane & 31, lh = lane >> 5;
    // row l32 of the slice: gate l32 & 3 of unit l32 >> 2
    float wf[NQ][4];
    load_rows<NQ>(wf, a.uh[d], H, u * 8 + (l32 >> 2), l32, lh, wave * NQ);
    const int NT = (B + 31) / 32;
    auto off = [&](int q) { return (unsigned)(min(wave * NQ + q, nu - 1) * 256 + lane * 4) * 4; };
    auto copy = [&](int n) { return a.hx + ((size_t)(frame(n) * 2 + d) * NT + tile) * nu * 256; };
    const unsigned x_off = (unsigned)u * 256 + ((tid >> 2) & 1) * 128 + r * 4 + (tid & 3);
    float c = 0.0f;
    float poison = ld_coh_u32(a.abort_word) != 0 ? __builtin_nanf("") : 0.0f;
    unsigned long long stored = 0;                       // when the last h went out
    for (int n = 0; n < T; ++n) {
        float4 sum = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (n > 0) {
            const __amdgpu_buffer_rsrc_t x = buffer(copy(n - 1), (size_t)nu * 256);
            uint4 af[NQ];
            pause_until(stored, fwd_pause(NQ));
            look<0, NQ>(af, x, off);
            if (settle<NQ>(af, x, off, false, a.abort_word, a.limit_ticks)) poison = __builtin_nanf("");
            // rows of the products: the slice's gates and units; columns: the tile's rows
            f32x16_t acc;
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[e] = 0.0f;
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wf[q][0], __builtin_bit_cast(float, af[q].x), acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wf[q][1], __builtin_bit_cast(float, af[q].y), acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wf[q][2], __builtin_bit_cast(float, af[q].z), acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wf[q][3], __builtin_bit_cast(float, af[q].w), acc, 0, 0, 0);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) part[n & 1][wave][l32 * PR + 2 * e + lh] = make_float4(acc[4 * e], acc[4 * e + 1], acc[4 * e + 2], acc[4 * e + 3]);
        }
        lds_barrier();                              // one a frame: everything in LDS is there twice
        const float4 ax = axs[n & 1][tid];
        if (n > 0) {
            float4 v[NWF];
#pragma unroll
            for (int w = 0; w < NWF; ++w) v[w] = part[n & 1][w][r * PR + (tid & 7)];
#pragma unroll
            for (int w = 0; w < NWF; ++w) { sum.x += v[w].x; sum.y += v[w].y; sum.z += v[w].z; sum.w += v[w].w; }
        }
        const float gi = sigmoidf_((junit ? ax.x : 0.0f) + sum.x), gf = sigmoidf_((junit ? ax.y : 0.0f) + sum.y);
        const float gg = tanhf_((junit ? ax.z : 0.0f) + sum.z), go = sigmoidf_((junit ? ax.w : 0.0f) + sum.w);
        c = junit ? gf * c + gi * gg : 0.0f;
        const float h = go * tanhf_(c) + poison;
        st_exchange(copy(n) + x_off, h);
        stored = __builtin_amdgcn_s_memtime();
        gates[n & 1][tid] = make_float4(gi, gf, gg, go);
        state[n & 1][tid] = make_float2(c, h);
    }
    lds_barrier();
}

template <int NQ>
__global__ __launch_bounds__(128 * NWF) void rec32_bwd_one_kernel(Rec32BwdArgs a) {
    constexpr int PS = 20;
    constexpr int SL = NQ < 16 ? NQ : NQ < 32 ? 8 : 4, NSL = NQ / SL;  // fragments a slab; two slabs in flight
    static_assert(NQ % SL == 0, "whole slabs");
    __shared__ float part[2][NWF][16 * PS];
    __shared__ float4 gates[2][64 * NWF], out[2][64 * NWF];   // out: dE/da, gate tid % 4 of four units
    __shared__ float2 in_s[2][64 * NWF];                 // dy, the cell state before
    const int T = a.T, B = a.B, H = a.H, nu = a.nu;
    const Place pl = place(nu, a.nbg);
    if (!pl.real) return;
    const int d = pl.d, u = pl.u, tile = pl.bg;
    const int tid = threadIdx.x & (64 * NWF - 1), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, lq = lane >> 4;
    const int r = tid >> 4, j = u * 16 + l16, jc = min(j, H - 1);
    const bool junit = j < H;
    const int row = tile * 16 + r, rc = min(row, B - 1);
    auto frame = [&](int k) { return d ? k : T - 1 - k; };   // (the last one visited forward comes first)
    const float* const c0 = a.c + (size_t)rc * 2 * H + d * H + jc;
    if (wave >= NWF) {
        const float* dy0 = a.dy + (size_t)rc * 2 * H + d * H + jc;
        const float* g0 = a.gates + (size_t)rc * 8 * H + (size_t)d * 4 * H + jc;
        struct In { float4 g; float dy, cp; };
        auto inputs = [&](int k0, In& in) __attribute__((always_inline)) {
            const int k = min(k0, T - 1);
            const size_t m = (size_t)frame(k) * B;
            in.dy = dy0[m * 2 * H];
            const float* g = g0 + m * 8 * H;
            in.g = make_float4(g[0], g[(size_t)H], g[2 * (size_t)H], g[3 * (size_t)H]);
            in.cp = c0[(size_t)frame(min(k + 1, T - 1)) * B * 2 * H];
        };
        const int j4 = u * 16 + (l16 & 12);              // the four units whose gate tid % 4 this thread stores
        float* const da0 = a.da + (size_t)row * 8 * H + (size_t)d * 4 * H + (size_t)(tid & 3) * H + j4;
        auto save = [&](int k) __attribute__((always_inline)) {
            const float4 v = out[k & 1][tid];
            if (row >= B) return;
            float* o = da0 + (size_t)frame(k) * B * 8 * H;
            if ((H & 3) == 0) { if (j4 < H) *reinterpret_cast<float4*>(o) = v; }
            else {
                const float e4[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) if (j4 + e < H) o[e] = e4[e];
            }
        };
        In in[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) inputs(k, in[k]);
        for (int k0 = 0; k0 < T; k0 += 4) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int k = k0 + i;
                if (k >= T) break;
                gates[k & 1][tid] = in[i].g;
                in_s[k & 1][tid] = make_float2(in[i].dy, k < T - 1 ? in[i].cp : 0.0f);   // (the frame visited first forward has no cell state before it)
                lds_barrier();
                inputs(k + 4, in[i]);
                if (k > 0) save(k - 1);
            }
        }
        lds_barrier();
        save(T - 1);
        return;
    }
    // row l16 of the products: unit l16's column of U_h's rows of gate `wave`
    float wf[NQ][4];
    load_columns<NQ>(wf, a.uh[d] + (size_t)wave * H * H, H, u * 16 + l16, lq);
    const int NT = (B + 15) / 16;
    const size_t XT = (size_t)4 * nu * 256;              // exchange floats of a (frame, direction, tile)
    auto off = [&](int q) { return (unsigned)((wave * nu + min(q, nu - 1)) * 256 + lane * 4) * 4; };
    auto copy = [&](int k) { return a.dax + ((size_t)(frame(k) * 2 + d) * NT + tile) * XT; };
    const unsigned x_off = (unsigned)(((tid & 3) * nu + u) * 256 + (l16 >> 2) * 64 + r * 4) * 4;
    float c = c0[(size_t)frame(0) * B * 2 * H], dcn = 0.0f;   // this frame's cell state (then the one before's), carried dE/dc
    float poison = ld_coh_u32(a.abort_word) != 0 ? __builtin_nanf("") : 0.0f;
    unsigned long long stored = 0;                       // when the last dE/da went out
    for (int k = 0; k < T; ++k) {
        float dh = 0.0f;
        if (k > 0) {
            const __amdgpu_buffer_rsrc_t x = buffer(copy(k - 1), XT);
            uint4 af[2][SL];
            bool gu = false;
            f32x4_t acc[2];
#pragma unroll
            for (int e = 0; e < 4; ++e) { acc[0][e] = 0.0f; acc[1][e] = 0.0f; }
            pause_until(stored, bwd_pause(NQ));
            look<0, SL>(af[0], x, off);
#pragma unroll
            for (int s = 0; s < NSL; ++s) {
                if (s + 1 < NSL) look<0, SL>(af[(s + 1) & 1], x, [&](int q) { return off((s + 1) * SL + q); });
                gu = settle<SL>(af[s & 1], x, [&](int q) { return off(s * SL + q); }, gu, a.abort_word, a.limit_ticks);
#pragma unroll
                for (int q = 0; q < SL; ++q) {
                    const uint4 v = af[s & 1][q];
                    acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[s * SL + q][0], __builtin_bit_cast(float, v.x), acc[0], 0, 0, 0);
                    acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[s * SL + q][1], __builtin_bit_cast(float, v.y), acc[1], 0, 0, 0);
                    acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[s * SL + q][2], __builtin_bit_cast(float, v.z), acc[0], 0, 0, 0);
                    acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[s * SL + q][3], __builtin_bit_cast(float, v.w), acc[1], 0, 0, 0);
                }
            }
            if (gu) poison = __builtin_nanf("");
            *reinterpret_cast<float4*>(&part[k & 1][wave][l16 * PS + 4 * lq]) = make_float4(acc[0][0] + acc[1][0], acc[0][1] + acc[1][1], acc[0][2] + acc[1][2], acc[0][3] + acc[1][3]);
        }
        lds_barrier();
        const float4 g = gates[k & 1][tid];
        const float2 in = in_s[k & 1][tid];
        if (k > 0) {
#pragma unroll
            for (int w = 0; w < NWF; ++w) dh += part[k & 1][w][r * PS + l16];
        }
        const float gi = g.x, gf = g.y, gg = g.z, go = g.w, cp = in.y;
        const float dht = in.x + dh + poison;
        const float tc = tanhf_(c);
        const float dc = dht * go * (1.0f - tc * tc) + dcn;
        float da[4];
        da[0] = dc * gg * gi * (1.0f - gi);
        da[1] = dc * cp * gf * (1.0f - gf);
        da[2] = dc * gi * (1.0f - gg * gg);
        da[3] = dht * tc * go * (1.0f - go);
#pragma unroll
        for (int e = 0; e < 4; ++e) da[e] = junit ? da[e] : 0.0f;
        const float4 v = quad_transpose(da);
        typedef unsigned u4 __attribute__((ext_vector_type(4)));
        const __amdgpu_buffer_rsrc_t x = buffer(copy(k), XT);
        __builtin_amdgcn_raw_buffer_store_b128(u4{exchange_bits(v.x), exchange_bits(v.y), exchange_bits(v.z), exchange_bits(v.w)}, x, (int)x_off, 0, SC1);
        stored = __builtin_amdgcn_s_memtime();
        out[k & 1][tid] = v;
        dcn = dc * gf; c = cp;
    }
    lds_barrier();
}

// (the workgroups that pad the grid to whole rounds of the eight XCDs leave at once)
template <auto KERNEL, typename A>
hipError_t run(const A& a, hipStream_t st, bool* launched) {
    const int real = 2 * a.nu * a.nbg;
    return launch_resident<KERNEL>(a, 64 * NWF, 0, (real + 7) & ~7, real, st, launched);
}
template <auto KERNEL, typename A>
hipError_t run_one(const A& a, hipStream_t st, bool* launched) {
    const int real = 2 * a.nu * a.nbg;
    return launch_resident<KERNEL>(a, 128 * NWF, 0, (real + 7) & ~7, real, st, launched);
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
// after the other, each a chain whose length goes with the width the kernel is built for (measured with the kernels for several tiles as they first were, us a tile and frame,
// forward / backward: 2.0 / 1.9 at 64 cells, 2.7 / 2.9 at 256, 3.8 / 4.8 at 512, 5.2 / 6.2 at 768, 6.9 / 7.6 at 1024).  One
// launch per frame: forward the chain of one round of 128x128 tiles, the cells, and the further rounds of tiles; backward
// the launches, the cells, and the product, which is split along K.  With the present kernels, of 168 shapes of 64 to 1024 cells and 96 to 8192
// sequences on both sides of the lines, the estimates pick the slower path by more than 6 % in four forward (1408 of 768 cells 4900 us a frame at a time, 4380 persistent) and in six
// backward: 8192, 6400 of 64 630, 510 persistent, 417, 374 a frame at a time; 3200 of 128 577 / 470; 512 of 512 754 / 676; 320 of 640 700 / 645; 150 of 900 827 a frame at a time, 693 persistent.
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
bool rec32_fwd_one(int B, int H) { return H <= 32 * ONE_MOST && tiles_a_workgroup(B, H, 8, 32) == 1; }
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
#define BLSTM_R32_ONE(NQ) if (a.tiles_per_group == 1 && a.H <= 32 * NQ) return run_one<rec32_fwd_one_kernel<NQ>>(a, st, launched)
    BLSTM_R32_ONE(1); BLSTM_R32_ONE(2); BLSTM_R32_ONE(4); BLSTM_R32_ONE(8); BLSTM_R32_ONE(12); BLSTM_R32_ONE(16); BLSTM_R32_ONE(20); BLSTM_R32_ONE(ONE_MOST);
#undef BLSTM_R32_ONE
    BLSTM_R32(1); BLSTM_R32(2); BLSTM_R32(4); BLSTM_R32(8); BLSTM_R32(12); BLSTM_R32(16); BLSTM_R32(20); BLSTM_R32(24); BLSTM_R32(32);
#undef BLSTM_R32
    return hipSuccess;
}
hipError_t launch_rec32_bwd(Rec32BwdArgs a, hipStream_t st, bool* launched) {
    *launched = false;
    split(a, 16, 16);
#define BLSTM_R32(NQ) if (a.H <= 16 * NQ) return run<rec32_bwd_kernel<NQ>>(a, st, launched)
#define BLSTM_R32_ONE(NQ) if (a.tiles_per_group == 1 && a.H <= 16 * NQ) return run_one<rec32_bwd_one_kernel<NQ>>(a, st, launched)
    BLSTM_R32_ONE(2); BLSTM_R32_ONE(4); BLSTM_R32_ONE(8); BLSTM_R32_ONE(16); BLSTM_R32_ONE(24); BLSTM_R32_ONE(32);
#undef BLSTM_R32_ONE
    BLSTM_R32(2); BLSTM_R32(4); BLSTM_R32(8); BLSTM_R32(16); BLSTM_R32(24); BLSTM_R32(32); BLSTM_R32(40); BLSTM_R32(48); BLSTM_R32(64);
#undef BLSTM_R32
    return hipSuccess;
}

}  // namespace blstm
