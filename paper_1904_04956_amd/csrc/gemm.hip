// What runs a product: tile, parts of K and edge treatment by shape, and the launches of the bf16 kernels of gemm_tile.hpp.
#include "gemm_tile.hpp"

namespace blstm {
namespace {

inline bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

template <typename TI>
int fast_flags(const void* p, long long ld, long long stride, int batch, bool rowfast) {
    const long long es = sizeof(TI);
    if (batch <= 1) stride = 0;
    int f = 0;
    if (!rowfast) {
        if (aligned(p, 16) && (ld * es) % 16 == 0 && (stride * es) % 16 == 0) f |= 1;
        if (es == 2 && aligned(p, 8) && (ld * es) % 8 == 0 && (stride * es) % 8 == 0) f |= 2;
    } else {
        const long long w = 4 * es;                       // four consecutive rows per load
        if (aligned(p, w) && (ld * es) % w == 0 && (stride * es) % w == 0) f |= 1;
        if (es == 2 && aligned(p, 16) && (ld * es) % 16 == 0 && (stride * es) % 16 == 0) f |= 4;   // eight rows per load
    }
    return f;
}

// ---- direct-mode kernels: bf16 operands, unguarded, forms X W^T, dA W and dA^T X -------------------------------
// variant 0: 128x128 tile, two LDS buffers, two workgroups per CU; 1: 128x128, three buffers (dA^T X, launches of at most one
// workgroup per CU); 2: 256x128 tile, one buffer, fragments in registers, two workgroups per CU; 3: 256x256 tile on
// eight wavefronts, two buffers, one workgroup per CU (the dA W form only: the softmax layer's input gradient).  X W^T and
// dA W also 4: 64x64, three buffers, three workgroups per CU; 5: 128x64, three buffers, two; 6: 128x128, one buffer, three.
template <typename TO, bool AT, bool BT, bool RS, int MODE>
hipError_t launch_direct_rs(const Params& P, int variant, dim3 grid, hipStream_t stream) {
    if (variant == 2) return launch_kernel<bf16_t, TO, AT, BT, 4, 2, 2, MODE, RS, 1>(P, grid, stream);
    if constexpr (!AT && BT && !RS) {
        if (variant == 3) return launch_kernel<bf16_t, TO, AT, BT, 4, 2, 4, MODE, false, 2>(P, grid, stream);
    }
    if constexpr (!AT) {
        if (variant == 4) return launch_kernel<bf16_t, TO, AT, BT, 1, 1, 2, MODE, false, 3>(P, grid, stream);
        if (variant == 5) return launch_kernel<bf16_t, TO, AT, BT, 2, 1, 2, MODE, false, 3>(P, grid, stream);
        if (variant == 6) return launch_kernel<bf16_t, TO, AT, BT, 2, 2, 2, MODE, false, 1>(P, grid, stream);
    }
    if (variant >= 3) return hipErrorInvalidValue;
    if constexpr (AT && BT) {
        if (variant == 1) return launch_kernel<bf16_t, TO, AT, BT, 2, 2, 2, MODE, RS, 3>(P, grid, stream);
    }
    return launch_kernel<bf16_t, TO, AT, BT, 2, 2, 2, MODE, RS, 2>(P, grid, stream);
}
template <typename TO, int MODE>
hipError_t launch_direct_mode(const GemmDesc& d, const Params& P, int variant, dim3 grid, hipStream_t stream) {
    if (d.atrans && d.btrans) {
        if constexpr (sizeof(TO) == 4) {                      // (row sums go with the float weight gradients)
            if (P.rowsum) return launch_direct_rs<TO, true, true, true, MODE>(P, variant, grid, stream);
        }
        if (P.rowsum) return hipErrorInvalidValue;
        return launch_direct_rs<TO, true, true, false, MODE>(P, variant, grid, stream);
    }
    if (P.rowsum) return hipErrorInvalidValue;
    if (!d.atrans && d.btrans) return launch_direct_rs<TO, false, true, false, MODE>(P, variant, grid, stream);
    if (!d.atrans && !d.btrans) return launch_direct_rs<TO, false, false, false, MODE>(P, variant, grid, stream);
    return hipErrorInvalidValue;
}
template <typename TO>
hipError_t launch_direct(const GemmDesc& d, const Params& P, int mode, int variant, dim3 grid, hipStream_t stream) {
    return mode == WHOLE ? launch_direct_mode<TO, WHOLE>(d, P, variant, grid, stream) : launch_direct_mode<TO, EDGE>(d, P, variant, grid, stream);
}

// ---- X W^T with a contraction of up to four slabs and many rows (the logits) ------------------------------------------
// A tile of such a product is over before its loads' latency and its output are: 5376 x 32000, K = 256 took 142 us where products
// alone take 75 and the output 60.  Here a workgroup keeps one column tile's weights in registers for the whole contraction
// (2 x 4 NK fragments a wavefront) and walks down the rows: only X is loaded, straight into a ring of four slabs that runs
// on across the tiles, half of the operand bytes a tile.  The weights are the first operand of the products, so that a lane
// has four neighbouring columns of one row; an exchange between the lane halves makes them eight, and the output leaves
// from registers in 16-byte stores that nothing waits for.  K = 256, N = 32000, in the
// step, us, 256x128 or one-buffer 128x128 tiles against this: 2688 rows 82 / 66, 3633 114 / 85, 5376 144 / 117, 10752 280 / 218.
// Rows and columns beyond the matrix repeat the last ones and are dropped by the stores' range check, so that every wavefront
// issues the same number of vector-memory instructions for every tile: the waits below count on it.
template <int NK>
__global__ __launch_bounds__(256, 2) void gemm_resident_kernel(Params P, int parts) {
    constexpr int SLAB = 128 * CHUNKS, BK = 64, NL = 4, NSTORE = 8;   // 16-byte words of a slab; loads a wavefront and slab, stores a wavefront and tile
    extern __shared__ uint4 smem[];                     // [4][SLAB], then the 128 columns' bias
    float* bias_s = reinterpret_cast<float*>(smem + 4 * SLAB);
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wv >> 1, wn = wv & 1, l32 = lane & 31, half = lane >> 5;
    const int ct = (int)blockIdx.x % P.ntn, part = (int)blockIdx.x / P.ntn;
    const int ntiles = (P.ntm - part + parts - 1) / parts;   // row tiles part, part + parts, ..: all workgroups go down the rows together
    if (ntiles <= 0) return;
    const int col0 = ct * 128;
    const bf16_t* A = static_cast<const bf16_t*>(P.A[0].p);
    const bf16_t* W = static_cast<const bf16_t*>(P.B[0].p);
    const long long lda = P.A[0].ld, ldb = P.B[0].ld;
    uint4 wf[2][4 * NK];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int q = 0; q < 4 * NK; ++q)
            wf[j][q] = *reinterpret_cast<const uint4*>(W + (long long)min(col0 + wn * 64 + j * 32 + l32, P.N - 1) * ldb + (2 * q + half) * 8);
    if (tid < 128) bias_s[tid] = P.bias && col0 + tid < P.N ? ld_f(static_cast<const bf16_t*>(P.bias) + col0 + tid) : 0.0f;
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");

    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) void*)smem;
    const int total = ntiles * NK;
    // slab s of this workgroup's sequence (the last one again beyond its end) into its slot; lane l of load j fetches the chunk that
    // belongs at word 64 (4 j + wv) + l of the swizzled layout
    auto issue = [&](int s) __attribute__((always_inline)) {
        const int sc = min(s, total - 1), it = sc / NK, row0 = (part + it * parts) * 128;
        const char* base = reinterpret_cast<const char*>(A + (long long)row0 * lda + (sc - it * NK) * BK);
        const unsigned slot = lds0 + (unsigned)((s & 3) * SLAB * 16);
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            const int r = 8 * (4 * j + wv) + (lane >> 3);
            const unsigned voff = (unsigned)(min(r, P.M - 1 - row0) * (int)lda * 2 + (((lane & 7) ^ swz(r)) << 4));
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" :: "s"(__builtin_amdgcn_readfirstlane(slot + (unsigned)((4 * j + wv) * 1024))), "v"(voff), "s"(base) : "memory");
        }
    };
    const int arow = wm * 64 + l32;
    int roff[CHUNKS / 2];
#pragma unroll
    for (int q = 0; q < CHUNKS / 2; ++q) roff[q] = arow * CHUNKS + ((2 * q + half) ^ swz(arow));
    for (int s = 0; s < 3; ++s) issue(s);
    for (int it = 0; it < ntiles; ++it) {
        f32x16_t acc[2][2];                             // [columns][rows]
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[j][i][e] = 0.0f;
#pragma unroll
        for (int q = 0; q < NK; ++q) {
            const int s = it * NK + q;
            // Younger than slab s's loads: those of two slabs, and the stores of the tiles that ended in the three slabs since
            // (in the first three slabs: of none, or of some, and waiting for fewer is only longer).
            int ended = 0;
#pragma unroll
            for (int j = 1; j <= 3; ++j) ended += (q - j + 3 * NK) % NK == NK - 1 ? 1 : 0;
            if (s < 3 || ended == 0) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(2 * NL) : "memory");
            else if (ended == 1) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(2 * NL + NSTORE) : "memory");
            else if (ended == 2) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(2 * NL + 2 * NSTORE) : "memory");
            else asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(2 * NL + 3 * NSTORE) : "memory");
            issue(s + 3);                               // (into the slot of slab s - 1, which every wavefront is done with)
            const uint4* a_s = smem + (s & 3) * SLAB;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint4 x[2] = {a_s[roff[k]], a_s[roff[k ^ 2] + 32 * CHUNKS]};
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int i = 0; i < 2; ++i)
                        acc[j][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, wf[j][4 * q + k]), __builtin_bit_cast(bf16x8_t, x[i]), acc[j][i], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        // register e of a lane: row l32 of C's block i, column 8 (e / 4) + 4 half + e % 4 of block j
        const int row0 = (part + it * parts) * 128;
        const __amdgpu_buffer_rsrc_t out = __builtin_amdgcn_make_buffer_rsrc(static_cast<bf16_t*>(P.C) + (long long)row0 * P.ldc, 0, min(P.M - row0, 128) * (int)P.ldc * 2, 0x00020000);
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int g = 0; g < 4; g += 2) {
                const int c = wn * 64 + j * 32 + 8 * g + 4 * half, n = col0 + wn * 64 + j * 32 + 8 * (g + half);
                const float4 b0 = *reinterpret_cast<const float4*>(bias_s + c), b1 = *reinterpret_cast<const float4*>(bias_s + c + 8);
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const f32x16_t& v = acc[j][i];
                    const unsigned x0 = pack_bf2(v[4 * g] + b0.x, v[4 * g + 1] + b0.y), x1 = pack_bf2(v[4 * g + 2] + b0.z, v[4 * g + 3] + b0.w);
                    const unsigned y0 = pack_bf2(v[4 * g + 4] + b1.x, v[4 * g + 5] + b1.y), y1 = pack_bf2(v[4 * g + 6] + b1.z, v[4 * g + 7] + b1.w);
                    const auto s0 = __builtin_amdgcn_permlane32_swap(x0, y0, false, false), s1 = __builtin_amdgcn_permlane32_swap(x1, y1, false, false);
                    const u32x4_t word = {s0[0], s1[0], s0[1], s1[1]};
                    const int off = n < P.Nst ? (wm * 64 + i * 32 + l32) * (int)P.ldc * 2 + n * 2 : -16;
                    __builtin_amdgcn_raw_buffer_store_b128(word, out, off, 0, 0);
                }
            }
        __builtin_amdgcn_sched_barrier(0);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");    // (the loads beyond the end)
}
template <int NK>
hipError_t launch_resident_nk(const Params& P, int parts, hipStream_t stream) {
    constexpr size_t lds = 4 * 128 * CHUNKS * 16 + 128 * sizeof(float);
    static thread_local bool attr_set = false;
    hipError_t e = allow_lds(&gemm_resident_kernel<NK>, lds, &attr_set);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((gemm_resident_kernel<NK>), dim3((unsigned)(P.ntn * parts)), dim3(256), lds, stream, P, parts);
    return hipGetLastError();
}

inline bool direct_form(const GemmDesc& d) { return !d.add && !(d.atrans && !d.btrans); }

// How the kernel of this tile shape runs the product.  Both unguarded forms need loads of the widest kind, per-thread
// offsets in 32 bits and (two segments) common leading dimensions.  WHOLE: only whole tiles and slabs.  EDGE, direct: any M,
// N and K whose 16-byte groups lie in memory: a row-fast operand's rows come in whole groups or it is padded to them; so does a
// k-fast operand's contraction, unless it is a padded A and B is row-fast (whose k-rows beyond the end are replaced by
// zeros).  EDGE, staged (X W^T, float operands, one segment or whole slabs of the first): any K.
// Measured: the products of the paper-shaped step at 173 sequences 1.72 ms guarded, 0.82 ms EDGE.
template <typename TI>
int run_mode(const GemmDesc& d, const Params& P, int tile_m, int tile_n, bool direct) {
    constexpr int VEC = Vec<TI>::N, bk = CHUNKS * VEC;
    const int Ne = d.Npad > 0 ? d.Npad : d.N;
    bool whole = d.M % tile_m == 0 && Ne % tile_n == 0;
    for (int s = 0; s < d.nseg; ++s) {
        if (!(P.A[s].fast & 1) || !(P.B[s].fast & 1)) return GUARDED;
        if (sizeof(TI) == 2 && ((d.atrans && !(P.A[s].fast & 4)) || (d.btrans && !(P.B[s].fast & 4)))) return GUARDED;
        if (d.seg[s].lda != d.seg[0].lda || d.seg[s].ldb != d.seg[0].ldb) return GUARDED;
        if (d.seg[s].lda * (long long)sizeof(TI) * 64 > 0x3FFFFFFF || d.seg[s].ldb * (long long)sizeof(TI) * 64 > 0x3FFFFFFF) return GUARDED;
        if (d.seg[s].K % bk) whole = false;
    }
    const bool loops = direct || (!d.atrans && !d.btrans);   // (of the staged forms X W^T alone has unguarded loops)
    if (!loops) return GUARDED;
    if (whole) return WHOLE;
    if ((d.atrans && d.M % VEC && !d.a_pad) || (d.btrans && d.N % VEC && d.Npad == 0)) return GUARDED;
    if (!direct) return sizeof(TI) == 4 && (d.nseg == 1 || d.seg[0].K % bk == 0) ? EDGE : GUARDED;     // (only the very last slab may be a part)
    for (int s = 0; s < d.nseg; ++s) {
        if (d.seg[s].K % VEC == 0) continue;
        if (!d.atrans && !(d.a_pad && d.btrans)) return GUARDED;
        if (!d.btrans) return GUARDED;
    }
    return EDGE;
}

constexpr int kTileM[7] = {128, 256, 256, 64, 128, 128, 128}, kTileN[7] = {128, 256, 128, 64, 64, 128, 128};
constexpr int kDirectVariant[6] = {0, 3, 2, 4, 5, 6};     // of launch_direct (0 and 1: by GemmPlan::deep)

GemmPlan make_plan(const GemmDesc& d, bool allow_r);

// Parts of the rows for gemm_resident_kernel, or 0 where it does not pay: two workgroups per CU walk one part of a column tile
// each, and loading its weights takes a workgroup about as long as one and a half tiles.  Not beyond 1 GiB of output, most
// of which has left the last-level cache when the row kernel comes to it: 43008 x 32000 986 to 1020 us here and 1130 to 1150 in the
// row kernel behind it, 1033 to 1146 and 1033 to 1046 with 256x128 tiles.
int resident_parts(const GemmDesc& d) {
    const int batch = d.batch > 0 ? d.batch : 1;
    if (!(d.in_type == DT_BF16 && d.out_type == DT_BF16 && !d.atrans && !d.btrans && d.nseg == 1 && batch == 1 && !d.add && !d.rowsum && d.Npad == 0 && d.N >= 8 && d.ldc <= 1 << 22)) return 0;
    if (d.seg[0].K < 64 || d.seg[0].K > 256 || d.seg[0].K % 64 || (long long)d.M * d.N > 1ll << 29) return 0;
    const int ntm = (d.M + 127) / 128, ntn = (d.N + 127) / 128;
    int parts = 0;
    double best = 1.6 * ntm * ntn / 512.0;
    for (int p = 1; p <= 512 && p * 5 <= ntm; ++p) {
        const double t = (double)(((long long)ntn * p + 511) / 512) * ((ntm + p - 1) / p + 1.5);
        if (t < best) { best = t; parts = p; }
    }
    return parts;
}

template <typename TI>
Params make_params(const GemmDesc& d) {
    Params P{};
    P.nseg = d.nseg;
    for (int s = 0; s < d.nseg; ++s) {
        const GemmSeg& g = d.seg[s];
        P.A[s] = Operand{g.A, g.lda, d.M, fast_flags<TI>(g.A, g.lda, g.sA, d.batch, d.atrans)};
        P.B[s] = Operand{g.B, g.ldb, d.N, fast_flags<TI>(g.B, g.ldb, g.sB, d.batch, d.btrans)};
        P.K[s] = g.K; P.sA[s] = g.sA; P.sB[s] = g.sB;
    }
    P.C = d.C; P.ldc = d.ldc; P.sC = d.sC;
    P.bias = d.bias; P.sBias = d.sBias;
    P.add = d.add; P.ldadd = d.ldadd; P.sAdd = d.sAdd;
    P.rowsum = d.rowsum; P.sRowsum = d.sRowsum;
    P.M = d.M; P.N = d.N;
    P.splits = 1;
    return P;
}
// Tile rows of a band.  Bands only order the tiles, and the figures are those of whole launches, us, bands of 4 / 8.
// bf16, X W^T (both directions in a launch; N, K of each): fewer rows, of which an XCD's workgroups then share columns too, gain while there are not many bands, 2688 x 2048, K = 1024
// 35 / 40 (2304, 1152 40 / 45), 5376 x 2048 55 / 58, 10752 x 4096, K = 2048 278 / 287, 16128 x 2048, K = 1024 148 / 153; beyond, eight read the right operand half as often, 21504 x 2048, K = 1024 208 / 199,
// K = 264 116 / 109, x 1280, K = 640 100 / 99, 31500 x 2176, K = 1088 351 / 326, x 2560, K = 1280 462 / 447, x 3328, K = 1664 720 / 698, unless it is large, x 3584, K = 1792 817 / 826, 43008 x 32000, K = 256
// 1114 / 1181, or has many columns for its size (63420 x 8918, K = 256: a step 2446 / 2494).
// dA W (N; K = 4 N): four up to 5376 rows, 2688 x 1152 52 / 55, 2688 x 1280 63 / 66, 5376 x 640 34 / 35, 5376 x 1024 to 1920 within 1 %; eight beyond, 10752 x 1024 121 / 119, 10752 x 1408 184 / 178,
// 14700 x 1280 247 / 237, 14700 x 2048 435 / 420, 21504 x 1024 153 / 147 (10752 x 1536 181 / 184, 31500 x 1664 and wider 1 to 3 % the other way); from 43008 rows on they are the same, and a step
// with eight is the slower (2048 sequences of 512 cells 11598 / 11636, 3000 9952 / 9996), as is one of
// few columns and a long contraction (24864 x 363, K = 32000, in a step of 6062 / 6116).
// dA^T X, the grouped weight gradients (M = 4 H; layers, features of the first): four, as for 5376 frames of 4 layers of 512 cells 288 / 312, of 320 167 / 172, 14700 of 4 of 1024 2346 / 2450, 31500 of 2 of 160, 320
// 242 / 261, but not for ten to twelve tile rows and as many tile columns (by measurement; the traffic of four should be the less there too): 6300 frames of 2 of 640, 1280 343 / 316, 14700 840 / 750, 5376 of 2 of 704, 1408
// 317 / 299, of 768, 1536 331 / 320, 14700 of 2 of 768, 1536 806 / 785 (fewer columns: 3633 frames, 3 of 256, 3500 classes 81 / 86; thirteen rows and more: 31500 of 2 of 832, 1664 2447 / 2526, 14700 of 4 of 896, 260
// 1941 / 1969, of 4 of 960, 260 2092 / 2250, though 14700 of 2 of 960, 260 1150 / 1107).
// float: 2, 4 and 8 within 0.5 % in all three forms.
int band_rows(const GemmDesc& d, int ntm, int ntn) {
    if (d.in_type == DT_F32) return 8;
    if (d.atrans) return ntm >= 10 && ntm <= 12 && ntn >= 10 ? 8 : 4;
    long long k = 0;
    for (int s = 0; s < d.nseg; ++s) k += d.seg[s].K;
    const long long right = k * d.N * 2, MB = 1 << 20;
    if (d.btrans) return d.M > 8192 && (right <= 4 * MB || (d.M <= 32768 && d.N >= 640 && right <= 32 * MB)) ? 8 : 4;
    return d.M > 16384 && right <= (d.N <= 4096 ? 12 : 4) * MB ? 8 : 4;
}
// Tile counts and store modes for a tile shape and edge treatment.
template <typename TO>
void set_tiles(const GemmDesc& d, Params& P, int tm, int tn, int mode) {
    const size_t w = sizeof(TO) == 4 ? 16 : 8;
    P.Nst = d.N;
    P.c_vec = aligned(d.C, w) && d.ldc % 4 == 0 && ((d.batch > 1 ? d.sC : 0) % 4 == 0);
    if (sizeof(TO) == 2 && P.c_vec && aligned(d.C, 16) && d.ldc % 8 == 0 && ((d.batch > 1 ? d.sC : 0) % 8 == 0)) P.c_vec = 2;   // 16-byte bf16 stores
    if (mode == EDGE) {                                  // the last group of columns of a row is stored whole or not at all
        if (d.c_pad) P.Nst = (d.N + 7) & ~7;
        if (P.c_vec == 2 && P.Nst % 8) P.c_vec = 1;
        if (P.c_vec == 1 && P.Nst % 4) P.c_vec = 0;
    }
    if (mode == WHOLE && d.Npad > 0) P.c_vec = 0;        // whole tiles are computed, the stores stop at column N
    P.p_vec = (d.N % 4 == 0 && !(mode == WHOLE && d.Npad > 0)) ? 1 : 0;   // (the scratch itself is 256-byte aligned)
    P.ntm = (d.M + tm - 1) / tm;
    P.ntn = ((mode == WHOLE && d.Npad > 0 ? d.Npad : d.N) + tn - 1) / tn;
    P.band = band_rows(d, P.ntm, P.ntn);
}

template <typename TI, typename TO>
hipError_t dispatch(const GemmDesc& given, hipStream_t stream) {
    GemmDesc d = given;
    Params P = make_params<TI>(d);
    const int batch = d.batch > 0 ? d.batch : 1;
    bool direct = direct_form(d);
    if (run_mode<TI>(d, P, 128, 128, direct) == GUARDED) d.guarded_parts = true;   // (whatever the tile)
    GemmPlan plan = make_plan(d, direct);
    // the plan's tile looks at the shape only: check it against the operands' alignment and fall back
    int mode = run_mode<TI>(d, P, kTileM[plan.tile], kTileN[plan.tile], direct);
    // (on the 128x128 tile with the plan's number of parts)
    if (plan.tile != GEMM_TILE_128 && (mode == GUARDED || (plan.tile == GEMM_TILE_256 && !(direct && !d.atrans && d.btrans)))) {
        plan.tile = GEMM_TILE_128; plan.deep = false;
        mode = run_mode<TI>(d, P, 128, 128, direct);
    }
    if (direct && mode == GUARDED) {
        direct = false;
        mode = run_mode<TI>(d, P, 128, 128, false);
    }
    if (plan.tile == GEMM_TILE_RESIDENT) {
        set_tiles<TO>(d, P, 128, 128, mode);
        if constexpr (sizeof(TI) == 2 && sizeof(TO) == 2) {
            if (P.c_vec == 2) {
                const int parts = resident_parts(d);
                switch (d.seg[0].K / 64) {
                case 1: return launch_resident_nk<1>(P, parts, stream);
                case 2: return launch_resident_nk<2>(P, parts, stream);
                case 3: return launch_resident_nk<3>(P, parts, stream);
                default: return launch_resident_nk<4>(P, parts, stream);
                }
            }
        }
        plan.tile = GEMM_TILE_128S;                        // (rows of C that take no 16-byte stores)
    }
    const int tm = kTileM[plan.tile], tn = kTileN[plan.tile];
    set_tiles<TO>(d, P, tm, tn, mode);
    P.splits = plan.splits;
    P.partial = plan.splits > 1 ? d.partial : nullptr;
    P.rs_partial = plan.splits > 1 ? d.partial + (size_t)plan.splits * batch * d.M * d.N : nullptr;
    dim3 grid((unsigned)(P.ntm * P.ntn), (unsigned)plan.splits, (unsigned)batch);
    auto launch = [&](auto to) {
        typedef decltype(to) T;
        if constexpr (sizeof(TI) == 4) return launch_f32(d, P, mode, direct, plan.tile, grid, stream);
        else if (!direct) return launch_staged<TI, T>(d, P, mode, grid, stream);
        else return launch_direct<T>(d, P, mode, plan.tile == GEMM_TILE_128 && plan.deep ? 1 : kDirectVariant[plan.tile], grid, stream);
    };
    if (plan.splits == 1) return launch(TO{});
    const hipError_t e = launch(float{});                  // partial tiles are float whatever the output type
    if (e != hipSuccess) return e;
    const long long total = (long long)d.M * d.N;
    const int vec4 = (P.c_vec && d.N % 4 == 0) ? 1 : 0;
    unsigned blocks = (unsigned)((total + 255) / 256 < 2048 ? (total + 255) / 256 : 2048);
    hipLaunchKernelGGL((splitk_reduce_kernel<TI, TO>), dim3(blocks, 1, batch), dim3(256), 0, stream, d.partial, plan.splits,
                       d.M, d.N, static_cast<TO*>(d.C), d.ldc, d.sC, static_cast<const TI*>(d.bias), d.sBias,
                       P.rs_partial, d.rowsum, d.sRowsum, vec4);
    return hipGetLastError();
}

// As many parts, up to `most`, as put no more than `target` workgroups on `tiles` tiles and leave each at least min_slabs slabs.
int parts_of(long long target, int most, long long tiles, int slabs, int min_slabs) {
    int s = (int)(target / tiles);
    if (s > most) s = most;
    while (s > 1 && slabs / s < min_slabs) --s;
    return s < 1 ? 1 : s;
}

// Estimated time (us) of `units` workgroups of a float tile with `slabs` slabs each.  The matrix cores of a CU take 1.71 us for a
// slab of 128x128 and 0.43 for one of 64x64 and are shared by the workgroups on it (measured 1.9 and 0.54, alone on a CU 2.35 and
// 0.66).  128x128 tiles come two to a CU and leave together: a last round of few of them still shares CUs, 3.8 a slab and round of
// 512.  What the small tile loses in every slab it gains there.  X W^T, us, 128x128 / 64x64: 1344 x 2048 twice, K = 1024 122 / 102;
// 1260 x 4096 twice, K = 2048 488 / 367, 2100 702 / 570, 1680 472 / 448, 2688 708 / 679, 840 240 / 237; 1344 x 32000, K = 256 210 / 187; 2048 x 1024 twice,
// K = 1280 91 / 53.
double f32_time(bool small, double units, double slabs) {
    const double x = units / 256.0;
    if (small) return slabs * (x <= 1.0 ? 0.66 : 0.54 * (double)(long long)(x + 0.999999));
    return slabs * (x <= 1.0 ? 2.35 : 3.8 * (double)(long long)(x / 2.0 + 0.999999));
}
// Float operands: tile and number of parts of K by the least estimated time.
void plan_f32(const GemmDesc& d, bool direct, int Ne, int Nr, GemmPlan* p) {
    const int batch = d.batch > 0 ? d.batch : 1;
    const long long t128 = (long long)((d.M + 127) / 128) * ((Ne + 127) / 128) * batch, t64 = (long long)((d.M + 63) / 64) * ((Ne + 63) / 64) * batch;
    int slabs = 0;
    for (int s = 0; s < d.nseg; ++s) slabs += (d.seg[s].K + 31) / 32;
    const double out_bytes = (double)batch * d.M * Nr * sizeof(float);
    int first = 1, last = 1;
    if (!d.add && d.partial) {
        if (d.long_parts) {
            if (d.nseg == 1 && t128 <= 256) {
                const int s1 = parts_of(256, 8, t128, slabs, 8), s2 = parts_of(512, 8, t128, slabs, 64), s = s1 > s2 ? s1 : s2;
                if ((size_t)s * batch * ((size_t)d.M * Nr + d.M) * sizeof(float) <= d.partial_bytes) first = last = s;
            }
        } else if (t128 <= 1024) last = 32;
    }
    auto search = [&](int tiles) {
        double best = 0.0;
        for (int s = first; s <= last; ++s) {
            const size_t need = s > 1 ? (size_t)s * batch * ((size_t)d.M * Nr + d.M) * sizeof(float) : 0;
            if (s > first && (slabs / s < 4 || need > d.partial_bytes || need > ((size_t)256 << 20))) break;
            for (int small = 0; small < tiles; ++small) {
                double t = f32_time(small != 0, (double)(small ? t64 : t128) * s, (slabs + s - 1) / s);
                if (s > 1) t = (t + 4.5 + 2.0 * s * out_bytes / 4e6) * (12.0 / 11.0);
                if (best == 0.0 || t < best) { best = t; p->tile = small ? GEMM_TILE_64 : GEMM_TILE_128; p->splits = s; p->partial_bytes = need; }
            }
        }
    };
    if (d.guarded_parts) { search(1); first = last = p->splits; }
    search(direct ? 2 : 1);
}

// Estimated time (us) of a slab of `tiles` bf16 tiles spread over the CUs: it grows by whole workgroups on the fullest CU.  64x64 with
// three buffers: one hides no load latency (0.335), several share the CU's matrix cores and LDS (measured 0.45, 0.64, 0.86, 1.04 for two to
// five); 128x64: two a CU, 0.47 alone and 0.65 for both, a third in a round of its own; 128x128: 0.7, a third less where two share a CU.
// X W^T and dA W of 84 to 8000 rows, 256 to 4096 columns and contractions of 256 to 32000 (270 products, all tiles and parts): the
// chosen plan takes 1.024 times the best one's time on average, where an estimate that grew smoothly took 1.05 and left long
// contractions unsplit, e.g. dA W, K = 4096 twice, us, 128x64 unsplit / 128x128 in two parts: 1660 x 2048 85 / 68, 672 x 2048 (64x64) 61 / 38 (in five).
double bf16_slab(int tile, double tiles) {
    const int most = (int)((tiles + 255.0) / 256.0);      // workgroups on a CU
    if (tile == GEMM_TILE_64) return most <= 1 ? 0.335 : 0.215 * most;
    if (tile == GEMM_TILE_128X64) return most / 2 * 0.644 + most % 2 * 0.47;
    return most <= 1 ? 0.7 : 0.462 * most;
}

// How a product of this shape is run.  allow_r: the 256x128 direct tile may be chosen (bf16 operands in one of its forms).
GemmPlan make_plan(const GemmDesc& d, bool allow_r) {
    GemmPlan p{GEMM_TILE_128, false, 1, 0};
    const int batch = d.batch > 0 ? d.batch : 1;
    const int Ne = d.Npad > 0 ? d.Npad : d.N;             // (the caller sets Npad only where the unguarded kernel applies)
    // (in whole pairs of 16-byte words: a product and its twin padded to them are planned alike)
    const int Nr = d.in_type == DT_BF16 ? (Ne + 15) & ~15 : (Ne + 7) & ~7;
    const long long t256 = (long long)((d.M + 255) / 256) * ((Ne + 255) / 256) * batch;
    const long long t128 = (long long)((d.M + 127) / 128) * ((Ne + 127) / 128) * batch;
    int ktot = 0;
    for (int s = 0; s < d.nseg; ++s) ktot += d.seg[s].K;
    if (d.in_type == DT_BF16) {
        if (allow_r && resident_parts(d) > 0) { p.tile = GEMM_TILE_RESIDENT; return p; }
        // Few large tiles and a very long contraction (the softmax layer's input gradient, dA W form): the 256x256 tile, which
        // moves half the operand bytes of 128x128 per flop and reads A once where N is 256.  Up to 64 tiles: split along K over
        // up to one workgroup per CU, if every part keeps at least 24 slabs and the parts fill three quarters of the CUs; up to
        // 239 (beyond, 256x128 tiles fill a round unsplit): in the smallest number of parts that fills whole rounds to 90 %, if every
        // part keeps 64 slabs.  N = 256, K = 32000, us, the best split of 256x128 / 128x128 / 256x256: 2688 rows 82 / 78 / 73 (20
        // parts), 5376 rows 125 / 131 / 115, 43008 rows 862 / 1018 / 755 (3 parts); 1344 rows (6 tiles) 128x128 45.
        if (allow_r && d.nseg == 1 && !d.rowsum && d.partial && !d.atrans && d.btrans && t256 < 240 && Nr % 256 == 0) {
            const int slabs = (d.seg[0].K + 63) / 64;
            int s = 0;
            if (t256 <= 64) {
                s = parts_of(256, 24, t256, slabs, 24);
                if (t256 * s < 192) s = 0;
            } else {
                for (int k = 2; k <= 8 && s == 0 && slabs / k >= 64; ++k) {
                    const double rounds = (double)t256 * k / 256.0;
                    if (rounds / (double)(long long)(rounds + 0.999999) >= 0.9) s = k;
                }
            }
            const size_t need = (size_t)s * batch * ((size_t)d.M * Nr + d.M) * sizeof(float);
            if (s > 1 && need <= d.partial_bytes) { p.tile = GEMM_TILE_256; p.splits = s; p.partial_bytes = need; return p; }
        }
        if (allow_r) {
            const long long tr = (long long)((d.M + 255) / 256) * ((Ne + 127) / 128) * batch;
            // Enough 256x128 tiles to put two on (nearly) every CU: the tile that moves 3/4 of the operand bytes of
            // 128x128 per flop, and the only one whose loop keeps the matrix cores above half of their rate.  With a contraction
            // of up to five slabs the first slab's latency and the output are most of a tile's time, and three workgroups of 128x128
            // per CU overlap those better while there are not many rounds of tiles (us, 256x128 / 128x128, K = 256: 336 x 32000
            // 15.8 / 14.4, 2688 x 32000 74.9 / 65.0, 3633 x 32000 106 / 110, 5376 x 32000 142 / 147; K = 264: 5376 x 2048 twice
            // 36.9 / 31.8, 10752 x 4096 twice 116 / 103; K = 512: 5376 x 2048 twice 35.9 / 36.1).
            if (tr >= 480) { p.tile = !d.atrans && ktot <= 320 && tr <= 3000 ? GEMM_TILE_128S : GEMM_TILE_256X128; return p; }
            // Fewer tiles than that but a long contraction next to a narrow output (the softmax layer's input gradient
            // at large batch): the same tile, split along K into the smallest number of parts that fills whole
            // rounds of 512 resident workgroups to 90 %, if every part keeps 64 slabs and the float partial tiles
            // stay below an eighth of the operand bytes.
            if (tr >= 128 && d.nseg == 1 && d.partial && !d.rowsum && (!d.long_parts || (d.M % 256 == 0 && Ne % 128 == 0 && (ktot + 15) / 16 % 4 == 0))) {
                const int slabs = (d.seg[0].K + 63) / 64;
                for (int s = 1; s <= 8; ++s) {
                    const double rounds = (double)tr * s / 512.0;
                    const double eff = rounds / (double)(long long)(rounds + 0.999999);
                    if (eff < 0.9 || slabs / s < 64) continue;
                    const size_t need = s > 1 ? (size_t)s * batch * ((size_t)d.M * Nr + d.M) * sizeof(float) : 0;
                    if (s > 1 && ((long long)16 * s * Nr > d.seg[0].K || need > d.partial_bytes)) break;
                    p.tile = GEMM_TILE_256X128; p.splits = s; p.partial_bytes = need;
                    return p;
                }
            }
        }
    }
    // Few output tiles, or a last round of them that is nearly empty: split K (both segments as one range of slabs) into the
    // number of parts whose estimated time is least, if that is a twelfth below not splitting.  A workgroup's slab takes
    // 1.9 us on a CU in float (the matrix rate), 0.7 us in bf16 (its chain of load, fragment reads and products; two
    // workgroups of a CU overlap, so more than one per CU costs by a third less).  Splitting adds a reduction launch and
    // the float partial tiles' way out and back.  Measured against at most eight parts of at least eight slabs and one
    // segment only: dz of 336 frames (6 tiles, K = 32000) 49 -> 21 us, the dA W products of the paper-shaped model in float
    // at batch 64 (dx: 88 tiles, K = 4096) 301 -> 137 us on average.
    // long_parts: at most eight parts of at least eight slabs, up to one workgroup per CU (of 64 slabs: up to two).  For the
    // logits, which are rounded to bf16 and then exponentiated: one ulp of a logit of 4 is 3 % of its class's probability,
    // so that another order of their sums shows in dz and the gradient.  Cut into parts of four slabs they moved single
    // elements of the gradient by 5e-2 of its root mean square (84 frames, z of 1024, 500 classes).
    if (d.in_type == DT_F32) {
        plan_f32(d, allow_r, Ne, Nr, &p);
        return p;
    }
    int slabs = 0;
    for (int s = 0; s < d.nseg; ++s) slabs += (d.seg[s].K + 63) / 64;
    const bool any_tile = allow_r && !d.atrans;           // X W^T and dA W come in every tile
    auto tiles = [&](int tile) { return (double)((d.M + kTileM[tile] - 1) / kTileM[tile]) * ((Ne + kTileN[tile] - 1) / kTileN[tile]) * batch; };
    auto need_of = [&](int s) { return s > 1 ? (size_t)s * batch * ((size_t)d.M * Nr + d.M) * sizeof(float) : (size_t)0; };
    const double tile_bytes = (double)batch * d.M * Nr * sizeof(float);
    auto estimate = [&](int tile, int s) {
        const double t = bf16_slab(tile, tiles(tile) * s) * ((slabs + s - 1) / s);
        return s == 1 ? t : t + 4.5 + 0.42e-6 * s * tile_bytes;
    };
    int most = 1;
    if (d.long_parts) {
        if (!d.add && d.partial && d.nseg == 1 && t128 <= 256) {
            const int s1 = parts_of(256, 8, t128, slabs, 8), s2 = parts_of(512, 8, t128, slabs, 64), s = s1 > s2 ? s1 : s2;
            if (s > 1 && need_of(s) <= d.partial_bytes) p.splits = s;
        }
    } else if (!d.add && d.partial && t128 <= 1024) most = 32;
    auto search = [&](int first, int last, bool all) {
        double best = 0.0;
        for (int s = first; s <= last; ++s) {
            if (s > first && (slabs / s < 4 || need_of(s) > d.partial_bytes || need_of(s) > ((size_t)256 << 20))) break;
            for (int tile : {GEMM_TILE_128, GEMM_TILE_64, GEMM_TILE_128X64}) {
                // (more than one a CU in many short parts: 336 x 256, K = 32000 2 us slower on 64x64 in 21 than on 128x128 in 32)
                if (tile != GEMM_TILE_128 && (!all || (s > 16 && tiles(tile) * s > 256.0))) continue;
                double t = estimate(tile, s);
                if (s > 1 && most > 1) t *= tile == GEMM_TILE_128 ? 12.0 / 11.0 : 1.2;
                if (best == 0.0 || t < best) { best = t; p.tile = tile; p.splits = s; p.partial_bytes = need_of(s); }
            }
        }
    };
    const int first = p.splits, last = most > first ? most : first;
    // The guarded kernel has 128x128 tiles only, so its number of parts is theirs: aligned operands of dz, 462 x 461, K = 2000, take 64x64
    // tiles unsplit, of which 16 guarded workgroups would walk 32 slabs each.  Softmax block of that model, us, in one part / in eight:
    // 222 / 97 (P = 66, V = 1500: 110 / 47 in six); in float, with eight and 13 parts, 119 / 112.
    if (d.guarded_parts) search(first, last, false);
    search(d.guarded_parts ? p.splits : first, d.guarded_parts ? p.splits : last, any_tile);
    // dA^T X, at most one 128x128 workgroup per CU: run the loads further ahead (three LDS buffers)
    p.deep = p.tile == GEMM_TILE_128 && d.atrans && d.btrans && t128 * p.splits <= 256;
    return p;
}

}  // namespace

size_t gemm_partial_bytes(int M, int N, int K, int batch, DType in_type, bool long_parts) {
    GemmDesc d{};
    d.long_parts = long_parts;
    d.M = M; d.N = N; d.batch = batch; d.nseg = 1; d.seg[0].K = K; d.in_type = in_type;
    d.partial = reinterpret_cast<float*>(16); d.partial_bytes = ~size_t(0);
    // the largest of what the tile families would use in any operand form: alignment decides between them only at launch time
    size_t need = make_plan(d, false).partial_bytes;
    for (int form = 0; form < 3; ++form) {
        d.atrans = form == 2; d.btrans = form >= 1;
        const size_t a = make_plan(d, true).partial_bytes;
        if (a > need) need = a;
    }
    return need;
}

// The split-K scratch that bounds what softmax_xent_fwd_bwd_noalloc accepts, for its product with the output M x N and the
// contraction K.  A fixed rule of its own: how the products are really split may change (they take what scratch there
// is), which calls fit the resident array may not.
size_t noalloc_partial_bytes(int M, int N, int K, DType in_type) {
    const long long t256 = (long long)((M + 255) / 256) * ((N + 255) / 256), t128 = (long long)((M + 127) / 128) * ((N + 127) / 128);
    const int bk = in_type == DT_BF16 ? 64 : 32, slabs = (K + bk - 1) / bk;
    auto bytes = [&](int s) { return s > 1 ? (size_t)s * ((size_t)M * N + M) * sizeof(float) : (size_t)0; };
    size_t need = 0;
    if (t128 <= 256) {
        const int s1 = parts_of(256, 8, t128, slabs, 8), s2 = parts_of(512, 8, t128, slabs, 64);
        if (in_type == DT_BF16 || !(t256 >= 512 && K >= 512)) need = bytes(s1 > s2 ? s1 : s2);
    }
    if (in_type == DT_BF16 && M % 256 == 0 && N % 128 == 0 && K % 64 == 0) {
        const long long tr = (long long)(M / 256) * (N / 128);
        if (tr >= 128 && tr < 480) {
            for (int s = 1; s <= 8; ++s) {
                const double rounds = (double)tr * s / 512.0, eff = rounds / (double)(long long)(rounds + 0.999999);
                if (eff < 0.9 || slabs / s < 64) continue;
                if (!(s > 1 && (long long)16 * s * N > K) && bytes(s) > need) need = bytes(s);
                break;
            }
        }
        if (tr < 480 && t256 <= 64 && N % 256 == 0) {
            const int s = parts_of(256, 16, t256, slabs, 24);
            if (s > 1 && t256 * s >= 192 && bytes(s) > need) need = bytes(s);
        }
    }
    return need;
}

hipError_t launch_gemm(const GemmDesc& d, hipStream_t stream) {
    if (d.M <= 0 || d.N <= 0) return hipSuccess;
    if (d.in_type == DT_F32 && d.out_type == DT_F32) return dispatch<float, float>(d, stream);
    if (d.in_type == DT_BF16 && d.out_type == DT_BF16) return dispatch<bf16_t, bf16_t>(d, stream);
    if (d.in_type == DT_BF16 && d.out_type == DT_F32) return dispatch<bf16_t, float>(d, stream);
    return hipErrorInvalidValue;
}

// Independent products of the dA^T X form with float results, one launch for up to GROUP_MAX of them (the weight gradients of
// several layers: together they fill the device, one by one most of them leave half of it idle).
template <typename TI>
static bool group_ok(const GemmDesc& d) {
    if (!(d.out_type == DT_F32 && d.atrans && d.btrans && !d.add && !d.bias && d.nseg == 1 && d.M > 0 && d.N > 0)) return false;
    const Params P = make_params<TI>(d);
    return run_mode<TI>(d, P, 128, 128, true) != GUARDED;
}
bool gemm_group_ok(const GemmDesc* descs, int n) {
    for (int i = 0; i < n; ++i) {
        if (descs[i].in_type != descs[0].in_type) return false;
        if (!(descs[i].in_type == DT_BF16 ? group_ok<bf16_t>(descs[i]) : group_ok<float>(descs[i]))) return false;
    }
    return n > 0;
}

namespace {
// The group's table for tiles of tm x tn; returns the number of tiles.
template <typename TI>
int fill_group(GroupParams& G, const GemmDesc* in, int m, int tm, int tn, int* mode) {
    *mode = WHOLE;
    for (int k = 0; k < m; ++k) { const Params P = make_params<TI>(in[k]); if (run_mode<TI>(in[k], P, tm, tn, true) != WHOLE) *mode = EDGE; }
    G.n = m;
    int total = 0;
    for (int k = 0; k < m; ++k) {
        G.p[k] = make_params<TI>(in[k]);
        set_tiles<float>(in[k], G.p[k], tm, tn, *mode);
        G.first[k] = total;
        total += G.p[k].ntm * G.p[k].ntn * (in[k].batch > 0 ? in[k].batch : 1);
    }
    G.first[m] = total;
    return total;
}

// Tile: 256x128 whenever its partly empty edge tiles cost less than a tenth more products than 128x128 tiles would.  A group
// of few tiles and a long contraction (narrow layers, many frames) would leave most of the device idle for the whole
// contraction: its products run one by one, each split along K (about 8 us of launches each against 0.8 us per slab saved to
// an eighth).
hipError_t launch_group_bf16(const GemmDesc* in, int m, hipStream_t stream) {
    long long t_r = 0, t_128 = 0;
    int longest = 0;                                      // slabs of the longest contraction
    for (int k = 0; k < m; ++k) {
        const GemmDesc& d = in[k];
        const long long batch = d.batch > 0 ? d.batch : 1, ntn = (d.N + 127) / 128;
        t_r += (d.M + 255) / 256 * ntn * batch * 2;
        t_128 += (d.M + 127) / 128 * ntn * batch;
        longest = longest > (d.seg[0].K + 63) / 64 ? longest : (d.seg[0].K + 63) / 64;
    }
    const bool large = t_r * 10 <= t_128 * 11;
    GroupParams G{};
    int mode = EDGE;
    const int total = fill_group<bf16_t>(G, in, m, large ? 256 : 128, 128, &mode);
    if (total <= 128 && longest > 16 * m) {
        for (int k = 0; k < m; ++k) { const hipError_t e = launch_gemm(in[k], stream); if (e != hipSuccess) return e; }
        return hipSuccess;
    }
    if (large) return mode == WHOLE ? launch_group_kernel<bf16_t, 4, 2, WHOLE, 1>(G, total, stream) : launch_group_kernel<bf16_t, 4, 2, EDGE, 1>(G, total, stream);
    return mode == WHOLE ? launch_group_kernel<bf16_t, 2, 2, WHOLE, 2>(G, total, stream) : launch_group_kernel<bf16_t, 2, 2, EDGE, 2>(G, total, stream);
}
// By the estimates of make_plan: one launch with either tile, or one by one (and split along K).
hipError_t launch_group_f32(const GemmDesc* in, int m, hipStream_t stream) {
    double together[2] = {0.0, 0.0}, alone = 0.0;
    for (int small = 0; small < 2; ++small) {
        const int t = small ? 64 : 128;
        double units = 0.0, work = 0.0;                   // (every tile with the mean of the contractions)
        int longest = 0;
        for (int k = 0; k < m; ++k) {
            const double n = (double)((in[k].M + t - 1) / t) * ((in[k].N + t - 1) / t) * (in[k].batch > 0 ? in[k].batch : 1);
            const int slabs = (in[k].seg[0].K + 31) / 32;
            units += n; work += n * slabs;
            longest = longest > slabs ? longest : slabs;
        }
        together[small] = f32_time(small != 0, units, units <= 256.0 ? longest : work / units);
    }
    for (int k = 0; k < m; ++k) {
        const GemmPlan p = make_plan(in[k], true);
        const double tiles = (double)((in[k].M + kTileM[p.tile] - 1) / kTileM[p.tile]) * ((in[k].N + kTileN[p.tile] - 1) / kTileN[p.tile]) * (in[k].batch > 0 ? in[k].batch : 1);
        alone += f32_time(p.tile == GEMM_TILE_64, tiles * p.splits, (in[k].seg[0].K + 32 * p.splits - 1) / (32 * p.splits)) + (p.splits > 1 ? 9.0 : 4.0);
    }
    const bool small = together[1] < together[0];
    if (alone < together[small]) {
        for (int k = 0; k < m; ++k) { const hipError_t e = launch_gemm(in[k], stream); if (e != hipSuccess) return e; }
        return hipSuccess;
    }
    GroupParams G{};
    int mode = EDGE;
    const int t = small ? 64 : 128, total = fill_group<float>(G, in, m, t, t, &mode);
    return launch_group_f32_tiles(G, total, mode, small ? GEMM_TILE_64 : GEMM_TILE_128, stream);
}
}  // namespace

// The products the grouped kernel can take run in it, the others one by one.
hipError_t launch_gemm_group(const GemmDesc* descs, int n, hipStream_t stream) {
    GemmDesc in[GROUP_MAX];
    for (int i = 0; i < n;) {
        int m = 0;
        hipError_t e;
        for (; i < n && m < GROUP_MAX; ++i) {
            if (gemm_group_ok(&descs[i], 1)) in[m++] = descs[i];
            else if ((e = launch_gemm(descs[i], stream)) != hipSuccess) return e;
        }
        if (m == 0) continue;
        if (m == 1) e = launch_gemm(in[0], stream);
        else e = in[0].in_type == DT_BF16 ? launch_group_bf16(in, m, stream) : launch_group_f32(in, m, stream);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace blstm
