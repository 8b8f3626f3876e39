// Row-wise softmax cross-entropy on a materialised logit matrix, with fixed-order sums.
#include "common.hpp"
#include "kernels.hpp"

namespace blstm {
namespace {

template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}
template <bool MAX> __device__ __forceinline__ float both(float a, float b) { return MAX ? fmaxf(a, b) : a + b; }
// Over the sixteen lanes of a row, in registers (quad_perm 1,0,3,2 and 2,3,0,1, row_half_mirror, row_mirror).
template <bool MAX>
__device__ __forceinline__ float row_reduce(float v) {
    v = both<MAX>(v, dpp<0xB1>(v)); v = both<MAX>(v, dpp<0x4E>(v));
    v = both<MAX>(v, dpp<0x141>(v)); return both<MAX>(v, dpp<0x140>(v));
}
// Over a workgroup of NW <= 16 wavefronts, one barrier: sh is free again behind the next one.
template <bool MAX, int NW>
__device__ __forceinline__ float block_reduce(float v, float* sh) {
    const int lane = threadIdx.x & 63, k = lane & 15;
    v = row_reduce<MAX>(v);
    v = both<MAX>(v, __shfl_xor(v, 16, 64)); v = both<MAX>(v, __shfl_xor(v, 32, 64));
    if (lane == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    return row_reduce<MAX>(k < NW ? sh[k] : MAX ? -INFINITY : 0.0f);
}

// One workgroup per row: max, sum of exponentials, loss term, then u <- s (p - onehot) in place.
// General form: three passes over the row (the second and third normally hit L2).
template <typename TS>
__global__ __launch_bounds__(256) void softmax_rows_kernel(TS* u, long long ldu, const int32_t* labels,
                                                           float* row_loss, int V, float s) {
    __shared__ float sh[2][4];
    const int m = blockIdx.x;
    TS* row = u + (long long)m * ldu;
    float mx = -INFINITY;
    for (int v = threadIdx.x; v < V; v += blockDim.x) mx = fmaxf(mx, ld_f(row + v));
    mx = block_reduce<true, 4>(mx, sh[0]);
    float sum = 0.0f;
    for (int v = threadIdx.x; v < V; v += blockDim.x) sum += expf(ld_f(row + v) - mx);
    sum = block_reduce<false, 4>(sum, sh[1]);
    // a label outside [0, V) is never used as an index: the frame's loss term becomes NaN and its row p without a one-hot
    const int lab = labels[m];
    const bool lab_ok = (unsigned)lab < (unsigned)V;
    const float inv = 1.0f / sum;
    if (threadIdx.x == 0) row_loss[m] = lab_ok ? s * (logf(sum) + mx - ld_f(row + lab)) : __builtin_nanf("");
    __syncthreads();                                   // the label's logit is read before it is overwritten
    for (int v = threadIdx.x; v < V; v += blockDim.x) {
        float p = expf(ld_f(row + v) - mx) * inv;
        st_f(row + v, s * (p - ((lab_ok && v == lab) ? 1.0f : 0.0f)));
    }
    // rows padded to whole 16-byte words: zeros in the padding (the products of dE/du may read it)
    if ((int)threadIdx.x < 8 && V + (int)threadIdx.x < (int)min(ldu, (long long)((V + 7) & ~7))) st_f(row + V + threadIdx.x, 0.0f);
}

// Rows that fit the registers of one workgroup (V <= NT * NC 16-byte words, rows 16-byte aligned and padded to whole ones: the
// padding counts as -inf on the way in and is zero on the way out): the row is read once with 16-byte loads and written back as
// dE/du with 16-byte stores, in between it stays in registers as exponentials (KEEP) or as it was read.  HBM traffic:
// one read and one write.
// A long row is spread over more threads rather than more registers per thread, so that several rows per CU are in flight and
// one row's loads and stores run under another's arithmetic.  What bounds it is the vector ALU nearly as much as the memory:
// taking each exponential once, and reducing in registers with one barrier, is 128 -> 104 us for 5376 rows of 32000 bf16 logits
// (5.4 -> 6.6 TB/s), 65 -> 53 for 2688.  In float, where the general kernel read the row three times and took two accurate
// exponentials, 1344 rows of 32000 159 -> 57 us.
// Short rows leave most of the threads without a word, and a wavefront whose lanes have none skips it: taking 32
// exponentials of -inf a thread instead, the whole softmax block of 86016 rows took 189 us where it takes 112 (64 classes, z of
// 32), 249 where 177 (1000).
template <typename TS> struct Word;
template <> struct Word<bf16_t> {
    static constexpr int N = 8;
    static __device__ __forceinline__ void unpack(const uint4& w, float (&x)[8]) {
        const uint32_t t[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) { x[2 * q] = bf2f((bf16_t)(t[q] & 0xFFFFu)); x[2 * q + 1] = bf2f((bf16_t)(t[q] >> 16)); }
    }
    static __device__ __forceinline__ uint4 pack(const float (&p)[8]) { return make_uint4(pack_bf2(p[0], p[1]), pack_bf2(p[2], p[3]), pack_bf2(p[4], p[5]), pack_bf2(p[6], p[7])); }
    // exp(x - mx) = exp2(x log2(e) - mx log2(e)): one multiply-add and the hardware exp2 (the argument is <= 0; a result
    // below the normal range flushes to 0, as its probability does in bf16)
    static __device__ __forceinline__ float exponential(float x, float mx) { return __builtin_amdgcn_exp2f(__builtin_fmaf(x, 1.44269504f, -mx * 1.44269504f)); }
    // s (p - onehot): the scaled sum and, in one element, the one-hot
    static __device__ __forceinline__ float out(float e, float inv, float sinv, float s, bool hot) { return hot ? e * sinv - s : e * sinv; }
};
template <> struct Word<float> {
    static constexpr int N = 4;
    static __device__ __forceinline__ void unpack(const uint4& w, float (&x)[4]) {
        x[0] = __builtin_bit_cast(float, w.x); x[1] = __builtin_bit_cast(float, w.y); x[2] = __builtin_bit_cast(float, w.z); x[3] = __builtin_bit_cast(float, w.w);
    }
    static __device__ __forceinline__ uint4 pack(const float (&p)[4]) {
        return make_uint4(__builtin_bit_cast(uint32_t, p[0]), __builtin_bit_cast(uint32_t, p[1]), __builtin_bit_cast(uint32_t, p[2]), __builtin_bit_cast(uint32_t, p[3]));
    }
    static __device__ __forceinline__ float exponential(float x, float mx) { return expf(x - mx); }
    static __device__ __forceinline__ float out(float e, float inv, float sinv, float s, bool hot) { return s * (e * inv - (hot ? 1.0f : 0.0f)); }
};
template <typename TS, int NC, int NT, bool KEEP>
__global__ __launch_bounds__(NT, 8) void softmax_rows_regs_kernel(TS* u, long long ldu, const int32_t* labels,
                                                               float* row_loss, int V, float s) {
    typedef Word<TS> W;
    constexpr int N = W::N, NW = NT / 64;
    __shared__ float sh[2][NW], label_logit;
    const int m = (int)(gridDim.x - 1 - blockIdx.x);   // from the end: the logits written last are in the last-level cache still
    TS* row = u + (long long)m * ldu;
    const int nchunks = (V + N - 1) / N, nout = (int)min(ldu, (long long)((V + 7) & ~7)) / N;   // words with logits, and with padding
    const int lab = labels[m];
    const bool lab_ok = (unsigned)lab < (unsigned)V;   // (as in the general kernel: an out-of-range label gives a NaN loss term)
    uint4 r[NC];
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        const int c = threadIdx.x + NT * i;
        r[i] = make_uint4(0, 0, 0, 0);
        if (c < nchunks) r[i] = *reinterpret_cast<const uint4*>(row + N * c);
    }
    // (in LDS in front of the barriers below: read before the row is overwritten)
    if (threadIdx.x == 0) label_logit = lab_ok ? ld_f(row + lab) : 0.0f;
    float e[KEEP ? NC : 1][N], mx = -INFINITY;
    // a word that no lane of the wavefront has (KEEP: uniform), or this thread has not
    const int first = KEEP ? __builtin_amdgcn_readfirstlane(threadIdx.x) : threadIdx.x;
    auto beyond = [&](int i) { return first + NT * i >= nchunks; };
    auto values = [&](int i, float (&x)[N]) __attribute__((always_inline)) {
        const int c = threadIdx.x + NT * i;
        if (!KEEP) asm volatile("" : "+v"(r[i].x), "+v"(r[i].y), "+v"(r[i].z), "+v"(r[i].w));   // (unpacked anew each time: kept, the values take more registers than there are)
        W::unpack(r[i], x);
        if (N * c + N > V) {                           // the row's last, partly padded word, and the threads beyond the row
#pragma unroll
            for (int k = 0; k < N; ++k) if (N * c + k >= V) x[k] = -INFINITY;
        }
    };
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        if (beyond(i)) continue;
        float x[N];
        values(i, x);
#pragma unroll
        for (int k = 0; k < N; ++k) {
            mx = fmaxf(mx, x[k]);
            if (KEEP) e[i % (KEEP ? NC : 1)][k] = x[k];
        }
    }
    mx = block_reduce<true, NW>(mx, sh[0]);
    float sum = 0.0f;
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        if (beyond(i)) continue;
        float x[N];
        if (!KEEP) values(i, x);
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const float v = W::exponential(KEEP ? e[i % (KEEP ? NC : 1)][k] : x[k], mx);
            sum += v;
            if (KEEP) e[i % (KEEP ? NC : 1)][k] = v;
        }
    }
    sum = block_reduce<false, NW>(sum, sh[1]);
    const float inv = 1.0f / sum, sinv = s / sum;
    if (threadIdx.x == 0) row_loss[m] = lab_ok ? s * (logf(sum) + mx - label_logit) : __builtin_nanf("");
    const int labc = lab_ok ? lab / N : -1;            // the one word whose output also carries the -s of the one-hot
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        const int c = threadIdx.x + NT * i;
        if (c >= nout) continue;
        float x[N], p[N];
        if (!KEEP) values(i, x);
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const float v = KEEP ? e[i % (KEEP ? NC : 1)][k] : W::exponential(x[k], mx);
            p[k] = W::out(v, inv, sinv, s, false);
        }
        if (c == labc) {
#pragma unroll
            for (int k = 0; k < N; ++k) {
                const float v = KEEP ? e[i % (KEEP ? NC : 1)][k] : W::exponential(x[k], mx);
                if (k == lab % N) p[k] = W::out(v, inv, sinv, s, true);
            }
        }
        if (N * c + N > V) {
#pragma unroll
            for (int k = 0; k < N; ++k) if (N * c + k >= V) p[k] = 0.0f;
        }
        *reinterpret_cast<uint4*>(row + N * c) = W::pack(p);
    }
}

__global__ __launch_bounds__(1024) void sum_to_scalar_kernel(const float* v, int M, float* out) {
    __shared__ float sh[16];
    float acc = 0.0f;
    for (int i0 = threadIdx.x; i0 < M; i0 += 8 * 1024) {   // eight loads in flight, added in order (43008 rows: one by one 20 us)
        float x[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) x[k] = i0 + 1024 * k < M ? v[i0 + 1024 * k] : 0.0f;
#pragma unroll
        for (int k = 0; k < 8; ++k) acc += x[k];
    }
    acc = block_reduce<false, 16>(acc, sh);
    if (threadIdx.x == 0) out[0] = acc;
}

}  // namespace

hipError_t launch_softmax_rows(void* u, long long ldu, const int32_t* labels, float* row_loss,
                               int M, int V, float s, DType store, hipStream_t st) {
    if (M <= 0) return hipSuccess;
    const bool bf = store == DT_BF16;
    const int n = bf ? 8 : 4;                          // elements of a 16-byte word
    const bool vec = ldu % n == 0 && ldu >= (V + n - 1) / n * n && reinterpret_cast<uintptr_t>(u) % 16 == 0;
    const long long words = (ldu < ((V + 7) & ~7) ? ldu : ((V + 7) & ~7)) / n;
#define BLSTM_SOFTMAX_REGS(NC, NT, KEEP) do { \
    if (bf) hipLaunchKernelGGL((softmax_rows_regs_kernel<bf16_t, NC, NT, KEEP>), dim3(M), dim3(NT), 0, st, static_cast<bf16_t*>(u), ldu, labels, row_loss, V, s); \
    else hipLaunchKernelGGL((softmax_rows_regs_kernel<float, NC, NT, true>), dim3(M), dim3(NT), 0, st, static_cast<float*>(u), ldu, labels, row_loss, V, s); } while (0)
    if (vec && words <= 4 * 256) BLSTM_SOFTMAX_REGS(4, 256, true);
    else if (vec && words <= 4 * 512) BLSTM_SOFTMAX_REGS(4, 512, true);
    else if (vec && words <= 4 * 1024) BLSTM_SOFTMAX_REGS(4, 1024, true);
    else if (vec && words <= 8 * 1024) BLSTM_SOFTMAX_REGS(8, 1024, false);
#undef BLSTM_SOFTMAX_REGS
    else if (bf) hipLaunchKernelGGL(softmax_rows_kernel<bf16_t>, dim3(M), dim3(256), 0, st, static_cast<bf16_t*>(u), ldu, labels, row_loss, V, s);
    else hipLaunchKernelGGL(softmax_rows_kernel<float>, dim3(M), dim3(256), 0, st, static_cast<float*>(u), ldu, labels, row_loss, V, s);
    return hipGetLastError();
}

hipError_t launch_sum_to_scalar(const float* v, int M, float* out, hipStream_t st) {
    hipLaunchKernelGGL(sum_to_scalar_kernel, dim3(1), dim3(1024), 0, st, v, M, out);
    return hipGetLastError();
}

}  // namespace blstm
