// Copies between compact tensors and zero-padded ones.  Bound by memory, a wavefront along a row, no division per element.
// Neither side need be aligned: compact rows are not, nor are padded ones of a width that is left as it is (W_x of the first
// layer in bf16 mode, whose D is not padded), so 16-byte words are moved as bytes of any alignment.  Measured on 45.6 M
// parameters (five layers of 583 cells): the weights padded in 93 us (182 MB), the gradient compacted in 110 us (365 MB);
// with a division per element 209 and 305.
#include "common.hpp"
#include "kernels.hpp"

namespace blstm {
namespace {

// One thread per 16-byte word of the padded side, 64 threads along a row, four rows a workgroup.
template <typename T>
__global__ __launch_bounds__(256) void pad_blocks_kernel(BlockCopies a, const T* __restrict__ compact, T* __restrict__ padded) {
    constexpr int VEC = 16 / (int)sizeof(T);
    const BlockTensor t = a.t[blockIdx.y];
    const T* src = compact + t.compact;
    T* dst = padded + t.padded;
    const unsigned rows = (unsigned)t.rg * (unsigned)t.rp;
    const int cols = t.cs * t.cp, ld = t.cs * t.c;
    for (unsigned r = blockIdx.x * 4 + (threadIdx.x >> 6); r < rows; r += gridDim.x * 4) {
        const unsigned g = r / (unsigned)t.rp;
        const int j = (int)(r - g * (unsigned)t.rp);
        const T* s = src + (size_t)(g * (unsigned)t.r + j) * ld;
        T* d = dst + (size_t)r * cols;
        // (a word lies in one segment: their padded widths are whole words, or there is one segment)
        for (int c = (threadIdx.x & 63) * VEC; c < cols; c += 64 * VEC) {
            const int seg = t.cs == 1 ? 0 : (int)((unsigned)c / (unsigned)t.cp), k = c - seg * t.cp;
            if (j < t.r && k + VEC <= t.c) {
                uint4 w;
                __builtin_memcpy(&w, s + seg * t.c + k, 16);
                __builtin_memcpy(d + c, &w, 16);
                continue;
            }
            T v[VEC];
#pragma unroll
            for (int e = 0; e < VEC; ++e) v[e] = (j < t.r && k + e < t.c) ? s[seg * t.c + k + e] : (T)0;
            if (c + VEC <= cols) {
                __builtin_memcpy(d + c, v, 16);
            } else {
#pragma unroll
                for (int e = 0; e < VEC; ++e) if (c + e < cols) d[c + e] = v[e];
            }
        }
    }
}

// One thread per element of the compact side.
template <typename T>
__global__ __launch_bounds__(256) void compact_blocks_kernel(BlockCopies a, const T* __restrict__ padded, T* __restrict__ compact) {
    const BlockTensor t = a.t[blockIdx.y];
    const T* src = padded + t.padded;
    T* dst = compact + t.compact;
    const unsigned rows = (unsigned)t.rg * (unsigned)t.r;
    for (unsigned r = blockIdx.x * 4 + (threadIdx.x >> 6); r < rows; r += gridDim.x * 4) {
        const unsigned g = r / (unsigned)t.r;
        const T* s = src + (size_t)(g * (unsigned)t.rp + (r - g * (unsigned)t.r)) * ((size_t)t.cs * t.cp);
        T* d = dst + (size_t)r * ((size_t)t.cs * t.c);
        for (int seg = 0; seg < t.cs; ++seg, s += t.cp, d += t.c) {
            int c = threadIdx.x & 63;
            for (; c + 192 < t.c; c += 256) {             // four loads in flight
                const T v0 = s[c], v1 = s[c + 64], v2 = s[c + 128], v3 = s[c + 192];
                d[c] = v0; d[c + 64] = v1; d[c + 128] = v2; d[c + 192] = v3;
            }
            for (; c < t.c; c += 64) d[c] = s[c];
        }
    }
}

// One thread per element to clear: columns h .. hp - 1 of every block of hp columns.
__global__ __launch_bounds__(256) void zero_columns_kernel(float* p, long long blocks, int hp, int h) {
    const int w = hp - h;
    const long long n = blocks * w;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
        const long long b = i / w;
        p[b * hp + h + (int)(i - b * w)] = 0.0f;
    }
}

template <bool PAD, typename T>
hipError_t run(const BlockTensor* tensors, int n, const void* src, void* dst, hipStream_t st) {
    for (int i = 0; i < n; i += BLOCK_COPIES_MAX) {
        BlockCopies a{};
        const int m = n - i < BLOCK_COPIES_MAX ? n - i : BLOCK_COPIES_MAX;
        long long most = 1;
        for (int k = 0; k < m; ++k) {
            a.t[k] = tensors[i + k];
            const long long rows = (long long)a.t[k].rg * a.t[k].rp;
            if (rows > most) most = rows;
        }
        const long long blocks = (most + 3) / 4 < 1024 ? (most + 3) / 4 : 1024;
        const dim3 grid((unsigned)blocks, (unsigned)m);
        if constexpr (PAD) hipLaunchKernelGGL(pad_blocks_kernel<T>, grid, dim3(256), 0, st, a, static_cast<const T*>(src), static_cast<T*>(dst));
        else hipLaunchKernelGGL(compact_blocks_kernel<T>, grid, dim3(256), 0, st, a, static_cast<const T*>(src), static_cast<T*>(dst));
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace

hipError_t launch_zero_columns(float* p, long long blocks, int hp, int h, hipStream_t st) {
    const long long n = (blocks * (hp - h) + 255) / 256;
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(zero_columns_kernel, dim3((unsigned)(n < 2048 ? n : 2048)), dim3(256), 0, st, p, blocks, hp, h);
    return hipGetLastError();
}
hipError_t launch_pad_blocks(const BlockTensor* t, int n, const void* compact, void* padded, DType type, hipStream_t st) {
    return type == DT_BF16 ? run<true, unsigned short>(t, n, compact, padded, st) : run<true, float>(t, n, compact, padded, st);
}
hipError_t launch_compact_blocks(const BlockTensor* t, int n, const void* padded, void* compact, DType type, hipStream_t st) {
    return type == DT_BF16 ? run<false, unsigned short>(t, n, padded, compact, st) : run<false, float>(t, n, padded, compact, st);
}

}  // namespace blstm
