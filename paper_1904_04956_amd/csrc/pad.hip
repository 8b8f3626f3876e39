// Copies between compact tensors and zero-padded ones (rows that start 16-byte aligned).  Bound by memory: about 5 TB/s
// of the larger side, the compact side's 2- or 4-byte accesses of neighbouring lanes share their cache lines.
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
    const long long rows = (long long)t.rg * t.rp;
    const int cols = t.cs * t.cp, ld = t.cs * t.c;
    for (long long r = (long long)blockIdx.x * 4 + (threadIdx.x >> 6); r < rows; r += (long long)gridDim.x * 4) {
        const long long g = r / t.rp;
        const int j = (int)(r - g * t.rp);
        const T* s = src + (g * t.r + j) * ld;
        for (int c = (threadIdx.x & 63) * VEC; c < cols; c += 64 * VEC) {
            T v[VEC];
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                const int seg = (c + e) / t.cp, k = c + e - seg * t.cp;
                v[e] = (j < t.r && k < t.c && c + e < cols) ? s[seg * t.c + k] : (T)0;
            }
            if (c + VEC <= cols) *reinterpret_cast<uint4*>(dst + r * cols + c) = *reinterpret_cast<const uint4*>(v);
            else for (int e = 0; c + e < cols; ++e) dst[r * cols + c + e] = v[e];
        }
    }
}

// One thread per element of the compact side.
template <typename T>
__global__ __launch_bounds__(256) void compact_blocks_kernel(BlockCopies a, const T* __restrict__ padded, T* __restrict__ compact) {
    const BlockTensor t = a.t[blockIdx.y];
    const T* src = padded + t.padded;
    T* dst = compact + t.compact;
    const long long rows = (long long)t.rg * t.r;
    const int cols = t.cs * t.c, ld = t.cs * t.cp;
    for (long long r = (long long)blockIdx.x * 4 + (threadIdx.x >> 6); r < rows; r += (long long)gridDim.x * 4) {
        const long long g = r / t.r;
        const T* s = src + (g * t.rp + (r - g * t.r)) * ld;
        for (int c = threadIdx.x & 63; c < cols; c += 64) {
            const int seg = c / t.c;
            dst[r * cols + c] = s[seg * t.cp + c - seg * t.c];
        }
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

hipError_t launch_pad_blocks(const BlockTensor* t, int n, const void* compact, void* padded, DType type, hipStream_t st) {
    return type == DT_BF16 ? run<true, unsigned short>(t, n, compact, padded, st) : run<true, float>(t, n, compact, padded, st);
}
hipError_t launch_compact_blocks(const BlockTensor* t, int n, const void* padded, void* compact, DType type, hipStream_t st) {
    return type == DT_BF16 ? run<false, unsigned short>(t, n, padded, compact, st) : run<false, float>(t, n, padded, compact, st);
}

}  // namespace blstm
