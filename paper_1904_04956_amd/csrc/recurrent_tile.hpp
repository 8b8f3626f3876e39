// What the kernels on 16-row tiles share (recurrent_tile.hip, recurrent_multi.hip).
#pragma once
#include "exchange.hpp"
#include "kernels.hpp"
#include "residency.hpp"
#include "xcd.hpp"
#include <type_traits>

namespace blstm {
namespace {

constexpr int NW = 4;                                    // wavefronts
constexpr int CHUNK = 16 * 8;                            // elements of eight columns of a tile

// NB floats, and as many bf16, as one access
template <int NB> struct Packs;
template <> struct Packs<2> { typedef float2 F; typedef unsigned W; };
template <> struct Packs<4> { typedef float4 F; typedef uint2 W; };
__device__ __forceinline__ float part(const float2& v, int b) { return b ? v.y : v.x; }
__device__ __forceinline__ float part(const float4& v, int b) { return b == 0 ? v.x : b == 1 ? v.y : b == 2 ? v.z : v.w; }
__device__ __forceinline__ float2 pack(const float (&v)[2]) { return make_float2(v[0], v[1]); }
__device__ __forceinline__ float4 pack(const float (&v)[4]) { return make_float4(v[0], v[1], v[2], v[3]); }
__device__ __forceinline__ unsigned pack(const unsigned (&v)[1]) { return v[0]; }
__device__ __forceinline__ uint2 pack(const unsigned (&v)[2]) { return make_uint2(v[0], v[1]); }
__device__ __forceinline__ unsigned word(unsigned v, int) { return v; }
__device__ __forceinline__ unsigned word(const uint2& v, int k) { return k ? v.y : v.x; }

// Keeps the weights of the fragments from FROM on in accumulation registers, which the products read as well as the others, and the
// others free: left to itself the compiler fills those with weights and reads the staged h one fragment at a time.
template <int FROM, int NB, int KQ>
__device__ __forceinline__ void park(uint4 (&w)[NB][KQ]) {
    typedef unsigned u4 __attribute__((ext_vector_type(4)));
    if constexpr (NB * KQ > 16) {
        __builtin_amdgcn_s_waitcnt(0x0F70);              // vmcnt(0): one wait for all of them
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int q = FROM; q < KQ; ++q) {
                u4 v = __builtin_bit_cast(u4, w[b][q]);
                asm volatile("" : "+a"(v));
                w[b][q] = __builtin_bit_cast(uint4, v);
            }
    }
}

// Stores by buffer: every lane issues them, what does not exist lies beyond the buffer and is dropped.
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));

constexpr int SC1 = 16;                                  // cache policy of an agent-scope store: write-through
// ... and of what is stored for later launches.  The fenced protocol's release, once a workgroup and frame, writes back whatever the XCD's L2 holds
// dirty: nothing, if all stores go through, and those that the signal need not wait for go out behind it.  us for two layers of 21 frames,
// forward / backward, write-back stores in front of the signal / so: 8 sequences of 512 cells 194 / 177 and 161 / 166, 128 620 / 580 and 480 / 475, 512
// 1125 / 1235 and 1080 / 1204, 2048 4500 / 4575 and 4280 / 4515, 64 of 1024 490 / 476 and 308 / 454.
constexpr int later(bool sentinel) { return sentinel ? 0 : SC1; }
constexpr unsigned DROP = 0x7FFFFFF0u;                   // an offset beyond every buffer
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer(void* p, unsigned bytes) { return __builtin_amdgcn_make_buffer_rsrc(p, 0, (int)bytes, 0x00020000); }
template <int AUX> __device__ __forceinline__ void put(__amdgpu_buffer_rsrc_t r, unsigned off, unsigned v) { __builtin_amdgcn_raw_buffer_store_b32(v, r, (int)off, 0, AUX); }
template <int AUX> __device__ __forceinline__ void put(__amdgpu_buffer_rsrc_t r, unsigned off, const uint2& v) { __builtin_amdgcn_raw_buffer_store_b64(u32x2_t{v.x, v.y}, r, (int)off, 0, AUX); }
template <int AUX> __device__ __forceinline__ void put(__amdgpu_buffer_rsrc_t r, unsigned off, const uint4& v) { __builtin_amdgcn_raw_buffer_store_b128(u32x4_t{v.x, v.y, v.z, v.w}, r, (int)off, 0, AUX); }
template <int AUX> __device__ __forceinline__ void put(__amdgpu_buffer_rsrc_t r, unsigned off, const float2& v) { put<AUX>(r, off, __builtin_bit_cast(uint2, v)); }
template <int AUX> __device__ __forceinline__ void put(__amdgpu_buffer_rsrc_t r, unsigned off, const float4& v) { put<AUX>(r, off, __builtin_bit_cast(uint4, v)); }
// For the exchange: write-back where the group shares an L2, else write-through.
template <typename V> __device__ __forceinline__ void put_exchange(bool write_back, __amdgpu_buffer_rsrc_t r, unsigned off, const V& v) {
    if (write_back) put<0>(r, off, v); else put<SC1>(r, off, v);
}
template <typename V> __device__ __forceinline__ V get(const void* base, unsigned off) { return *reinterpret_cast<const V*>(static_cast<const char*>(base) + off); }

// The N 16-byte words at off of a buffer, past the L1 (a look that came too early leaves no stale lines there), and again until no
// element of them is "not written yet".  Returns true if the wait was abandoned.
template <int N>
__device__ __forceinline__ void look_through(uint4 (&f)[N], __amdgpu_buffer_rsrc_t r, const unsigned (&off)[N]) {
#pragma unroll
    for (int q = 0; q < N; ++q) f[q] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off[q], 0, SC1));
}
template <int N>
__device__ __forceinline__ bool await(uint4 (&f)[N], __amdgpu_buffer_rsrc_t r, const unsigned (&off)[N], bool gave_up, unsigned* abort_word, unsigned long long limit) {
    return wait_written<false, N>(f, [&]() __attribute__((always_inline)) { look_through<N>(f, r, off); }, gave_up, abort_word, limit);
}

// A row-major tensor's piece of a tile (16 rows of the slice's units) is moved in whole lines: a wavefront takes four rows, sixteen
// neighbouring lanes one row's piece.  With a lane to a row every lane of a load of 16 bytes is in a line of its own, and a CU
// looks up one line a clock for every four lanes: 64 clocks an instruction instead of 16.  The cells' owners (row l16, units 4 NB wave + NB lq)
// and those lanes meet in LDS, where word p of a row's sixteen (or fewer) lies at p ^ row.
__device__ __forceinline__ int turned(int row, int p) { return row * 16 + (p ^ row); }

// Workgroups a CU holds of these kernels (their registers, and the launch bounds).  multi: those of recurrent_multi.hip.
constexpr int fwd_per_cu(int nb, int kq, bool multi) { return nb == 4 ? (kq <= (multi ? 4 : 8) ? 2 : 1) : kq == 4 ? (multi ? 2 : 4) : kq <= 12 ? 2 : 1; }
constexpr int bwd_per_cu(int nb, int kq, bool multi) { return nb == 4 ? (kq == 4 ? 2 : 1) : kq == 4 ? (multi ? 2 : 4) : kq <= 12 ? 2 : 1; }

// The groups of tiles a direction is cut into.
struct Cut { int nbg, per_group, grid, real; };

}  // namespace

// Several tiles a workgroup, slices of 16 NB units, width up to 32 KQ (recurrent_multi.hip).
hipError_t launch_rec_multi(const RecFwdArgs& a, int nb, int kq, bool sentinel, int grid, int real, hipStream_t st, bool* launched);
hipError_t launch_rec_multi(const RecBwdArgs& a, int nb, int kq, bool sentinel, int grid, int real, hipStream_t st, bool* launched);

}  // namespace blstm
