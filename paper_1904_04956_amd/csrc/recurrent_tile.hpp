// What the kernels on 16-row tiles share (recurrent_tile.hip, recurrent_multi.hip).
#pragma once
#include "exchange.hpp"
#include "kernels.hpp"
#include "residency.hpp"
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
