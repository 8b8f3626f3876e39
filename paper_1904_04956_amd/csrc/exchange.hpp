// The pieces of the sentinel protocol that the persistent bf16 kernels share (see recurrent.hip).
#pragma once
#include "common.hpp"

namespace blstm {

constexpr unsigned SENT16 = 0xFFFFu;

__device__ __forceinline__ unsigned ld_coh_u32(const unsigned* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

__device__ __forceinline__ bf16_t coh_bf16(float v) {
    bf16_t b = f2bf(v);
    return b == SENT16 ? (bf16_t)0x7FC0 : b;             // a NaN result must not look like "not written yet"
}
__device__ __forceinline__ void st_coh_8B(bf16_t* p, const uint2& v) {
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), (unsigned long long)v.x | ((unsigned long long)v.y << 32),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// One 16-byte store with the cache policy of an agent-scope atomic store (write-through to L2: sc1), written in assembly
// because atomics stop at 8 bytes and a store instruction costs the memory pipeline the same whatever its width.  The
// protocol needs no atomicity beyond each 16-bit element's, which every aligned store gives.  (The compiler does not
// count this store in its vmcnt bookkeeping; its own waits then only wait for more than they need.)
typedef unsigned int u32x4s_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void st_coh_16B(bf16_t* p, const uint4& v) {
    const u32x4s_t w = {v.x, v.y, v.z, v.w};
    // (s_nop: a store of more than 8 bytes reads its data registers over several cycles, and a vector-ALU write to them
    // must not follow at once; the compiler inserts that wait state for stores it knows, but cannot see into this one)
    asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" :: "v"(p), "v"(w) : "memory");
}
__device__ __forceinline__ uint4 ld_coh_16B(const bf16_t* p) {
    const unsigned long long* q = reinterpret_cast<const unsigned long long*>(p);
    const unsigned long long lo = __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned long long hi = __hip_atomic_load(q + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return make_uint4((unsigned)lo, (unsigned)(lo >> 32), (unsigned)hi, (unsigned)(hi >> 32));
}
// The chunks are checked on every frame, so the test is branch-free and one operation per word:
// 0xFFFF is the largest 16-bit value, so a packed unsigned maximum over all words has a 0xFFFF half
// iff some word has one; the zero-halfword test on the complement of that maximum decides.
typedef unsigned short u16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ unsigned max_halves(unsigned x, unsigned y) {
    return __builtin_bit_cast(unsigned, __builtin_elementwise_max(__builtin_bit_cast(u16x2_t, x), __builtin_bit_cast(u16x2_t, y)));
}
__device__ __forceinline__ unsigned max_halves(const uint4& v) { return max_halves(max_halves(v.x, v.y), max_halves(v.z, v.w)); }
__device__ __forceinline__ bool has_sentinel_half(unsigned w) { return ((~w - 0x00010001u) & w & 0x80008000u) != 0; }

// Barrier for LDS hazards only: waits for this wave's LDS operations, not for its global loads and
// write-through stores (a full __syncthreads would drain the loads issued ahead for the next item
// and the acknowledgements of the exchange stores on every item).
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

}  // namespace blstm
