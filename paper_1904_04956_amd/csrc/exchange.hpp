// The pieces of the protocols that the persistent kernels share (see recurrent.hip).
#pragma once
#include "common.hpp"

namespace blstm {

constexpr unsigned SENT16 = 0xFFFFu;

__device__ __forceinline__ unsigned ld_coh_u32(const unsigned* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// The cell state.  Spelt out: left to the compiler, which of the two products is rounded first differs from kernel to kernel and, with
// several units a lane, from unit to unit.
__device__ __forceinline__ float next_cell(float f, float c, float i, float g) { return __builtin_fmaf(f, c, i * g); }

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
// count this store in its vmcnt bookkeeping; its own waits then only wait for more than they need.  Not for the FENCED
// protocol: with nothing else in flight, the compiler leaves out the wait between a release's write-back and the counter.)
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
__device__ __forceinline__ unsigned max3(unsigned a, unsigned b, unsigned c) {   // (one instruction)
    const unsigned m = a > b ? a : b;
    return m > c ? m : c;
}

// Whether every element of every lane's f is written.  Branch-free, as it is asked on every frame, and half an operation a word: a lane's stores to an
// exchange copy are aligned words of 32 bits and more, and so is the marking, so that both elements of a word are written or neither
// is, and 0xFFFF in the upper one is what makes a word the largest.  APART: a chunk's words meet before they join m, for the backward kernels of 32-row tiles of 513 to 640 cells or
// several tiles a workgroup (us a launch, in one chain / apart: 100 sequences of 544 cells 95 / 88, 128 of 640 98 / 92, 700 of 1024 552 / 549; 100 of 768 97 / 98, and few sequences of 512 the same to 1 us slower).
template <int N, bool APART = false>
__device__ __forceinline__ bool all_written(const uint4 (&f)[N]) {
    unsigned m = 0;
#pragma unroll
    for (int q = 0; q < N; ++q) m = APART ? max3(m, max3(f[q].x, f[q].y, f[q].z), f[q].w) : max3(max3(m, f[q].x, f[q].y), f[q].z, f[q].w);
    return __all(m < SENT16 << 16);
}
// ... and of a copy of floats, whose words are stored each by itself.
constexpr unsigned SENT32 = 0xFFFFFFFFu;
template <int N>
__device__ __forceinline__ bool all_written32(const uint4 (&f)[N]) {
    unsigned m = 0;
#pragma unroll
    for (int q = 0; q < N; ++q) m = max3(max3(m, f[q].x, f[q].y), f[q].z, f[q].w);
    return __all(m != SENT32);
}
// The bounded wait for an operand: `look` loads it (past the caches that a look which came too early may have left stale lines in) until it is `whole`.
// Returns true if the wait was abandoned, at the time limit or as someone raised the abort word.  Wave-uniform.
template <bool NAP, typename W, typename L>
__device__ __forceinline__ bool look_until(W whole, L look, unsigned* abort_word, unsigned long long limit) {
    const unsigned long long t0 = wall_clock64();
    for (unsigned it = 1;; ++it) {
        asm volatile("" ::: "memory");                   // (loads by buffer are not taken to see what others store)
        look();
        if (whole()) return false;
        if constexpr (NAP) __builtin_amdgcn_s_sleep(1);
        if ((it & 31u) == 0) {
            if (ld_coh_u32(abort_word) != 0) return true;
            if (wall_clock64() - t0 > limit) {
                __hip_atomic_store(abort_word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                return true;
            }
        }
    }
}
template <bool NAP, int N, typename L>
__device__ __forceinline__ bool look_again(uint4 (&f)[N], L look, unsigned* abort_word, unsigned long long limit) {
    return look_until<NAP>([&]() __attribute__((always_inline)) { return all_written<N>(f); }, look, abort_word, limit);
}
// ... behind a first look, unless that found everything or an earlier wait was abandoned.
template <bool NAP, int N, typename L>
__device__ __forceinline__ bool wait_written(uint4 (&f)[N], L look, bool gave_up, unsigned* abort_word, unsigned long long limit) {
    if (gave_up || all_written<N>(f)) return gave_up;
    return look_again<NAP, N>(f, look, abort_word, limit);
}
template <int N, typename L>
__device__ __forceinline__ bool wait_written32(uint4 (&f)[N], L look, bool gave_up, unsigned* abort_word, unsigned long long limit) {
    if (gave_up || all_written32<N>(f)) return gave_up;
    return look_until<true>([&]() __attribute__((always_inline)) { return all_written32<N>(f); }, look, abort_word, limit);
}

// Barrier for LDS hazards only: waits for this wave's LDS operations, not for its global loads and
// write-through stores (a full __syncthreads would drain the loads issued ahead for the next item
// and the acknowledgements of the exchange stores on every item).
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// ---- FENCED protocol ----------------------------------------------------------------------------
// Waits until *cnt >= target; thread 0 polls.  One barrier inside.  Returns true (to every thread) if the
// wait was abandoned.
__device__ __forceinline__ bool wait_counter(unsigned* cnt, unsigned target, unsigned* abort_word, unsigned long long limit_ticks) {
    int gave_up = 0;
    if (threadIdx.x == 0) {
        const unsigned long long t0 = wall_clock64();
        unsigned it = 0;
        while (ld_coh_u32(cnt) < target) {
            __builtin_amdgcn_s_sleep(1);
            if ((++it & 63u) == 0) {
                if (ld_coh_u32(abort_word) != 0) { gave_up = 1; break; }
                if (wall_clock64() - t0 > limit_ticks) {
                    __hip_atomic_store(abort_word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    gave_up = 1;
                    break;
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    return __syncthreads_or(gave_up) != 0;
}
// After the workgroup's stores: the barrier orders them before thread 0's agent-scope release.
__device__ __forceinline__ void signal_counter(unsigned* cnt) {
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}

// ---- 16-row tiles (recurrent_small.hip, recurrent_tile.hip): fragments of 32 columns of 16 rows, one KB each ----------------
__device__ __forceinline__ f32x4_t mfma16(const uint4& a, const uint4& b, f32x4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

}  // namespace blstm
