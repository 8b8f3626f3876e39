// Enough of the device language to run the wait loops of csrc/exchange.hpp as host code, as a wavefront of one lane.  Loads past
// the caches are counted: `on_load` sees each before it reads, and more than `load_limit` of them end the program's patience.
#pragma once
#include <math.h>
#include <stdint.h>
#include <functional>

struct too_many_loads {};
inline unsigned long long loads = 0, load_limit = 1000000, clock_now = 0;
inline std::function<void(unsigned long long)> on_load;
template <typename T> T past_the_caches(const T* p) {
    if (++loads > load_limit) throw too_many_loads{};
    if (on_load) on_load(loads);
    return *p;
}

#define __device__
#define __forceinline__ inline
#define __shared__ static
#define __ATOMIC_RELAXED 0
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __hip_atomic_load(p, order, scope) past_the_caches(p)
#define __hip_atomic_store(p, v, order, scope) (void)(*(p) = (v))
#define __hip_atomic_fetch_add(p, v, order, scope) (void)(*(p) += (v))
#define __builtin_amdgcn_s_sleep(n) (void)0
#define __builtin_amdgcn_fence(order, scope) (void)0
#define __builtin_amdgcn_rcpf(x) (1.0f / (x))
#define __builtin_amdgcn_exp2f(x) exp2f(x)
#define __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, x, y, z) (c)
#define __all(x) (x)

struct uint2 { unsigned x, y; };
struct uint4 { unsigned x, y, z, w; };
inline uint4 make_uint4(unsigned x, unsigned y, unsigned z, unsigned w) { return {x, y, z, w}; }
struct { unsigned x, y, z; } static threadIdx;
inline void __syncthreads() {}
inline int __syncthreads_or(int v) { return v; }
inline unsigned long long wall_clock64() { return ++clock_now; }
