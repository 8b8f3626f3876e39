// Shared device helpers of the HIP kernels (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <utility>

namespace blstm {

typedef unsigned short bf16_t;                       // raw bfloat16 bits

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

// float -> bfloat16, round to nearest even (the hardware conversion of gfx950).
__device__ __forceinline__ bf16_t f2bf(float x) {
    return __builtin_bit_cast(unsigned short, (__bf16)x);
}
__device__ __forceinline__ float bf2f(bf16_t b) {
    return __builtin_bit_cast(float, ((uint32_t)b) << 16);
}
__device__ __forceinline__ uint32_t pack_bf2(float lo, float hi) {
    return (uint32_t)f2bf(lo) | ((uint32_t)f2bf(hi) << 16);
}

// f(FROM), f(FROM + 1), .. f(TO - 1), the number as a type
template <int FROM, typename F, int... K>
__device__ __forceinline__ void each_of(std::integer_sequence<int, K...>, F&& f) { (f(std::integral_constant<int, FROM + K>{}), ...); }
template <int FROM, int TO, typename F>
__device__ __forceinline__ void each(F&& f) { each_of<FROM>(std::make_integer_sequence<int, TO - FROM>{}, f); }

// Element load/store by storage type.
__device__ __forceinline__ float ld_f(const float* p) { return *p; }
__device__ __forceinline__ float ld_f(const bf16_t* p) { return bf2f(*p); }
__device__ __forceinline__ void st_f(float* p, float v) { *p = v; }
__device__ __forceinline__ void st_f(bf16_t* p, float v) { *p = f2bf(v); }

// Logistic function and tanh in float, without fast-math shortcuts: expf is the
// library's accurate version; the forms below stay finite for every input.
__device__ __forceinline__ float sigmoidf_(float a) { return 1.0f / (1.0f + expf(-a)); }
__device__ __forceinline__ float tanhf_(float a) { return tanhf(a); }

// Hardware exp2/rcp forms for the bf16 path: absolute error of a few 1e-7, far below the
// 2^-9 relative step of the bf16 values they feed; both saturate cleanly for large |a|.
// (v_exp_f32 and v_rcp_f32 directly: 1 ulp each, no range fix-ups; exp2 underflows to 0 and
// overflows to +inf, which the reciprocal maps to the right limits.)
__device__ __forceinline__ float fast_sigmoid(float a) {
    return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.44269504f * a));
}
__device__ __forceinline__ float fast_tanh(float a) {
    return 1.0f - 2.0f * __builtin_amdgcn_rcpf(__builtin_amdgcn_exp2f(2.88539008f * a) + 1.0f);
}

}  // namespace blstm
