// lane_group.h -- what the kernels that share a pixel quad between the lanes of
// a group have in common (group.hip, adjoint.hip).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <utility>

namespace convcrf {

template <typename F, int... I>
__device__ __forceinline__ void static_for(F&& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}

typedef float f32x4 __attribute__((ext_vector_type(4)));

// N consecutive 16-byte pieces from an aligned LDS address, read whole: use()
// in front of their first use keeps the compiler from narrowing a read to the
// floats that are used, which splits it into unaligned ones.
template <int N>
__device__ __forceinline__ void read_row(const float* p, f32x4 (&v)[N]) {
#pragma unroll
    for (int j = 0; j < N; ++j) v[j] = *reinterpret_cast<const f32x4*>(p + 4 * j);
}
__device__ __forceinline__ void use(f32x4& v) { asm volatile("" : "+v"(v)); }

// lanes 0..31: a + a of lane + 32; lanes 32..63: b + b of lane - 32
__device__ __forceinline__ float add_halves(float a, float b) {
    const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false,
                                                    false);
    return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}
// the same over the two 16-lane rows of each half
__device__ __forceinline__ float add_rows(float a, float b) {
    const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false,
                                                    false);
    return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}

}  // namespace convcrf
