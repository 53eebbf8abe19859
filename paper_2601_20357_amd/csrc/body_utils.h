// What the kernels of the draft body share: bf16 conversions and vector types.
#pragma once
#include <hip/hip_bf16.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tabed {

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4b;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4b;

__device__ __forceinline__ uint16_t f32_to_bf16_bits(float f) {            // round to nearest even
    return __builtin_bit_cast(uint16_t, (__bf16)f);
}

__device__ __forceinline__ uint2 pack_bf16x4(float a, float b, float c, float d) {
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
    typedef __attribute__((ext_vector_type(2))) float f32x2;
    return make_uint2(__builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2)),      // one instruction a pair
                      __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{c, d}, bf16x2)));
}

}  // namespace tabed
