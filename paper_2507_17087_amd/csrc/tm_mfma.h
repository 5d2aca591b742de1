// tm_mfma.h -- bf16 conversion and the matrix instruction the ranker's kernels share.
//
// MFMA fragment layout used throughout (16x16x32, one wave): lane l holds row
// (l % 16) of A and column (l % 16) of B, eight consecutive k values starting at
// 8 * (l / 16); the result holds rows 4 * (l / 16) + r (r = 0..3) of column l % 16.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tmk {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));

// Round to nearest even: one v_cvt_pk_bf16_f32 for two values.
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}
__device__ __forceinline__ uint16_t f2bf(float f) { return (uint16_t)pack_bf16(f, 0.f); }
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__device__ __forceinline__ bf16x8 as_bf(u16x8 v) { return __builtin_bit_cast(bf16x8, v); }

__device__ __forceinline__ f32x4 mfma16(u16x8 a, u16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf(a), as_bf(b), c, 0, 0, 0);
}

}  // namespace tmk
