// Splitting values into three bf16 parts, hi + mid + lo, two values at a time
// with gfx950's packed conversion (v_cvt_pk_bf16_f32: round to nearest even;
// compared with the integer form of that rounding on all finite and infinite
// FP32 values: the same bits).  A pair takes 3 conversions instead of 24
// integer operations, and a NaN stays a NaN whatever its payload.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace zp {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t bf16_pair(float a, float b)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{a, b}), bf16x2));
}
__device__ __forceinline__ float bf16_first(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_second(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// x, y -> w[p] = part p of x in the low half, of y in the high half.  T =
// float: the residuals are exact in FP32; T = double: exact in FP64.
template <class T> __device__ __forceinline__ void split3_pair(T x, T y, uint32_t (&w)[3])
{
    w[0] = bf16_pair((float)x, (float)y);
    x -= (T)bf16_first(w[0]);
    y -= (T)bf16_second(w[0]);
    w[1] = bf16_pair((float)x, (float)y);
    x -= (T)bf16_first(w[1]);
    y -= (T)bf16_second(w[1]);
    w[2] = bf16_pair((float)x, (float)y);
}

} // namespace zp
