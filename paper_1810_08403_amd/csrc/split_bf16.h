// fp32 values as sums of three bf16 values, for products on the bf16 matrix instructions (see gemm.hip).
#pragma once
#include <hip/hip_runtime.h>

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t bf16_pair(float lo, float hi)  // the chip's conversion: nearest even, two at a time
{
    return __builtin_bit_cast(uint32_t, (bf16x2){(__bf16)lo, (__bf16)hi});
}
// fp32 rows and weights are split times 2^16: the third part of any fp32 value, 2^-149 too, is then a bf16 value (they end at
// 2^-133). What that takes past the largest value gives a result that is not finite and is formed again (redo).
constexpr float kScale = 65536.f;
// two fp32 values into the three pairs of their parts
__device__ __forceinline__ void split_pair(float x, float y, uint32_t& p0, uint32_t& p1, uint32_t& p2)
{
    p0 = bf16_pair(x, y);
    x -= __uint_as_float(p0 << 16);
    y -= __uint_as_float(p0 & 0xffff0000u);
    p1 = bf16_pair(x, y);
    x -= __uint_as_float(p1 << 16);
    y -= __uint_as_float(p1 & 0xffff0000u);
    p2 = bf16_pair(x, y);
}
// what a value contributes to its row's sign: the mantissa, and whether it is zero. Neither the sign nor the exponent: a
// row times a power of two gives its results times that power, bit for bit.
__device__ __forceinline__ uint32_t row_code(uint32_t bits) { return bits << 9 | min(bits << 1, 1u); }
