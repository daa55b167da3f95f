// An fp32 number in three bf16 planes (not installed).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace psd {

// A factor is multiplied by 2^24 before it is cut, and a sum of products by 2^-48 in the end.  Every fp32 number is a multiple of
// 2^-149, so what is cut is one of 2^-125, and so is each of its planes: none of them is smaller than the smallest normal bf16
// (2^-126), however small the number.  (Cut as they are, numbers below 2^-109 lose their last plane and numbers below 2^-117 two,
// which shows where the other factor is large: errors of 1e-41 with activations of 1e12 gave a dW of zero.)  Products below
// 2^-126 are 2^-174 of a sum, nothing beside the smallest fp32 number.  Above 2^104 the planes are not finite any more, nor is a
// sum above 2^80.
constexpr float kPlaneScale = 0x1p24f, kPlaneUnscale = 0x1p-48f;

// (x0, x1) times 2^24 = h + m + l, the differences are exact: |m| <= 2^-8 |x|, |l| <= 2^-17 |x|.
// to_bf16: two floats to the nearest bf16 (even at ties), the first in the low half.
template <class ToBf16>
__host__ __device__ __forceinline__ void cut(float x0, float x1, uint32_t& h, uint32_t& m, uint32_t& l, ToBf16 to_bf16)
{
    auto low = [](uint32_t x) { return __builtin_bit_cast(float, x << 16); };
    auto high = [](uint32_t x) { return __builtin_bit_cast(float, x & 0xffff0000u); };
    x0 *= kPlaneScale;
    x1 *= kPlaneScale;
    h = to_bf16(x0, x1);
    x0 -= low(h);
    x1 -= high(h);
    m = to_bf16(x0, x1);
    l = to_bf16(x0 - low(m), x1 - high(m));
}

}  // namespace psd
