// The cut of an fp32 number into bf16 planes (csrc/psd_planes.h), for tests/test_planes.py.
#include "psd_planes.h"

namespace {
uint32_t nearest(float x)                          // nearest bf16, even at ties; subnormal ones become zero
{
    const uint32_t b = __builtin_bit_cast(uint32_t, x);
    if ((b & 0x7f800000u) == 0x7f800000u) return b >> 16 | (b & 0x007fffffu ? 0x40u : 0u);
    const uint32_t r = (b + 0x7fffu + (b >> 16 & 1u)) >> 16;
    return (r & 0x7f80u) == 0 ? r & 0x8000u : r;
}
}  // namespace

extern "C" void planes_of(int n, const float* x, uint32_t* h, uint32_t* m, uint32_t* l)        // n even, two numbers per word
{
    for (int i = 0; i < n / 2; ++i)
        psd::cut(x[2 * i], x[2 * i + 1], h[i], m[i], l[i], [](float a, float b) { return nearest(a) | nearest(b) << 16; });
}
extern "C" float scale_of_factors() { return psd::kPlaneScale; }
extern "C" float scale_of_sums() { return psd::kPlaneUnscale; }
