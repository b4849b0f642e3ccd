// Which rows (or columns) of a filter fall inside the image: plain integer logic, shared by the
// K-split convolution kernel (device) and by a host-side check against the definition.
#pragma once

#if defined(__HIPCC__)
#define SGPRS_HD __host__ __device__ __forceinline__
#else
#define SGPRS_HD inline
#endif

namespace sgprs {

constexpr int kTapMaskBits = 16;

// Bit t (t < kTapMaskBits - 1) is set when input row first + t lies in [0, size); no bit from kTapMaskBits on.
// Both ends are clamped: with wide padding a window may lie wholly before or past the image, where -first
// exceeds any shift and size - first is negative.  The clamps are constants, one instruction each, and need
// no filter size: whoever reads the mask asks for the bits of the filter's taps only.
SGPRS_HD unsigned tap_mask(int first, int size)
{
    const int before = -first, left = size - first;
    const int lo = before < 0 ? 0 : before > kTapMaskBits - 1 ? kTapMaskBits - 1 : before;
    const int hi = left < 0 ? 0 : left > kTapMaskBits - 1 ? kTapMaskBits - 1 : left;
    return ((1u << hi) - 1u) & ~((1u << lo) - 1u);
}

}  // namespace sgprs
