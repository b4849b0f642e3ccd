// Which rows (or columns) of a filter fall inside the image: plain integer logic, shared by the
// K-split convolution kernel (device) and by a host-side check against the definition.
#pragma once

#if defined(__HIPCC__)
#define SGPRS_HD __host__ __device__ __forceinline__
#else
#define SGPRS_HD inline
#endif

namespace sgprs {

// Bit t (t < taps) is set when input row first + t lies in [0, size).  Both ends are clamped: with
// wide padding a window may lie wholly before or past the image, where -first exceeds taps and
// size - first is negative.
SGPRS_HD unsigned tap_mask(int first, int size, int taps)
{
    const int before = -first, left = size - first;
    const int lo = before < 0 ? 0 : before < taps ? before : taps;
    const int hi = left < lo ? lo : left < taps ? left : taps;
    return (1u << hi) - (1u << lo);
}

}  // namespace sgprs
