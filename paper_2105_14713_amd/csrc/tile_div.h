// Division of tile and pixel offsets through an fp32 reciprocal (a few
// instructions against some twenty of an integer division).  Plain C++, so
// that it can be checked on the host.
#pragma once

#include <cstdint>

#ifdef __HIPCC__
#define ONEXN_TILE_FN __host__ __device__ __forceinline__
#else
#define ONEXN_TILE_FN inline
#endif

namespace onexn {

// i / d for 0 <= i < 2^20, given 1 / d: the half keeps the product 0.5 / d
// from either neighbouring integer, more than its rounding.  For counts
// inside a tile only.
ONEXN_TILE_FN int32_t small_div(int32_t i, float inv) { return int32_t((float(i) + 0.5f) * inv); }

// i / d for any 0 <= i < 2^31 with a quotient below 2^20, given 1 / d: the
// product is then less than one off, and the remainder says which way.  For
// offsets that an image's size bounds (a row of 6556022 pixels is the first
// that small_div divides wrongly).
ONEXN_TILE_FN int32_t row_div(int32_t i, int32_t d, float inv) {
    const int32_t q = int32_t(float(i) * inv);
    const int32_t r = int32_t(uint32_t(i) - uint32_t(q) * uint32_t(d));
    return q + (r >= d) - (r < 0);
}

}  // namespace onexn
