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

// i / d, given 1 / d, for 0 <= i < 2^20, and for 0 <= i < d + 1024 with d up
// to kDivMax (an offset in an image's row or rows, plus a tile): the half
// keeps the product 0.5 / d from either neighbouring integer, more than its
// rounding.  The first wrong one: i = d - 1 at d = 6556022.  (A correction by
// the remainder makes it exact for every d, and the kernels 1 % slower.)
constexpr int32_t kDivMax = 1 << 22;
ONEXN_TILE_FN int32_t small_div(int32_t i, float inv) { return int32_t((float(i) + 0.5f) * inv); }

}  // namespace onexn
