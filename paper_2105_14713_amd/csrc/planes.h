// bf16 operand planes of the matrix-core kernels that run both precisions on
// the bf16 matrix instructions.
//
// A bf16 operand is one plane.  An fp32 operand is three: the value cut (not
// rounded) to its top 16 bits, the remainder cut likewise, and the rest, which
// together are the value exactly (3 x 8 significand bits; cutting never
// overflows).  A product then takes the six plane products of weight 2^-16
// and above; the three left out are below 2^-24 of it.  a1*b1 goes to one
// accumulator, the five smaller ones to another, added at the end: the small
// terms are then not rounded to the large ones' last place.  Measured against
// 64 bits on normal and ReLU'd operands over contractions of 64 to 50176: 0.4
// to 0.7 times the error of v_mfma_f32_32x32x2_f32 (one accumulator for all
// six: 0.85 to 1.5 times, and biased).  Six bf16 products run at 2500 / 6 =
// 417 TFLOP/s against 157 of the fp32 instruction.
//
// Infinities and NaN do not survive the cut (inf - inf is NaN in the second
// plane), so a kernel on three planes looks at its accumulators at the end
// and computes outputs that are not finite again in plain fp32.
#pragma once

#include "conv_common.h"

namespace onexn {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

template <typename T> struct Planes;
// `reg` is what a value is held as between its load and its cut: bf16 values
// in whole registers (16-bit variables are packed in pairs as they arrive,
// which waits for every load in turn).
template <> struct Planes<float> { static constexpr int NP = 3; typedef float reg; };
template <> struct Planes<uint16_t> { static constexpr int NP = 1; typedef uint32_t reg; };

// High halves of two words: (lo >> 16) | (hi & 0xffff0000).
__device__ __forceinline__ uint32_t pack_high(uint32_t lo, uint32_t hi) {
    return __builtin_amdgcn_perm(hi, lo, 0x07060302u);
}

// Words k of the planes of eight consecutive contraction entries: entries 2k
// and 2k + 1.
__device__ __forceinline__ void cut_pair(float v0, float v1, int k, u32x4 (&p)[3]) {
    uint32_t a = __float_as_uint(v0), b = __float_as_uint(v1);
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        p[t][k] = pack_high(a, b);
        if (t == 2) break;
        a = __float_as_uint(__uint_as_float(a) - __uint_as_float(a & 0xffff0000u));
        b = __float_as_uint(__uint_as_float(b) - __uint_as_float(b & 0xffff0000u));
    }
}
__device__ __forceinline__ void cut_pair(uint32_t v0, uint32_t v1, int k, u32x4 (&p)[1]) {
    p[0][k] = __builtin_amdgcn_perm(v1, v0, 0x05040100u);
}

// Eight consecutive contraction entries of one row as planes of 8 bf16.
__device__ __forceinline__ void to_planes(const float (&v)[8], u32x4 (&p)[3]) {
#pragma unroll
    for (int k = 0; k < 4; ++k) cut_pair(v[2 * k], v[2 * k + 1], k, p);
}
__device__ __forceinline__ void to_planes(const uint32_t (&v)[8], u32x4 (&p)[1]) {
#pragma unroll
    for (int k = 0; k < 4; ++k) cut_pair(v[2 * k], v[2 * k + 1], k, p);
}

template <int N> struct PlaneMfma;
template <> struct PlaneMfma<32> {   // 32x32x16 bf16
    typedef f32x16 acc_t;
    static constexpr int ACC = 16, COLS = 32;
    __device__ static acc_t mma(u32x4 a, u32x4 b, acc_t c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                       0, 0, 0);
    }
    __device__ static int row(int lane, int r) { return 8 * (r / 4) + 4 * (lane / 32) + (r % 4); }
};
template <> struct PlaneMfma<16> {   // 16x16x32 bf16
    typedef f32x4 acc_t;
    static constexpr int ACC = 4, COLS = 16;
    __device__ static acc_t mma(u32x4 a, u32x4 b, acc_t c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                       0, 0, 0);
    }
    __device__ static int row(int lane, int r) { return 4 * (lane / 16) + r; }
};

// Accumulator of one MFMA tile: one for bf16 operands, two for fp32 ones.
template <int N, int NP>
struct PlaneAcc {
    typedef PlaneMfma<N> M;
    static constexpr int NA = NP == 1 ? 1 : 2;
    typename M::acc_t c[NA];
    __device__ __forceinline__ void zero() {
#pragma unroll
        for (int i = 0; i < NA; ++i)
#pragma unroll
            for (int r = 0; r < M::ACC; ++r) c[i][r] = 0.f;
    }
    // Product i of MMAS of one contraction step.
    static constexpr int MMAS = NP == 1 ? 1 : 6;
    template <int i>
    __device__ __forceinline__ void product(const u32x4 (&a)[NP], const u32x4 (&b)[NP]) {
        if constexpr (NP == 1) {
            c[0] = M::mma(a[0], b[0], c[0]);
        } else {
            constexpr int pa[6] = {2, 0, 0, 1, 1, 0}, pb[6] = {0, 0, 2, 1, 0, 1};
            constexpr int acc = i == 1 ? 0 : 1;
            c[acc] = M::mma(a[pa[i]], b[pb[i]], c[acc]);
        }
    }
    __device__ __forceinline__ float value(int r) const {
        if constexpr (NA == 1) return c[0][r];
        else return c[0][r] + c[1][r];
    }
};

// First entry of a col-group's [zb, ze) with I >= c0 (I ascends; ze if none).
__device__ __forceinline__ int32_t lower_entry(const int32_t* __restrict__ I, int32_t zb, int32_t ze, int32_t c0) {
    int32_t lo = zb, hi = ze;
    while (hi - lo > 16) {                               // 16 independent samples a round
        const int32_t step = (hi - lo + 15) / 16;
        int32_t below = 0;
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int32_t e = lo + k * step;
            below += (e < hi && I[min(e, ze - 1)] < c0) ? 1 : 0;
        }
        const int32_t nlo = below == 0 ? lo : lo + (below - 1) * step + 1;
        hi = below == 0 ? lo : min(hi, lo + below * step);
        lo = nlo;
    }
    int32_t below = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) below += (lo + k < hi && I[min(lo + k, ze - 1)] < c0) ? 1 : 0;
    return lo + below;
}

__device__ __forceinline__ bool not_finite(float v) { return (__float_as_uint(v) & 0x7f800000u) == 0x7f800000u; }

}  // namespace onexn
