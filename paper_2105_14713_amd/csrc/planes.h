// bf16 operand planes of the matrix-core kernels that run both precisions on
// the bf16 matrix instructions.
//
// A bf16 operand is one plane.  An fp32 operand is three: the value rounded to
// nearest bf16, the remainder rounded likewise, and the rest.  Each remainder
// is exact and at most half a unit of the plane above, so the rest fits bf16's
// 8 significand bits and the planes are the value exactly, down to 2^-110 (below
// that the rest loses what lies under 2^-133, bf16's last subnormal bit).
// A product takes the six plane products of weight 2^-16 and above; the three
// left out, a2*b3 + a3*b2 + a3*b3, are below 2^-24 * (1 + 2^-9) of it (2^-8
// and 2^-17 bound planes two and three; 0.9 * 2^-24 is the most seen) and
// have no preferred sign.  (Planes cut instead of rounded leave out up to
// 2^-21, always towards zero.)  a1*b1 goes to one accumulator, the five
// smaller ones to another, added at the end: the small terms are then not
// rounded to the large ones' last place.  Error against 64 bits, as a share of
// the fp32 instruction's kernels' on normal and ReLU'd operands: forward layers
// of 512 to 1024 channels that the dispatch takes 0.39 to 0.70, input gradients
// of 8 to 1024 channels 0.30 to 0.35; single products 1.4 * 2^-24 at most
// against 1.0 (cut: 7.8), their mean zero.  128 -> 128 3x3 at 28x28, batch 64,
// N = 32: 63.0 us, 63.7 with planes cut.
// Six bf16 products run at 2500 / 6 = 417 TFLOP/s against 157 of the fp32
// instruction.
//
// Infinities, NaN and values that round to infinity do not survive (inf - inf
// is NaN in the second plane), so a kernel on three planes looks at its
// accumulators at the end and computes outputs that are not finite again in
// plain fp32.
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

// Two floats rounded to nearest-even bf16, v0 in the low half.
__device__ __forceinline__ uint32_t round_pair(float v0, float v1) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{v0, v1}), bf16x2));
}

// Words k of the planes of eight consecutive contraction entries: entries 2k
// and 2k + 1.
__device__ __forceinline__ void cut_pair(float v0, float v1, int k, u32x4 (&p)[3]) {
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        const uint32_t w = round_pair(v0, v1);
        p[t][k] = w;
        if (t == 2) break;
        v0 -= __uint_as_float(w << 16);
        v1 -= __uint_as_float(w & 0xffff0000u);
    }
}
__device__ __forceinline__ void cut_pair(uint32_t v0, uint32_t v1, int k, u32x4 (&p)[1]) {
    p[0][k] = __builtin_amdgcn_perm(v1, v0, 0x05040100u);
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
