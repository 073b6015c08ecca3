// Weight gradient of a 1xN-pruned convolution in bf16, NCHW, N in {16, 32},
// on the matrix cores.  Any kernel size, stride and padding.
//
// Paper: Lin et al., "1xN Pattern for Pruning Convolutional Neural Networks"
// (arXiv 2105.14713), Sec. 3.4 and 4.1 (fine-tuning with the pattern fixed):
//     dD[z][i][q][r] = sum_{b,oh,ow} dY[b][gN+i][oh][ow] * X[b][I[z]][oh*sh-ph+q][ow*sw-pw+r],
// per col-group a contraction over the output pixels of its N rows of dY with
// one row of X per (kept block, tap) pair, pairs numbered tap-major.
//
// Work.  A workgroup computes the entries of 32 pairs and R rows of one
// col-group (R = N, or half of N = 32 for layers of few tiles).  The
// contraction runs along the pixels, which are contiguous in both operands, so
// a fragment entry is eight neighbouring pixels of a row: a lane loads eight
// with one 16-byte load and stores them to LDS as they are;
// nothing is transposed.  Octets are cut per output row (a 1x1 layer without
// stride or padding is one row per image); the last one of a row is masked in
// dY, and columns outside the image are masked in X.  Octets are stored
// [octet][row] with an odd row pitch: neither the stores (lanes along octets)
// nor the reads (lanes along rows) conflict.  Sixteen waves each take their
// part of every 512-pixel chunk, with two chunks of loads in flight, and the
// partial sums are added through LDS in wave order: one workgroup makes each
// entry, so results do not vary from run to run.
//
// What bounds it: the loads in flight.  A workgroup reads N + 32 rows of all
// pixels, and a layer has t * KK / 32 workgroups of pairs.  256 -> 1024 at
// 14x14, batch 64, N = 32 (t = 4096): 1920 us with one workgroup per block and
// lanes along the pixels, without matrix cores; 44 us here.  64 -> 256 at 56x56
// (16 tiles of pairs for 256 compute units): 7090 and 410 us.
//
// Sums that are not finite are computed again in plain fp32 over the pixels
// whose tap lies inside the image (masked columns multiply as zeros, and zero
// times infinity is NaN), a wave per sum,
// until it is NaN.  256 -> 1024 1x1 at 14x14, batch 64 (44 us): 52 us with a NaN
// in dY, 163 with an infinity, 250 with nothing else in it; 64 -> 256 at 56x56
// (410 us): 410, 2300 and 500 (by one thread per sum: 33, 32 and 48 ms).

#include <algorithm>
#include <utility>

#include "planes.h"

namespace onexn {
namespace {

struct DwArgs {
    const int32_t* P;
    const int32_t* I;
    const void* x;
    const void* dy;
    float* dD;
    int32_t m, n, G, t, KK, kw;
    int32_t H, W, Ho, Wo, batch, sh, sw, ph, pw;
    int32_t noct;                    // octets of an output row
    int32_t chunks;                  // chunks of octets
    int32_t tiles;                   // tiles of pairs per col-group (upper bound)
    int32_t dk, drow, db, doh;       // a chunk's step in (octet, row), and that row step in (image, row)
    int32_t x_total, y_total;        // elements of x and dY
    int32_t total;                   // workgroups
};

// How X's octets are read: kFlat, one image row of pixels, no taps; kTap,
// stride-1 columns, shifted and masked per tap; kStrided, element by element.
enum DwMode { kFlat, kTap, kStrided };

constexpr int kDwWaves = 16, kDwThreads = 64 * kDwWaves;
constexpr int kDwPairs = 32;         // pairs of a tile
constexpr int kDwOcts = 64;          // octets of a chunk: one per lane, so a wave stages one row at a time
constexpr int kDwRS = kDwThreads / kDwOcts;   // rows staged per item

// R: rows of dY of a workgroup (16 or 32).
template <int R> struct DwShape {
    static constexpr int RP = kDwPairs + R + 1;          // odd
    static constexpr int UX = kDwPairs / kDwRS, UY = R / kDwRS;
    static constexpr int OPW = kDwOcts / kDwWaves;       // octets a wave multiplies per chunk
    static constexpr int KG = R == 32 ? 2 : 4;           // octets of one MFMA
    static constexpr int STEPS = OPW / KG;
    static_assert(kDwOcts * RP * 16 >= kDwWaves * kDwPairs * R * 4, "the partial sums fit the staging space");
};

// Eight values between load and store: as loaded, or element by element.
template <bool kVec> struct Oct;
template <> struct Oct<true> { u32x4 v; };
template <> struct Oct<false> { uint32_t v[8]; };

__device__ __forceinline__ void load_oct(const uint16_t* p, Oct<true>& o) { __builtin_memcpy(&o.v, p, 16); }
// Element by element, `step` apart, indices clamped into [0, total).
__device__ __forceinline__ void load_each(const uint16_t* p, int32_t at, int32_t step, int32_t total,
                                          uint32_t (&v)[8]) {
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = p[max(0, min(at + j * step, total - 1))];
}
__device__ __forceinline__ void load_each(const uint16_t* p, int32_t at, int32_t step, int32_t total, u32x4& v) {
    uint32_t e[8];
    load_each(p, at, step, total, e);
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = e[2 * k] | (e[2 * k + 1] << 16);
}

// All ones where bit j of m is set.
__device__ __forceinline__ uint32_t bit_ones(uint32_t m, int j) { return uint32_t(int32_t(m << (31 - j)) >> 31); }
__device__ __forceinline__ uint32_t pair_ones(uint32_t m, int k) {
    return (bit_ones(m, 2 * k) & 0xffffu) | (bit_ones(m, 2 * k + 1) & 0xffff0000u);
}
__device__ __forceinline__ u32x4 masked(u32x4 v, uint32_t m) {
    if (__any(m != 255u)) {
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] &= pair_ones(m, k);
    }
    return v;
}
__device__ __forceinline__ u32x4 masked(const uint32_t (&v)[8], uint32_t m) {
    u32x4 p;
#pragma unroll
    for (int k = 0; k < 4; ++k) p[k] = (v[2 * k] | (v[2 * k + 1] << 16)) & pair_ones(m, k);
    return p;
}

template <int N, int R, int MODE>
__global__ void __launch_bounds__(kDwThreads, 4) bwd_weight_bf16(DwArgs a) {
    typedef DwShape<R> S;
    typedef PlaneMfma<R> M;
    constexpr int NB = kDwPairs / M::COLS;               // column blocks of a tile's pairs
    typedef Oct<MODE != kStrided> XOct;
    typedef Oct<true> YOct;
    __shared__ u32x4 sU[kDwOcts * S::RP];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Consecutive ids: the tiles of one col-group (one L2).
    const int32_t L = xcd_remap(int32_t(blockIdx.x), a.total);
    const int32_t tile = L % a.tiles, rowset = L / a.tiles;
    const int32_t g = rowset / (N / R), r0 = (rowset - g * (N / R)) * R;   // col-group, its first row here
    const int32_t zb = max(0, min(a.P[g], a.t)), cnt = max(zb, min(a.P[g + 1], a.t)) - zb;
    const int32_t pairs = cnt * a.KK, pr0 = tile * kDwPairs;
    if (pr0 >= pairs) return;                            // (uniform: before any barrier)
    const uint16_t* const x = static_cast<const uint16_t*>(a.x);
    const uint16_t* const dy = static_cast<const uint16_t*>(a.dy);
    const int32_t HW = a.H * a.W, HWo = a.Ho * a.Wo;

    // ---- Staging roles: octet `lane` of rows wave + kDwRS u.
    const int oct = lane, srow = wave;
    int32_t xoff[S::UX], xtap[S::UX];                    // element offset of (channel, tap), or -1 for no pair
#pragma unroll
    for (int u = 0; u < S::UX; ++u) {
        const int32_t pr = pr0 + srow + kDwRS * u;
        const int32_t tap = pr / max(cnt, 1), zi = pr - tap * cnt;
        const int32_t c = pr < pairs ? a.I[zb + zi] : -1;
        const int32_t q = tap / a.kw, r = tap - q * a.kw;
        xtap[u] = pr < pairs && c >= 0 && c < a.m ? (q << 8) | r : -1;
        xoff[u] = c * HW + q * a.W + r;
    }
    // The octet's place: image, output row, octet of the row; advanced by one
    // chunk per load.
    int32_t b, oh, k;
    {
        const int32_t p = oct, row = p / a.noct;
        k = p - row * a.noct;
        b = row / a.Ho;
        oh = row - b * a.Ho;
    }
    XOct xv[2][S::UX];
    YOct yv[2][S::UY];
    uint32_t xm[2][S::UX], ym[2];            // valid columns, one bit each
    int32_t xe[2][S::UX], ye[2][S::UY];      // element of an octet that crosses the tensor's ends, or -1
    auto load = [&](auto SET) __attribute__((always_inline)) {
        constexpr int s = decltype(SET)::value;
        const bool in = b < a.batch;
        const int32_t left = a.Wo - 8 * k;               // columns of the row from this octet on
        ym[s] = in ? (left >= 8 ? 255u : (1u << left) - 1) : 0u;
        const int32_t yb = int32_t(uint32_t(b * a.n + g * N + r0) * uint32_t(HWo)) + oh * a.Wo + 8 * k;
#pragma unroll
        for (int u = 0; u < S::UY; ++u) {
            const int32_t row = srow + kDwRS * u;
            const bool ok = in && g * N + r0 + row < a.n;
            const int32_t at = ok ? yb + row * HWo : 0;
            ye[s][u] = ok && at > a.y_total - 8 ? at : -1;
            if (!ok) ye[s][u] = -2;                      // no such row: zeros
            load_oct(dy + min(at, a.y_total - 8), yv[s][u]);
        }
        const int32_t ih0 = oh * a.sh - a.ph, iw0 = 8 * k * a.sw - a.pw;
        const int32_t xb = int32_t(uint32_t(b) * uint32_t(a.m * HW)) + ih0 * a.W + iw0;
#pragma unroll
        for (int u = 0; u < S::UX; ++u) {
            bool ok = in && xtap[u] >= 0;
            uint32_t m = 255u;
            if constexpr (MODE != kFlat) {
                const int32_t ih = ih0 + (xtap[u] >> 8), iw = iw0 + (xtap[u] & 255);
                ok = ok && ih >= 0 && ih < a.H;
                if constexpr (MODE == kTap) {
                    const int32_t lo = max(0, min(-iw, 8)), hi = max(0, min(a.W - iw, 8));
                    m = ((1u << hi) - 1) & ~((1u << lo) - 1);
                } else {
                    m = 0;
#pragma unroll
                    for (int j = 0; j < 8; ++j) m |= uint32_t(uint32_t(iw + j * a.sw) < uint32_t(a.W)) << j;
                }
            }
            xm[s][u] = ok ? m : 0u;
            const int32_t at = ok ? xb + xoff[u] : 0;
            if constexpr (MODE == kStrided) {
                load_each(x, at, a.sw, a.x_total, xv[s][u].v);
            } else {
                xe[s][u] = ok && (at < 0 || at > a.x_total - 8) ? at : INT32_MIN;
                load_oct(x + max(0, min(at, a.x_total - 8)), xv[s][u]);
            }
        }
        // One chunk on.
        k += a.dk;
        int32_t carry = k >= a.noct;
        k -= carry ? a.noct : 0;
        oh += a.doh + carry;
        carry = oh >= a.Ho;
        oh -= carry ? a.Ho : 0;
        b += a.db + carry;
    };
    auto store = [&](auto SET) __attribute__((always_inline)) {
        constexpr int s = decltype(SET)::value;
#pragma unroll
        for (int u = 0; u < S::UX; ++u) {
            if constexpr (MODE != kStrided) {
                if (xe[s][u] != INT32_MIN) load_each(x, xe[s][u], 1, a.x_total, xv[s][u].v);
            }
            sU[oct * S::RP + srow + kDwRS * u] = masked(xv[s][u].v, xm[s][u]);
        }
#pragma unroll
        for (int u = 0; u < S::UY; ++u) {
            if (ye[s][u] >= 0) load_each(dy, ye[s][u], 1, a.y_total, yv[s][u].v);
            sU[oct * S::RP + kDwPairs + srow + kDwRS * u] = masked(yv[s][u].v, ye[s][u] == -2 ? 0u : ym[s]);
        }
    };

    // ---- Compute roles: each wave takes OPW octets of a chunk.
    const int kg = lane / M::COLS, col = lane % M::COLS;
    PlaneAcc<R, 1> acc[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[nb].zero();
    const u32x4* const lb = sU + (wave * S::OPW + kg) * S::RP + col;
    const u32x4* const la = lb + kDwPairs;
    auto multiply = [&]() __attribute__((always_inline)) {
        u32x4 af[S::STEPS][1], bf[S::STEPS][NB][1];
#pragma unroll
        for (int st = 0; st < S::STEPS; ++st) {
            af[st][0] = la[S::KG * st * S::RP];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) bf[st][nb][0] = lb[S::KG * st * S::RP + nb * M::COLS];
        }
#pragma unroll
        for (int st = 0; st < S::STEPS; ++st)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) acc[nb].template product<0>(af[st], bf[st][nb]);
    };
    typedef std::integral_constant<int, 0> Set0;
    typedef std::integral_constant<int, 1> Set1;
    load(Set0{});
    if (1 < a.chunks) load(Set1{});
    for (int32_t ch = 0; ch < a.chunks; ch += 2) {
        store(Set0{});
        __syncthreads();
        if (ch + 2 < a.chunks) load(Set0{});
        multiply();
        __syncthreads();
        if (ch + 1 >= a.chunks) break;
        store(Set1{});
        __syncthreads();
        if (ch + 3 < a.chunks) load(Set1{});
        multiply();
        __syncthreads();
    }

    // ---- Sums over the waves of a pair block, in wave order, and the store:
    // entry (row, pair) at dD[z][row][tap].  A thread sums one entry at most.
    float* const part = reinterpret_cast<float*>(sU);
    constexpr int E = NB * M::ACC * 64;                  // entries of a wave's tile
    static_assert(E <= kDwThreads, "one entry per thread");
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int r = 0; r < M::ACC; ++r) part[wave * E + (nb * M::ACC + r) * 64 + lane] = acc[nb].value(r);
    __syncthreads();
    auto entry_row = [&](int e) { return r0 + M::row(e & 63, (e >> 6) % M::ACC); };
    auto entry_pair = [&](int e) { return pr0 + ((e >> 6) / M::ACC) * M::COLS + (e & 63) % M::COLS; };
    auto put = [&](int32_t row, int32_t pr, float v) __attribute__((always_inline)) {
        const int32_t tap = pr / cnt, z = zb + pr - tap * cnt;
        a.dD[(int64_t(z) * N + row) * a.KK + tap] = v;
    };
    bool bad = false;                                    // to be computed again
    if (tid < E) {
        float v = 0.f;
#pragma unroll
        for (int j = 0; j < kDwWaves; ++j) v += part[j * E + tid];
        const int32_t row = entry_row(tid), pr = entry_pair(tid);
        const bool real = g * N + row < a.n;
        bad = pr < pairs && real && not_finite(v);
        if (pr < pairs && !bad) put(row, pr, real ? v : 0.f);
    }
    if (!__syncthreads_or(bad)) return;

    // Again in plain fp32 over the pixels inside the image: a wave per entry, a
    // lane per octet, and the lanes' sums in a fixed order.  A sum that is NaN
    // stays NaN.
    int32_t* const list = reinterpret_cast<int32_t*>(sU);
    if (tid == 0) list[0] = 0;
    __syncthreads();
    if (bad) list[1 + atomicAdd(&list[0], 1)] = tid;
    __syncthreads();
    const int32_t left = list[0], rows = a.batch * a.Ho;
#pragma unroll 1
    for (int32_t i = wave; i < left; i += kDwWaves) {
        const int e = list[1 + i];
        const int32_t row = entry_row(e), pr = entry_pair(e);
        const int32_t tap = pr / cnt, c = a.I[zb + pr - tap * cnt], q = tap / a.kw, r = tap - q * a.kw;
        float v = 0.f;
        if (c >= 0 && c < a.m) {
#pragma unroll 1
            for (int32_t p0 = 0; p0 < a.chunks * kDwOcts && !__any(v != v); p0 += 64) {
                const int32_t p = p0 + lane, orow = p / a.noct, bb = orow / a.Ho, oo = orow - bb * a.Ho;
                const int32_t ih = oo * a.sh - a.ph + q, w0 = 8 * (p - orow * a.noct);
                if (orow >= rows || ih < 0 || ih >= a.H) continue;
                const uint16_t* const yr = dy + (int64_t(bb) * a.n + g * N + row) * HWo + oo * a.Wo;
                const uint16_t* const xr = x + (int64_t(bb) * a.m + c) * HW + ih * a.W;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int32_t ow = w0 + j, iw = ow * a.sw - a.pw + r;
                    if (ow < a.Wo && iw >= 0 && iw < a.W) v = fmaf(to_f32(yr[ow]), to_f32(xr[iw]), v);
                }
            }
        }
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) v += __shfl_xor(v, d);
        if (lane == 0) put(row, pr, v);
    }
}

int64_t dw_tiles(int32_t m, int32_t KK) { return (int64_t(m) * KK + kDwPairs - 1) / kDwPairs; }
// Most workgroups of a launch (each row block of a col-group takes dw_tiles).
constexpr int64_t kDwMaxGrid = INT32_MAX / kDwThreads;

template <int N, int R, int MODE>
onexn_status launch_dw(DwArgs d, hipStream_t s) {
    const int64_t octs = int64_t(d.batch) * d.Ho * d.noct;
    d.chunks = int32_t((octs + kDwOcts - 1) / kDwOcts);
    d.tiles = int32_t(dw_tiles(d.m, d.KK));
    d.dk = kDwOcts % d.noct;
    d.drow = kDwOcts / d.noct;
    d.db = d.drow / d.Ho;
    d.doh = d.drow % d.Ho;
    d.total = d.G * (N / R) * d.tiles;
    hipLaunchKernelGGL((bwd_weight_bf16<N, R, MODE>), dim3(uint32_t(d.total)), dim3(kDwThreads), 0, s, d);
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return fail(ONEXN_ERR_HIP, "conv2d_bwd_weight: launch failed: %s", hipGetErrorString(err));
    return ONEXN_OK;
}

bool dw_flat(const ConvArgs& a) { return a.KK == 1 && a.sh == 1 && a.sw == 1 && a.ph == 0 && a.pw == 0; }

// Whether a layer with strided columns, whose octets are loaded element by
// element, is faster here than on the general kernel.  us fitted to both over
// 1300 layers: 0.07 per octet here, less where a col-group's pairs do not fill a
// tile, more by a sixth per column that a short row lacks; there, per pixel, by
// the col-group's rows, and more with the (block, tap) pairs, one workgroup
// each.  General and here, at stride 2: 64 -> 64 1x1 at 7x7, batch 64: N = 16
// 12.0 and 33.2, N = 32 20.0 and 33.2; at 28x28, batch 64: N = 16 158 and 133, N
// = 32 438 and 133; 256 -> 256 1x1 at 7x7, batch 8, N = 16: 13.0 and 7.7; 64 ->
// 64 3x3 at 9x9, batch 64, N = 16: 23.8 and 33.2; 32 -> 8 3x3 at 28x28, batch 64,
// N = 32: 78 and 130.  The worst choices of the fit, both taken here: 32 -> 8 1x1
// at 56x56, batch 64, N = 16, 348 against 265; 256 -> 64 3x3 at 7x7, batch 64, N
// = 16, 54 against 42.
bool dw_strided_preferred(const ConvArgs& a, int32_t batch) {
    const double px = double(batch) * a.HWo, pairs = double(a.t) * a.KK, octs = double(batch) * a.Ho * ((a.Wo + 7) / 8);
    const double rows = std::min(a.N, a.n), fill = std::min(1.0, pairs / a.G / kDwPairs);
    const double here = 2.8 + octs * (0.033 + 0.0395 * fill) * (1 + 0.15 * std::max(0, 8 - a.Wo));
    const double per_px = rows * std::max(0.0005 * (1 + 2 / rows), pairs * 0.53e-6);
    // (It reads its operands once per pair: slower when an L2 does not hold them.)
    const double mb = 2e-6 * batch * (double(a.m) * a.H * a.W + double(a.n) * a.HWo);
    const double far = 1 + std::min(1.0, std::max(0.0, mb - 3) / 4);
    const double general = 4.5 + pairs * 0.00015 * rows + px * far * (a.Wo < 5 ? 0.8 : 1.0) * per_px;
    return here < general;
}

}  // namespace

bool bwd_weight_bf16_applies(const ConvArgs& a, onexn_dtype xdt, int32_t batch) {
    if (a.N != 16 && a.N != 32) return false;
    if (batch < 1 || a.t < 1 || xdt != ONEXN_BF16) return false;
    // An octet is read whole inside its tensor.
    if (int64_t(batch) * a.m * a.H * a.W < 8 || int64_t(batch) * a.n * a.HWo < 8) return false;
    if (a.G * dw_tiles(a.m, a.KK) > kDwMaxGrid) return false;
    // Rows of few columns waste most of their octet.
    if ((dw_flat(a) ? a.HWo : a.Wo) < 4) return false;
    return a.sw == 1 || tuning(kTuneBwdKernel) == 4 || dw_strided_preferred(a, batch);
}

onexn_status launch_bwd_weight_bf16(const ConvArgs& a, int32_t batch, const void* x, const void* dy, float* dD,
                                    hipStream_t s) {
    DwArgs d{};
    d.P = a.P;
    d.I = a.I;
    d.x = x;
    d.dy = dy;
    d.dD = dD;
    d.m = a.m;
    d.n = a.n;
    d.G = a.G;
    d.t = a.t;
    d.KK = a.KK;
    d.kw = a.kw;
    d.batch = batch;
    d.H = a.H;
    d.W = a.W;
    d.Ho = a.Ho;
    d.Wo = a.Wo;
    d.sh = a.sh;
    d.sw = a.sw;
    d.ph = a.ph;
    d.pw = a.pw;
    if (dw_flat(a)) {
        d.H = d.Ho = 1;
        d.W = d.Wo = a.HWo;
    }
    d.noct = (d.Wo + 7) / 8;
    d.x_total = batch * a.m * a.H * a.W;
    d.y_total = batch * a.n * a.HWo;
    auto by_mode = [&](auto MODE) {
        constexpr int m = decltype(MODE)::value;
        if (a.N == 16) return launch_dw<16, 16, m>(d, s);
        // Half the rows per workgroup where the halves still fit three
        // quarters of the compute units (a workgroup fills one): 256 -> 512 1x1
        // at 28x28, batch 32 (72 tiles) 57 us against 68; 256 -> 128 at 14x14,
        // batch 64 (18) 33 against 41; but 1000 -> 200 at 7x7 (112) 27 against
        // 19 and 256 -> 1024 at 14x14 (144) 65 against 44.
        const int64_t tiles = (int64_t(a.t) * a.KK + kDwPairs - 1) / kDwPairs + a.G / 2;
        const bool half = 8 * tiles < 3 * int64_t(device_cu_count()) && 2 * a.G * dw_tiles(a.m, a.KK) <= kDwMaxGrid;
        return half ? launch_dw<32, 16, m>(d, s) : launch_dw<32, 32, m>(d, s);
    };
    if (dw_flat(a)) return by_mode(std::integral_constant<int, kFlat>{});
    if (a.sw == 1) return by_mode(std::integral_constant<int, kTap>{});
    return by_mode(std::integral_constant<int, kStrided>{});
}

}  // namespace onexn
