// Input gradient of a bf16 1x1 layer, NCHW, N >= 8, any stride and padding,
// on the matrix cores: dX = Omega-bar^T dY as a dense contraction over the
// output channels (zero weights where pruned).
//
// Paper: Lin et al., "1xN Pattern for Pruning Convolutional Neural Networks"
// (arXiv 2105.14713), Sec. 3.4 (Eq. 7) and Sec. 4.1 (fine-tuning with the
// pattern fixed).
//
// Work.  A workgroup of four waves computes 32 WM input channels x 256 / WM
// pixels in chunks of 4 WM octets of output channels (WM = 4: 128 x 64, 128
// channels a chunk; WM = 2: 64 x 128, 64).  Each thread stages one octet of
// four pixels (eight 8-byte loads, or four times eight single values where
// images are not whole quads) and WM^2 / 2 octets of weights, which are
// contiguous in D, and holds them one chunk ahead in registers; the
// wave then multiplies 16 (8) times per barrier pair.  LDS as in
// conv_planes.hip: 16-byte octets, pixels by residue modulo 4.
//
// Strided layers: the output pixel (oh, ow) feeds input pixel (oh*s - p, ow*s
// - p) only; the other input pixels are multiplied as zeros.
//
// What bounds it: the latency of a chunk's loads.  256 -> 1024 at 14x14, batch
// 64, N = 32: 2780 us on the general kernel, 50 in chunks of 32 channels, 34
// here.
//
// An output that is not finite is computed again over the kept blocks alone (a
// pruned zero times an infinity is NaN), four rows of a lane's pixel at a time:
// the same layer takes 1250 us with a NaN or an infinity in dY, 350 with
// nothing else in it (one output at a time: 2570 and 2730).

#include <algorithm>

#include "lds_copy.h"
#include "planes.h"

namespace onexn {
namespace {

constexpr int kBfThreads = 256;
constexpr int kBfMaxG = 512;         // col-groups (each with WM runs in LDS)

struct BfArgs {
    const int32_t* P;
    const int32_t* I;
    const uint16_t* D;
    const uint16_t* dy;
    void* dx;
    int32_t N, G, t, n, m;
    int32_t H, W, Ho, Wo;            // input (dX) and output (dY) images
    int32_t batch, s, ph, pw;
    int32_t rblocks, total;
};

template <int WM> struct BfShape {
    static constexpr int ROWS = 32 * WM, NB = 2, TP = (4 / WM) * NB * 32;
    static constexpr int OCT = 4 * WM, QUADS = TP / 4;
    static constexpr int QX = QUADS + 4, XU = 4 * QX;    // units of a pixel residue, of an octet
    static constexpr int WP = ROWS + 4;                  // units of an octet's weights
    static constexpr int UW = ROWS * OCT / kBfThreads;
    static_assert(NB == 2 && QUADS * OCT == kBfThreads && QX % 16 == 4 && WP % 16 == 4, "one quad per thread, no conflicts");
};

template <int WM, bool kQuad, typename TY>
__global__ void __launch_bounds__(kBfThreads, 3) bwd_data_pw_bf16(BfArgs a) {
    typedef BfShape<WM> S;
    typedef PlaneMfma<32> M;
    __shared__ u32x4 sX[S::OCT * S::XU];
    __shared__ u32x4 sW[S::OCT * S::WP];
    __shared__ int32_t sFirst[kBfMaxG * WM];
    __shared__ uint32_t sMask[kBfMaxG * WM];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Consecutive ids: the channel blocks of one pixel tile (one L2).
    const int32_t L = xcd_remap(int32_t(blockIdx.x), a.total);
    const int32_t rb = L % a.rblocks, p0 = (L / a.rblocks) * S::TP, c0 = rb * S::ROWS;
    const int32_t HW = a.H * a.W, HWo = a.Ho * a.Wo, npx = a.batch * HW;

    // ---- Index: of col-group g and 32-channel tile w, the first kept block
    // in the tile and the mask of its channels.
    for (int32_t i = tid; i < a.G * WM; i += kBfThreads) {
        const int32_t g = i / WM, cb = c0 + 32 * (i - g * WM);
        const int32_t lo = max(0, min(a.P[g], a.t)), hi = max(lo, min(a.P[g + 1], a.t));
        const int32_t first = lo < hi ? lower_entry(a.I, lo, hi, cb) : lo;
        uint32_t mask = 0;
#pragma unroll
        for (int k = 0; k < 32; ++k) {
            const int32_t c = first + k < hi ? a.I[first + k] : INT32_MAX;
            if (c >= cb && c < cb + 32 && c < a.m) mask |= 1u << (c - cb);
        }
        sFirst[i] = first;
        sMask[i] = mask;
    }

    // ---- Staging: octet xoct of the quad's pixels; element offset of dY at
    // channel 0, or -1 where the pixel takes nothing.
    const int xoct = tid / S::QUADS, quad = tid % S::QUADS;
    int32_t xo[kQuad ? 1 : 4];
#pragma unroll
    for (int k = 0; k < (kQuad ? 1 : 4); ++k) {
        const int32_t p = p0 + 4 * quad + k, b = p / HW, hw = p - b * HW;
        if constexpr (kQuad) {
            xo[k] = p < npx ? b * a.n * HWo + hw : -1;
        } else {
            const int32_t ih = hw / a.W, uh = ih + a.ph, uw = hw - ih * a.W + a.pw;
            const int32_t oh = uh / a.s, ow = uw / a.s;
            xo[k] = p < npx && oh * a.s == uh && ow * a.s == uw && oh < a.Ho && ow < a.Wo
                        ? b * a.n * HWo + oh * a.Wo + ow : -1;
        }
    }
    u32x2 xq[8];
    u32x4 wq[S::UW];
    const __amdgpu_buffer_rsrc_t rD = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t*>(a.D), 0, __builtin_amdgcn_readfirstlane(a.t * a.N * 2), kRawBufferFlags);
    const int32_t nchunk = (a.n + 8 * S::OCT - 1) / (8 * S::OCT);
    auto load = [&](int32_t ch) __attribute__((always_inline)) {
        const int32_t o0 = 8 * (ch * S::OCT + xoct);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int32_t at = min(o0 + j, a.n - 1) * HWo;
            if constexpr (kQuad) {
                __builtin_memcpy(&xq[j], a.dy + max(xo[0], 0) + at, 8);
            } else {
#pragma unroll
                for (int k = 0; k < 2; ++k)
                    xq[j][k] = uint32_t(a.dy[max(xo[2 * k], 0) + at]) | (uint32_t(a.dy[max(xo[2 * k + 1], 0) + at]) << 16);
            }
        }
#pragma unroll
        for (int u = 0; u < S::UW; ++u) {
            // Four octets of a row next to each other: 64 contiguous bytes of D at N = 32.
            const int32_t i = (tid + kBfThreads * u) >> 2;
            const int32_t row = i % S::ROWS, o = 8 * (ch * S::OCT + 4 * (i / S::ROWS) + (tid & 3));
            const int32_t g = o / a.N, run = min(g, a.G - 1) * WM + row / 32;
            const uint32_t mask = sMask[run];
            const int32_t z = sFirst[run] + __popc(mask & ((1u << (row & 31)) - 1));
            const bool kept = (g < a.G) & ((mask >> (row & 31)) & 1);
            wq[u] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(
                rD, kept ? (z * a.N + o - g * a.N) * 2 : int32_t(kBufferOutOfRange), 0, 0));
        }
    };
    auto store = [&](int32_t ch) __attribute__((always_inline)) {
        const int32_t o0 = 8 * (ch * S::OCT + xoct);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            u32x4 p;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const uint32_t v = __builtin_amdgcn_perm(xq[2 * w + 1][k / 2], xq[2 * w][k / 2],
                                                         k & 1 ? 0x07060302u : 0x05040100u);
                // Channels past n were read from the last one.
                const uint32_t there = (o0 + 2 * w < a.n ? 0xffffu : 0u) | (o0 + 2 * w + 1 < a.n ? 0xffff0000u : 0u);
                p[w] = xo[kQuad ? 0 : k] >= 0 ? v & there : 0u;
            }
            sX[xoct * S::XU + k * S::QX + quad] = p;
        }
#pragma unroll
        for (int u = 0; u < S::UW; ++u) {
            const int32_t i = (tid + kBfThreads * u) >> 2;
            sW[(4 * (i / S::ROWS) + (tid & 3)) * S::WP + i % S::ROWS] = wq[u];
        }
    };

    const int wm = wave % WM, wn = wave / WM, kg = lane >> 5, col = lane & 31;
    PlaneAcc<32, 1> acc[S::NB];
    const u32x4* xl[S::NB];
#pragma unroll
    for (int nb = 0; nb < S::NB; ++nb) {
        acc[nb].zero();
        const int32_t i = (wn * S::NB + nb) * 32 + col;
        xl[nb] = sX + kg * S::XU + (i & 3) * S::QX + (i >> 2);
    }
    const u32x4* const wl = sW + kg * S::WP + 32 * wm + col;
    __syncthreads();
    load(0);
    for (int32_t ch = 0; ch < nchunk; ++ch) {
        store(ch);
        __syncthreads();
        if (ch + 1 < nchunk) load(ch + 1);
#pragma unroll
        for (int st = 0; st < S::OCT / 2; ++st) {
            const u32x4 af[1] = {wl[2 * st * S::WP]};
#pragma unroll
            for (int nb = 0; nb < S::NB; ++nb) {
                const u32x4 bf[1] = {xl[nb][2 * st * S::XU]};
                acc[nb].template product<0>(af, bf);
            }
        }
        __syncthreads();
    }

    // ---- Store.
    bool bad = false;
#pragma unroll
    for (int nb = 0; nb < S::NB; ++nb)
#pragma unroll
        for (int r = 0; r < M::ACC; ++r) bad |= not_finite(acc[nb].value(r));
    bad = __any(bad);
    // Stores column block nb but for the rows in `skip`.
    auto store_block = [&](int nb, uint32_t skip) __attribute__((always_inline)) {
        const int32_t p = p0 + (wn * S::NB + nb) * 32 + col;
        if (p >= npx) return;
        const int32_t b = p / HW, hw = p - b * HW;
        TY* const yp = static_cast<TY*>(a.dx) + int64_t(b) * a.m * HW + hw;
#pragma unroll
        for (int r = 0; r < M::ACC; ++r) {
            const int32_t c = c0 + 32 * wm + M::row(lane, r);
            if (c < a.m && !((skip >> r) & 1)) yp[int64_t(c) * HW] = from_f32<TY>(acc[nb].value(r));
        }
    };
    if (!bad) {
#pragma unroll
        for (int nb = 0; nb < S::NB; ++nb) store_block(nb, 0);
        return;
    }
    // Outputs that are not finite, four rows of a column block together (more
    // cost the kernel registers), until all of them are NaN, which they then stay.
    uint32_t again[S::NB];
#pragma unroll
    for (int nb = 0; nb < S::NB; ++nb) {
        again[nb] = 0;
#pragma unroll
        for (int r = 0; r < M::ACC; ++r)
            again[nb] |= uint32_t(not_finite(acc[nb].value(r)) && c0 + 32 * wm + M::row(lane, r) < a.m) << r;
        if (p0 + (wn * S::NB + nb) * 32 + col >= npx) again[nb] = 0;
        store_block(nb, again[nb]);
    }
#pragma unroll 1
    for (int four = 0; four < S::NB * M::ACC / 4; ++four) {
        const int nb = four / (M::ACC / 4), q4 = 4 * (four - nb * (M::ACC / 4));
        const uint32_t rows = ((nb == 0 ? again[0] : again[1]) >> q4) & 15;
        if (!__any(rows != 0)) continue;
        const int32_t p = p0 + (wn * S::NB + nb) * 32 + col;
        const int32_t b = p / HW, hw = p - b * HW, uh = hw / a.W + a.ph, uw = hw % a.W + a.pw;
        const int32_t oh = uh / a.s, ow = uw / a.s;
        const bool in = rows != 0 && oh * a.s == uh && ow * a.s == uw && oh < a.Ho && ow < a.Wo;
        const uint16_t* const dyp = a.dy + int64_t(b) * a.n * HWo + oh * a.Wo + ow;
        const int row0 = M::row(lane, q4);               // the four are consecutive
        float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int32_t g = 0; g < a.G; ++g) {
            const uint32_t mask = sMask[g * WM + wm];
            const int32_t first = sFirst[g * WM + wm];
            if (!mask) continue;
            bool open = false;
#pragma unroll
            for (int r = 0; r < 4; ++r) open |= ((rows >> r) & 1) && v[r] == v[r];
            if (!__any(in && open)) break;
#pragma unroll 1
            for (int32_t k = 0; k < min(a.N, a.n - g * a.N) && in; ++k) {
                const float xf = to_f32(dyp[int64_t(g * a.N + k) * HWo]);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int rr = row0 + r;
                    const int64_t z = first + __popc(mask & ((1u << rr) - 1));
                    if ((mask >> rr) & 1) v[r] = fmaf(xf, to_f32(a.D[z * a.N + k]), v[r]);
                }
            }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int32_t c = c0 + 32 * wm + row0 + r;
            if ((rows >> r) & 1) static_cast<TY*>(a.dx)[(int64_t(b) * a.m + c) * HW + hw] = from_f32<TY>(v[r]);
        }
    }
}

constexpr int kBfFewM = 64;          // input channels up to which WM is 2

// Workgroups of a launch (32 wm input channels x 256 / wm pixels each).
int64_t bf_grid(int wm, int32_t batch, int32_t H, int32_t W, int32_t m) {
    const int64_t px = 256 / wm, rows = 32 * wm;
    return (int64_t(batch) * H * W + px - 1) / px * ((m + rows - 1) / rows);
}

template <int WM, bool kQuad, typename TY>
onexn_status launch_bf(BfArgs a, hipStream_t s) {
    typedef BfShape<WM> S;
    a.rblocks = (a.m + S::ROWS - 1) / S::ROWS;
    a.total = int32_t(bf_grid(WM, a.batch, a.H, a.W, a.m));
    hipLaunchKernelGGL((bwd_data_pw_bf16<WM, kQuad, TY>), dim3(uint32_t(a.total)), dim3(kBfThreads), 0, s, a);
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return fail(ONEXN_ERR_HIP, "conv2d_bwd_data: launch failed: %s", hipGetErrorString(err));
    return ONEXN_OK;
}

}  // namespace

bool bwd_data_pw_bf16_applies(const ConvArgs& a, onexn_dtype wdt, int32_t batch) {
    if (bf_grid(a.m <= kBfFewM ? 2 : 4, batch, a.H, a.W, a.m) > INT32_MAX / kBfThreads) return false;
    // A chunk is 64 output channels: layers of few, over few pixels, take less on
    // the general kernel.  32 -> 8 at 7x7, batch 16, N = 8: 7.3 us there, 10.0
    // here; 28x28, batch 16: 10.9 and 8.2; 16 -> 16 at 7x7: 10.4 and 9.0.
    // (Its grid takes 65535 channels.)
    if (a.n <= 8 && a.m <= 65535 && int64_t(batch) * a.H * a.W <= 8192) return false;
    return wdt == ONEXN_BF16 && a.KK == 1 && a.N >= 8 && a.sh == a.sw && a.G <= kBfMaxG &&
           reinterpret_cast<uintptr_t>(a.D) % 16 == 0 && int64_t(a.t) * a.N * 2 < (int64_t(1) << 31);
}

onexn_status launch_bwd_data_pw_bf16(const ConvArgs& a, onexn_dtype dxdt, int32_t batch, const void* dy, void* dx,
                                     hipStream_t s) {
    BfArgs b{};
    b.P = a.P;
    b.I = a.I;
    b.D = static_cast<const uint16_t*>(a.D);
    b.dy = static_cast<const uint16_t*>(dy);
    b.dx = dx;
    b.N = a.N;
    b.G = a.G;
    b.t = a.t;
    b.n = a.n;
    b.m = a.m;
    b.H = a.H;
    b.W = a.W;
    b.Ho = a.Ho;
    b.Wo = a.Wo;
    b.batch = batch;
    b.s = a.sh;
    b.ph = a.ph;
    b.pw = a.pw;
    // A quad of neighbouring pixels lies in one image and is four neighbouring dY pixels.
    const bool quad = a.sh == 1 && a.ph == 0 && a.pw == 0 && a.H * a.W % 4 == 0;
    auto go = [&](auto ty) {
        typedef decltype(ty) TY;
        if (a.m <= kBfFewM) return quad ? launch_bf<2, true, TY>(b, s) : launch_bf<2, false, TY>(b, s);
        return quad ? launch_bf<4, true, TY>(b, s) : launch_bf<4, false, TY>(b, s);
    };
    if (dxdt == ONEXN_BF16) return go(uint16_t{});
    return go(float{});
}

}  // namespace onexn
