// Convolutions of a 1xN-pruned layer, NCHW, on the bf16 matrix instructions:
// forward (N in {16, 32}) and input gradient (N >= 8) of 3x3 layers, for bf16
// operands and, at stride 1, for fp32 ones as three bf16 planes (planes.h),
// and the forward of bf16 1x1 layers.
//
// Paper: Lin et al., "1xN Pattern for Pruning Convolutional Neural Networks"
// (arXiv 2105.14713), Sec. 3.4 (Eq. 8 over P, I, D) and Sec. 4.1 (fine-tuning
// with the pattern fixed).
//
// Work.  A workgroup of four waves computes a tile of destination pixels for
// one block of rows: forward, the N output channels of one col-group, over
// its kept blocks; input gradient, 32 input channels, over all output
// channels (Omega-bar's transpose as a dense operand, zero where pruned).  It
// walks the contraction in chunks of OCT octets (8 source channels each):
// the next chunk's values are loaded into registers while this one is
// multiplied, then cut into planes and stored to LDS between two barriers.
//
// LDS layout: a 16-byte unit holds the 8 channels of an octet at one position
// (or, for the weights, of one row), so a lane's MFMA fragment is one 16-byte
// read, consecutive lanes read consecutive units (no bank conflict), and the
// gather over channels costs nothing: an octet's 8 channels are whichever the
// col-group keeps.  The units are [octet][plane][position].
//
// Positions (3x3).  A tile is TP consecutive pixels of a strip of `tw` output
// columns, rows batch-major, so it may span images.  It stages every source
// row its pixels' windows touch, per image segment n + (K - 1) / s rows for n
// output rows, split by residue modulo the stride into planes of rows and
// columns, so that a tap (q, r) is one offset for all pixels and neighbouring
// pixels stay neighbours at any stride.  Positions outside the source read
// are zeroed once and never written.  A lane loads four neighbouring source
// columns of eight channels (eight 16-byte loads, 8-byte for bf16) and stores
// four positions: with one position per lane the loads were four times as
// many and bounded the bf16 kernel (256 -> 256 3x3 at 14x14, batch 64, N = 32:
// 38 -> 25 us; 238 on the generic kernel before).
//
// What bounds it, fp32: issue.  Per chunk of 16 channels a wave at N = 32 has
// 108 matrix products (3456 cycles) and, around them, some 430 vector
// instructions, most of them the cuts, of which the positions' go between the
// products; with two waves per SIMD that is 10300 of the 12000 cycles a chunk
// takes.  128 -> 128 3x3 at 28x28, batch 64, N = 32, ReLU: 88 us on the fp32
// instruction, 64 here; its input gradient 188 and 118.  bf16: the latency of
// a chunk's loads, one chunk ahead (two to four workgroups per unit).
//
// Input gradient of a strided layer: dY's pixels lie `dil` = stride apart in
// the staged tile, with zeros between them.  Of the nine taps a pixel then
// multiplies, one, two or four are not zero; the general kernel, which is the
// other choice for bf16, has no matrix cores (256 -> 256 3x3 stride 2 at 14x14,
// batch 64: 3474 us against 56).
//
// Non-finite results.  Planes of infinities are NaN, and the dense gradient
// multiplies pruned zeros; outputs that are not finite are computed again in
// plain fp32 over the kept blocks only, four rows of a lane's pixel at a time.
// us with a NaN or an infinity in the source, and with nothing else in it: fp32
// 128 -> 128 3x3 at 28x28, batch 64: 74, 412 and 99 (73 finite; one output at a
// time 4050, 4030 and 8800), its input gradient 620, 630 and 1220 (118; 7700 and
// 17400); bf16 input gradient of 256 -> 256 at 14x14: 2140, 2180 and 1400 (57;
// 16400 and 17700).

#include <algorithm>
#include <utility>

#include "lds_copy.h"
#include "planes.h"
#include "tile_div.h"

namespace onexn {
namespace {

struct PlArgs {
    const int32_t* P;
    const int32_t* I;
    const void* D;
    const void* x;            // source: forward x, gradient dY
    void* y;                  // destination: forward y, gradient dX
    int32_t NG, G, t;         // block length, col-groups, kept blocks
    int32_t C, R;             // source and destination channels
    int32_t H, W, Ho, Wo;     // source and destination images
    int32_t batch, s, ph, pw; // stride (1 for the gradient), padding (may be negative there)
    int32_t dil;              // distance of source pixels (the gradient's stride; 1 forward)
    int32_t rows;             // batch * Ho
    int32_t tw, tps, rblocks; // strip width, tiles per strip, row blocks
    int32_t total;
    const float* ep_scale;
    const float* ep_bias;
    int32_t ep_act;
};

constexpr int kPlThreads = 256;
// Col-groups of the gradient's index in LDS (fp32: two workgroups of 81792
// bytes fit a compute unit).
constexpr int kPlMaxRuns = 240;

// Entries (positions, weights) are stored by residue modulo 4: entry e at unit
// (e % 4) * Q + e / 4.  A lane writes four consecutive entries, so with plain
// order a write's lanes would lie 64 bytes apart (two to three of them on one
// bank); by residue they are consecutive, and with Q = 4 (positions) or 12
// (weights, read KK entries apart) modulo 16 reads conflict no more than before.
constexpr int up_to(int v, int mod16) { return v + (mod16 - v % 16 + 16) % 16; }
template <int Q> __device__ __forceinline__ int32_t unit_of(int32_t e) { return (e & 3) * Q + (e >> 2); }

// Shape of a kernel's instance.  QUAD: four neighbouring source columns per
// lane and load (3x3; 1x1 with stride 1, no padding and images of a multiple
// of four pixels), else one position per lane.
template <typename TX, int N, int K, int NBW, int XCAP, int UQ, bool QUAD>
struct PlShape {
    static constexpr int NP = Planes<TX>::NP;
    static constexpr int KK = K * K;
    static constexpr int OCT = K == 1 ? 4 : 2;           // octets per chunk
    static constexpr int TP = 4 * 32 * NBW;       // pixels per tile
    static constexpr int WPO = 4 / OCT;                  // waves that stage an octet
    static constexpr int XP = K == 1 ? TP : XCAP;        // staged positions (capacity)
    static constexpr int QX = up_to(XP / 4, 4);          // units of a residue's positions,
    static constexpr int XU = 4 * QX;                    // and of an octet's plane
    static constexpr int PER = QUAD ? 4 : 1;             // positions per item
    static constexpr int UX = K == 1 ? (TP + 64 * PER - 1) / (64 * PER) : UQ;   // items per thread
    static constexpr int XITEMS = 64 * WPO * UX;         // items per octet (capacity)
    static constexpr int WE = N * KK;                    // weight entries row * KK + tap
    static constexpr int QW = up_to(WE / 4, 12);
    static constexpr int WU = 4 * QW;
    // Steps: N = 16 multiplies taps in pairs (K = 32), the tenth with zeros.
    static constexpr int STEPS = K == 1 ? (N == 16 ? OCT / 4 : OCT / 2) : (N == 16 ? (KK + 1) / 2 : KK);
    static_assert(K != 1 || WPO == 1, "a wave per octet");
    static_assert(K == 1 || QUAD, "3x3 tiles are staged in quads");
};

__device__ __forceinline__ float load_f(__amdgpu_buffer_rsrc_t r, int32_t v, int32_t s, float*) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, v, s, 0));
}
__device__ __forceinline__ uint32_t load_f(__amdgpu_buffer_rsrc_t r, int32_t v, int32_t s, uint16_t*) {
    return __builtin_amdgcn_raw_buffer_load_b16(r, v, s, 0);
}
// Four consecutive values of a row as they are held between load and cut.
template <typename T> struct Quad;
template <> struct Quad<float> { typedef f32x4 type; };
template <> struct Quad<uint16_t> { typedef u32x2 type; };

__device__ __forceinline__ void load_quad(__amdgpu_buffer_rsrc_t r, int32_t v, int32_t s, f32x4& q) {
    q = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, v, s, 0));
}
__device__ __forceinline__ void load_quad(__amdgpu_buffer_rsrc_t r, int32_t v, int32_t s, u32x2& q) {
    q = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(r, v, s, 0));
}

template <typename F, int... Is>
__device__ __forceinline__ void for_each_index_impl(F&& f, std::integer_sequence<int, Is...>) {
    (f(std::integral_constant<int, Is>{}), ...);
}
template <int Count, typename F>
__device__ __forceinline__ void for_each_index(F&& f) {
    for_each_index_impl(f, std::make_integer_sequence<int, Count>{});
}

template <bool kDx, typename TX, typename TY, int N, int K, int NBW, int XCAP, int UQ, bool kS1, bool kQuad, bool kEp>
__global__ void __launch_bounds__(kPlThreads, 2) plane_conv(PlArgs a) {
    typedef PlShape<TX, N, K, NBW, XCAP, UQ, kQuad> S;
    typedef typename Planes<TX>::reg reg_t;
    typedef typename Quad<TX>::type quad_t;
    typedef PlaneMfma<N> M;
    constexpr int NP = S::NP, KK = S::KK, OCT = S::OCT, ES = int(sizeof(TX));
    constexpr int NB = NBW * 32 / M::COLS;               // MFMA column blocks per wave
    static_assert(!kDx || N == 32, "the gradient's row tiles are 32 channels");
    __shared__ u32x4 sX[OCT * NP * S::XU];
    __shared__ u32x4 sW[OCT * NP * S::WU];
    __shared__ float sEp[kEp ? 2 * N : 1];
    __shared__ int32_t sFirst[kDx ? kPlMaxRuns : 1];
    __shared__ uint32_t sMask[kDx ? kPlMaxRuns : 1];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int32_t L = xcd_remap(int32_t(blockIdx.x), a.total);
    const int32_t rb = L % a.rblocks, tile = L / a.rblocks;
    const int32_t strip = tile / a.tps, p0 = (tile - strip * a.tps) * S::TP;

    // ---- Tile geometry (all uniform).
    const int32_t st = kS1 ? 1 : a.s;
    const int32_t E = kS1 ? K - 1 : (K - 1) / st;        // source rows beyond the first per segment
    const int32_t PL = kS1 ? 1 : min(st, K);             // row and column planes
    const int32_t r0 = p0 / a.tw, r1 = min(a.rows - 1, (p0 + S::TP - 1) / a.tw);
    const int32_t b0 = r0 / a.Ho, oh0 = r0 - b0 * a.Ho, b1 = r1 / a.Ho;
    const int32_t rem0 = p0 - r0 * a.tw;                 // the tile's first pixel in row r0
    const int32_t RT = r1 - r0 + 1 + (b1 - b0 + 1) * E;
    // (Row pitch: a multiple of 4, so that a tap's row moves a position by whole units.)
    const int32_t CH = K == 1 ? a.tw : (a.tw + E + 3) / 4 * 4;
    const int32_t vpitch = PL * CH, qplane = RT * vpitch;
    const float itw = 1.f / float(a.tw), iHo = 1.f / float(a.Ho);
    const int64_t x_img = int64_t(a.C) * a.H * a.W;
    const int32_t chb = a.H * a.W * ES;                  // bytes between source channels
    const __amdgpu_buffer_rsrc_t rX = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char*>(static_cast<const char*>(a.x) + int64_t(b0) * x_img * ES), 0,
        __builtin_amdgcn_readfirstlane(int32_t(int64_t(b1 - b0 + 1) * x_img * ES)), kRawBufferFlags);
    const __amdgpu_buffer_rsrc_t rD = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<void*>(a.D), 0, __builtin_amdgcn_readfirstlane(int32_t(int64_t(a.t) * a.NG * KK * ES)),
        kRawBufferFlags);

    // ---- Staging roles: this wave stages octet `oct` of each chunk.  An
    // item's byte offset at channel 0 (from image b0) and its positions (-1:
    // none; four consecutive ones of a stride-1 item are the first and a mask).
    const int oct = wave % OCT, part = wave / OCT;
    int32_t xo[S::UX], xp[S::UX][S::PER];
    if constexpr (K == 1) {
#pragma unroll
        for (int u = 0; u < S::UX; ++u) {
            const int32_t i = S::PER * (lane + 64 * u);  // the tile's pixel
            const int32_t dr = small_div(rem0 + i, itw), db = small_div(oh0 + dr, iHo);
            const int32_t ih = (oh0 + dr - db * a.Ho) * st - a.ph, iw = (rem0 + i - dr * a.tw) * st - a.pw;
            const bool in = i < S::TP && r0 + dr < a.rows && ih >= 0 && ih < a.H && iw >= 0 && iw < a.W;
            xo[u] = in ? int32_t((int64_t(db) * x_img + ih * a.W + iw) * ES) : (kQuad ? 0 : int32_t(kBufferOutOfRange));
#pragma unroll
            for (int k = 0; k < S::PER; ++k) xp[u][k] = (kQuad ? in : i < S::TP) ? unit_of<S::QX>(i + k) : -1;
        }
    } else {
        // Source columns [wlo, whi) of the strip's windows in quads; the last
        // quad of a row moves back into the image.
        const int32_t w0 = strip * a.tw * st - a.pw;     // column of ci = 0 in column plane 0
        const int32_t dil = kDx ? a.dil : 1;
        const int32_t wlo = max(0, (w0 + dil - 1) / dil),
                      whi = max(wlo, min(a.W, kDx ? max(0, w0 + a.tw + E - 1 + dil) / dil : w0 + (a.tw + E - 1) * st + PL));
        const int32_t nq = (whi - wlo + 3) / 4, nrow = PL * RT;
        const float inq = 1.f / float(max(nq, 1)), iR = 1.f / float(RT), is = 1.f / float(a.Ho + E);
        const int32_t L0 = min(a.Ho - oh0, r1 - r0 + 1) + E;
#pragma unroll
        for (int u = 0; u < S::UX; ++u) {
            const int32_t i = lane + 64 * (part + S::WPO * u);
            const int32_t row = small_div(i, inq), col = min(wlo + 4 * (i - row * nq), a.W - 4);
            const int32_t qpl = kS1 ? 0 : small_div(row, iR), v = row - qpl * RT;
            const int32_t w = v - L0, dw = small_div(max(w, 0), is);
            const int32_t db = w < 0 ? 0 : 1 + dw, orow = w < 0 ? oh0 + v : w - dw * (a.Ho + E);
            const int32_t vh = orow * st - a.ph + qpl, ih = kDx ? vh / dil : vh;
            const bool in = i < nrow * nq && vh >= 0 && ih < a.H && ih * dil == vh;
            xo[u] = in ? int32_t((int64_t(db) * x_img + ih * a.W + col) * ES) : 0;
            const int32_t base = qpl * qplane + v * vpitch;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int32_t c = (col + k) * dil - w0;  // column among the strip's
                const int32_t ci = kS1 ? c : small_div(max(c, 0), 1.f / float(st)), cpl = c - ci * st;
                xp[u][k] = in && c >= 0 && cpl < PL && ci < a.tw + E ? unit_of<S::QX>(base + cpl * CH + ci) : -1;
            }
        }
    }

    // ---- Rows: a col-group's kept blocks (forward), or the index of the
    // blocks that keep this tile's channels (gradient): of col-group g, the
    // first such block and the mask of its channels.
    int32_t zb = 0, ze = 0, nchunk;
    const int32_t c0 = rb * N;
    if constexpr (kDx) {
        for (int32_t i = tid; i < a.G; i += kPlThreads) {
            const int32_t lo = max(0, min(a.P[i], a.t)), hi = max(lo, min(a.P[i + 1], a.t));
            const int32_t first = lo < hi ? lower_entry(a.I, lo, hi, c0) : lo;
            uint32_t mask = 0;
#pragma unroll
            for (int k = 0; k < 32; ++k) {
                const int32_t e = first + k;
                const int32_t c = e < hi ? a.I[e] : INT32_MAX;
                if (c >= c0 && c < c0 + 32 && c < a.R) mask |= 1u << (c - c0);
            }
            sFirst[i] = first;
            sMask[i] = mask;
        }
        nchunk = (a.C + 8 * OCT - 1) / (8 * OCT);
    } else {
        zb = max(0, min(a.P[rb], a.t));
        ze = max(zb, min(a.P[rb + 1], a.t));
        nchunk = (ze - zb + 8 * OCT - 1) / (8 * OCT);
        if constexpr (kEp) {
            if (tid < 2 * N) {
                const int32_t o = rb * N + tid % N;
                const float* p = tid < N ? a.ep_scale : a.ep_bias;
                sEp[tid] = p && o < a.R ? p[o] : (tid < N ? 1.f : 0.f);
            }
        }
    }
    // Positions that no item writes (padding) read as zeros.
    if constexpr (K != 1 || kQuad)
        for (int i = tid; i < OCT * NP * S::XU; i += kPlThreads) sX[i] = u32x4{0, 0, 0, 0};
    __syncthreads();

    // ---- Registers of the chunk in flight.  An octet's channels are read one
    // chunk ahead of its values, one per lane (-1: none, or past the col-group).
    // Weights: forward, one quad of the D row per lane; gradient, (row, tap)s.
    constexpr int UW = kDx ? (S::WE + 64 * S::WPO - 1) / (64 * S::WPO) : (S::WE / 4 + 64 * S::WPO - 1) / (64 * S::WPO);
    quad_t xq[kQuad ? S::UX : 1][8], wq[kDx ? 1 : UW][8];
    reg_t xv[kQuad ? 1 : S::UX][8], wv[kDx ? UW : 1][8];
    int32_t iv = -1;
    auto load_index = [&](int32_t ch) __attribute__((always_inline)) {
        if constexpr (!kDx) {
            const int32_t z = zb + ch * (8 * OCT) + 8 * oct + (lane & 7);
            iv = z < ze ? a.I[z] : -1;
        }
    };
    int32_t e0 = 0, co[8];                               // the octet's first entry, byte offsets of its channels,
    uint32_t none[8];                                    // all ones: no such entry
    uint32_t there[4];                                   // bf16: pairs of channels, ones where there is one
    auto begin_load = [&](int32_t ch) __attribute__((always_inline)) {
        e0 = ch * (8 * OCT) + 8 * oct;
        if constexpr (!kDx) iv = iv < a.C ? iv : -1;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int32_t c = kDx ? (e0 + j < a.C ? e0 + j : -1) : __builtin_amdgcn_readlane(iv, j);
            none[j] = uint32_t(min(c, 0) >> 31);
            co[j] = max(c, 0) * chb;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) there[k] = ~((none[2 * k] >> 16) | (none[2 * k + 1] << 16));
    };
    // Items of a chunk's load: positions, then weight entries.
    constexpr int ITEMS = S::UX + UW;
    const char* const xbase = static_cast<const char*>(a.x) + int64_t(b0) * x_img * ES;
    auto load_item = [&](auto I) __attribute__((always_inline)) {
        constexpr int i = decltype(I)::value;
        if constexpr (i < S::UX) {
            if constexpr (kQuad) {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    // (bf16 rows may start at any even address: a global load,
                    // which is not range-checked.)
                    if constexpr (ES == 4) load_quad(rX, int32_t(uint32_t(xo[i]) | none[j]), co[j], xq[i][j]);
                    else __builtin_memcpy(&xq[i][j], xbase + uint32_t(co[j]) + uint32_t(xo[i]), sizeof(quad_t));
                }
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    xv[i][j] = load_f(rX, int32_t(uint32_t(xo[i]) | none[j]), co[j], static_cast<TX*>(nullptr));
            }
        } else {
            constexpr int u = i - S::UX;
            const int32_t e = lane + 64 * (part + S::WPO * u);
            if constexpr (kDx) {
                const int32_t g = e0 / a.NG, ol = e0 - g * a.NG;
                const int32_t row = e / KK, tap = e - row * KK;
                const int32_t run = min(g, a.G - 1);
                const uint32_t mask = sMask[run];
                const int32_t z = sFirst[run] + __popc(mask & ((1u << (row & 31)) - 1));
                const bool kept = (e < S::WE) & (g < a.G) & ((mask >> (row & 31)) & 1);
                const int32_t at = kept ? ((z * a.NG + ol) * KK + (KK - 1 - tap)) * ES : int32_t(kBufferOutOfRange);
#pragma unroll
                for (int j = 0; j < 8; ++j) wv[u][j] = load_f(rD, at, j * KK * ES, static_cast<TX*>(nullptr));
            } else {
                const uint32_t eo = e < S::WE / 4 ? uint32_t(4 * e * ES) : kBufferOutOfRange;
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    load_quad(rD, int32_t(eo | none[j]), (zb + e0 + j) * (N * KK * ES), wq[u][j]);
            }
        }
    };
    // Cutting, in pieces of one pair of channels that go between the products
    // of the chunk being multiplied.  (A wave whose next product waits for the
    // matrix pipe holds the vector issue port, so two waves of a SIMD do not
    // overlap products with vector work; one wave's own instructions between
    // its products are free.)  Units: positions, then weights, 4 pieces each.
    constexpr int CX = S::UX * S::PER, CW = kDx ? UW : 4 * UW, ALL = 4 * (CX + CW);
    // (fp32: the positions only; with the weights the registers do not fit.)
    constexpr int PIECES = NP == 1 ? ALL : 4 * CX;
    u32x4 cx[CX][NP], cw[CW][NP];
    auto cut_piece = [&](auto I) __attribute__((always_inline)) {
        // A quad's pieces go pair by pair, so that loaded registers die early.
        constexpr int piece = decltype(I)::value, PX = S::PER, PW = kDx ? 1 : 4;
        if constexpr (piece < 4 * CX) {
            constexpr int u = piece / (4 * PX), k = piece / PX % 4, i = piece % PX, unit = u * PX + i;
            if constexpr (!kQuad) {
                cut_pair(xv[u][2 * k], xv[u][2 * k + 1], k, cx[unit]);
            } else if constexpr (ES == 4) {
                cut_pair(xq[u][2 * k][i], xq[u][2 * k + 1][i], k, cx[unit]);
            } else {
                // Channels that are not there (the last chunk) were read from channel 0.
                cx[unit][0][k] = __builtin_amdgcn_perm(xq[u][2 * k + 1][i / 2], xq[u][2 * k][i / 2],
                                                       i & 1 ? 0x07060302u : 0x05040100u) & there[k];
            }
        } else {
            constexpr int left = piece - 4 * CX, k = left / PW % 4, w = left / (4 * PW) * PW + left % PW;
            if constexpr (kDx) {
                cut_pair(wv[w][2 * k], wv[w][2 * k + 1], k, cw[w]);
            } else if constexpr (ES == 4) {
                cut_pair(wq[w / 4][2 * k][w % 4], wq[w / 4][2 * k + 1][w % 4], k, cw[w]);
            } else {
                cw[w][0][k] = __builtin_amdgcn_perm(wq[w / 4][2 * k + 1][(w % 4) / 2], wq[w / 4][2 * k][(w % 4) / 2],
                                                    w & 1 ? 0x07060302u : 0x05040100u);
            }
        }
    };
    auto store = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < CX; ++u) {
            const int32_t at = xp[u / S::PER][u % S::PER];
            if (at < 0) continue;
#pragma unroll
            for (int t = 0; t < NP; ++t) sX[(oct * NP + t) * S::XU + at] = cx[u][t];
        }
#pragma unroll
        for (int w = 0; w < CW; ++w) {
            // Entry of the octet's 8 x WE weights.
            const int32_t e = kDx ? lane + 64 * (part + S::WPO * w) : 4 * (lane + 64 * (part + S::WPO * (w / 4))) + w % 4;
            if (e >= S::WE) continue;
#pragma unroll
            for (int t = 0; t < NP; ++t) sW[(oct * NP + t) * S::WU + unit_of<S::QW>(e)] = cw[w][t];
        }
    };

    // ---- Compute roles.
    const int wn = wave;
    const int kg = lane / M::COLS, col = lane % M::COLS;
    int32_t xb[NB][K];                                   // unit of block nb's pixel at tap (0, r)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int32_t i = (wn * NB + nb) * M::COLS + col;
        if constexpr (K == 1) {
            xb[nb][0] = unit_of<S::QX>(i);
        } else {
            const int32_t dr = small_div(rem0 + i, itw), c = rem0 + i - dr * a.tw, rr = min(dr, r1 - r0);
            const int32_t base = (rr + small_div(oh0 + rr, iHo) * E) * vpitch + c;
#pragma unroll
            for (int r = 0; r < K; ++r) xb[nb][r] = unit_of<S::QX>(base + (kS1 ? r : (r % st) * CH + r / st));
        }
    }
    // Octet and tap of a lane's fragment entries: 3x3, N = 32: the lane half's
    // octet of every tap; N = 16: the quarter's octet (low bit) and tap of the
    // pair (high bit); 1x1: the step's octets in turn.
    const int koct = K == 1 ? kg : (kg & 1), ktap = K != 1 && N == 16 ? kg >> 1 : 0;
    int32_t tq[K];                                       // units of a tap's row
#pragma unroll
    for (int q = 0; q < K; ++q) tq[q] = (kS1 ? q * CH : (q % st) * qplane + (q / st) * vpitch) / 4;
    int32_t wb[K == 1 ? 1 : 4];                          // unit of the lane's row at taps 0 .. 3
#pragma unroll
    for (int t = 0; t < (K == 1 ? 1 : 4); ++t) wb[t] = unit_of<S::QW>(col * KK + t);
    PlaneAcc<N, NP> acc[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[nb].zero();
    const u32x4* const xl = sX + koct * NP * S::XU;
    const u32x4* const wl = sW + koct * NP * S::WU;

    // Fragments, read DIST groups of products ahead of their use.  fp32: a
    // group is one column block's six products; bf16: a step's products.
    constexpr int GB = NP == 1 ? NB : 1, GROUPS = S::STEPS * NB / GB, DIST = NP == 1 ? 2 : 1, SL = DIST + 1;
    u32x4 af[SL][NP], bf[SL][GB][NP];
    auto read_group = [&](auto G) __attribute__((always_inline)) {
        constexpr int g = decltype(G)::value, st = g * GB / NB, nb0 = g * GB % NB;
        constexpr int TS = N == 16 ? 2 : 1, t0 = TS * st, t1 = TS == 2 && t0 + 1 < KK ? t0 + 1 : t0;   // (3x3)
        if constexpr (nb0 == 0) {
#pragma unroll
            for (int t = 0; t < NP; ++t) {
                if constexpr (K == 1) {
                    af[st % SL][t] = wl[wb[0] + (st * (N == 16 ? 4 : 2) * NP + t) * S::WU];
                } else {
                    const int32_t u0 = wb[t0 % 4] + t0 / 4, u1 = wb[t1 % 4] + t1 / 4;
                    af[st % SL][t] = wl[(TS == 2 && ktap ? u1 : u0) + t * S::WU];
                    if constexpr (TS == 2 && t0 + 1 == KK)     // the tenth tap
                        if (ktap) af[st % SL][t] = u32x4{0, 0, 0, 0};
                }
            }
        }
#pragma unroll
        for (int i = 0; i < GB; ++i)
#pragma unroll
            for (int t = 0; t < NP; ++t) {
                const int nb = nb0 + i;
                if constexpr (K == 1) {
                    bf[g % SL][i][t] = xl[xb[nb][0] + (st * (N == 16 ? 4 : 2) * NP + t) * S::XU];
                } else {
                    const int32_t u0 = xb[nb][t0 % K] + tq[t0 / K], u1 = xb[nb][t1 % K] + tq[t1 / K];
                    bf[g % SL][i][t] = xl[(TS == 2 && ktap ? u1 : u0) + t * S::XU];
                    // (No zero weight times an infinity; fp32 checks its results.)
                    if constexpr (TS == 2 && t0 + 1 == KK && NP == 1)
                        if (ktap) bf[g % SL][i][t] = u32x4{0, 0, 0, 0};
                }
            }
    };

    load_index(0);
    if (nchunk > 0) {
        begin_load(0);
        for_each_index<ITEMS>([&](auto I) __attribute__((always_inline)) { load_item(I); });
        for_each_index<PIECES>([&](auto I) __attribute__((always_inline)) { cut_piece(I); });
    }
    load_index(1);
    // Products of a chunk, and the first of them after which a piece of the
    // next chunk is cut (its loads were issued before the first product).
    constexpr int MMAS = S::STEPS * NB * PlaneAcc<N, NP>::MMAS;
    constexpr int CUT0 = NP == 1 ? MMAS - 1 : MMAS * 2 / 5;
    for (int32_t ch = 0; ch < nchunk; ++ch) {
        for_each_index<ALL - PIECES>([&](auto I) __attribute__((always_inline)) {
            cut_piece(std::integral_constant<int, PIECES + decltype(I)::value>{});
        });
        store();
        __syncthreads();
        for_each_index<DIST>([&](auto G) __attribute__((always_inline)) { read_group(G); });
        begin_load(ch + 1);
        load_index(ch + 2);
        for_each_index<ITEMS>([&](auto I) __attribute__((always_inline)) { load_item(I); });
        for_each_index<GROUPS>([&](auto G) __attribute__((always_inline)) {
            constexpr int g = decltype(G)::value, st = g * GB / NB, nb0 = g * GB % NB;
            if constexpr (g + DIST < GROUPS) read_group(std::integral_constant<int, g + DIST>{});
            __builtin_amdgcn_sched_barrier(0);           // reads and loads go ahead of the products
            for_each_index<GB>([&](auto B) __attribute__((always_inline)) {
                for_each_index<PlaneAcc<N, NP>::MMAS>([&](auto Q) __attribute__((always_inline)) {
                    constexpr int i = decltype(B)::value, q = decltype(Q)::value;
                    acc[nb0 + i].template product<q>(af[st % SL], bf[g % SL][i]);
                    constexpr int mma = (st * NB + nb0 + i) * PlaneAcc<N, NP>::MMAS + q;
                    if constexpr (mma >= CUT0) {
                        constexpr int lo = (mma - CUT0) * PIECES / (MMAS - CUT0),
                                      hi = (mma + 1 - CUT0) * PIECES / (MMAS - CUT0);
                        for_each_index<hi - lo>([&](auto I) __attribute__((always_inline)) {
                            cut_piece(std::integral_constant<int, lo + decltype(I)::value>{});
                        });
                        if constexpr (NP > 1) __builtin_amdgcn_sched_barrier(0);   // pieces stay between products
                    }
                });
            });
            __builtin_amdgcn_sched_barrier(0);
        });
        __syncthreads();
    }

    // ---- Store.
    constexpr bool kCheck = kDx || NP > 1;
    bool bad = false;
    if constexpr (kCheck) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int r = 0; r < M::ACC; ++r) bad |= not_finite(acc[nb].value(r));
        bad = __any(bad);
    }
    const int32_t HWo = a.Ho * a.Wo;
    auto put = [&](TY* p, int rr, float v) __attribute__((always_inline)) {
        if constexpr (kEp) {
            v = fmaf(v, sEp[rr], sEp[N + rr]);
            if (a.ep_act == ONEXN_ACT_RELU) v = fmaxf(v, 0.f);
            else if (a.ep_act == ONEXN_ACT_RELU6) v = fminf(fmaxf(v, 0.f), 6.f);
        }
        if (sizeof(TY) == 4) store_out(p, from_f32<TY>(v));
        else *p = from_f32<TY>(v);
    };
    // Pixel of column block nb: image, row and column, or false.
    auto pixel = [&](int nb, int32_t& b, int32_t& oh, int32_t& ow) __attribute__((always_inline)) {
        const int32_t i = rem0 + (wn * NB + nb) * M::COLS + col;
        const int32_t dr = small_div(i, itw), db = small_div(oh0 + dr, iHo);
        b = b0 + db;
        oh = oh0 + dr - db * a.Ho;
        ow = strip * a.tw + i - dr * a.tw;
        return r0 + dr < a.rows && ow < a.Wo;
    };
    // Stores column block nb but for the rows in `skip`.
    auto store_block = [&](int nb, uint32_t skip) __attribute__((always_inline)) {
        int32_t b, oh, ow;
        if (!pixel(nb, b, oh, ow)) return;
        TY* const yp = static_cast<TY*>(a.y) + int64_t(b) * a.R * HWo + oh * a.Wo + ow;
#pragma unroll
        for (int r = 0; r < M::ACC; ++r) {
            const int rr = M::row(lane, r);
            const int32_t o = c0 + rr;
            if (o < a.R && !((skip >> r) & 1)) put(yp + int64_t(o) * HWo, rr, acc[nb].value(r));
        }
    };
    if (!bad) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) store_block(nb, 0);
        return;
    }
    if constexpr (kCheck) {
        // Outputs that are not finite: plain fp32 over the kept blocks (see the
        // top of the file), four rows of a column block together (more cost the
        // kernel registers), until all of them are NaN, which they then stay.
        uint32_t again[NB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            int32_t b, oh, ow;
            again[nb] = 0;
#pragma unroll
            for (int r = 0; r < M::ACC; ++r)
                again[nb] |= uint32_t(not_finite(acc[nb].value(r)) && c0 + M::row(lane, r) < a.R) << r;
            if (!pixel(nb, b, oh, ow)) again[nb] = 0;
            store_block(nb, again[nb]);
        }
        const TX* const D = static_cast<const TX*>(a.D);
#pragma unroll 1
        for (int four = 0; four < NB * M::ACC / 4; ++four) {
            const int nb = four / (M::ACC / 4), q4 = 4 * (four - nb * (M::ACC / 4));
            uint32_t rows = again[0];
#pragma unroll
            for (int i = 1; i < NB; ++i) rows = nb == i ? again[i] : rows;
            rows = (rows >> q4) & 15;
            if (!__any(rows != 0)) continue;
            int32_t b, oh, ow;
            pixel(nb, b, oh, ow);
            const TX* const x = static_cast<const TX*>(a.x) + int64_t(b) * x_img;
            const int32_t hb = oh * st - a.ph, wb = ow * st - a.pw, dil = kDx ? a.dil : 1;
            const int row0 = M::row(lane, q4);           // the four are consecutive
            float v[4] = {0.f, 0.f, 0.f, 0.f};
            auto open = [&]() __attribute__((always_inline)) {
                bool o = false;
#pragma unroll
                for (int r = 0; r < 4; ++r) o |= ((rows >> r) & 1) && v[r] == v[r];
                return __any(o);
            };
            int32_t at[KK];                              // source pixel under each tap, or -1
#pragma unroll
            for (int tap = 0; tap < KK; ++tap) {
                const int32_t vh = hb + tap / K, vw = wb + tap % K, ih = vh / dil, iw = vw / dil;
                const bool in = vh >= 0 && ih < a.H && vw >= 0 && iw < a.W && ih * dil == vh && iw * dil == vw;
                at[tap] = rows && in ? ih * a.W + iw : -1;
            }
            auto load = [&](int32_t c, float (&xf)[KK]) __attribute__((always_inline)) {
                const TX* const xc = x + int64_t(c) * a.H * a.W;
#pragma unroll
                for (int tap = 0; tap < KK; ++tap) xf[tap] = at[tap] >= 0 ? to_f32(xc[at[tap]]) : 0.f;
            };
            float xf[KK];
            if constexpr (kDx) {
#pragma unroll 1
                for (int32_t g = 0; g < a.G && open(); ++g) {
                    const uint32_t mask = sMask[g];
                    if (!mask) continue;
                    const TX* w[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        w[r] = D + int64_t(sFirst[g] + __popc(mask & ((1u << (row0 + r)) - 1))) * a.NG * KK;
                    const uint32_t kept = mask >> row0;
                    const int32_t lim = min(a.NG, a.C - g * a.NG);
#pragma unroll 1
                    for (int32_t i = 0; i < lim; ++i) {
                        load(g * a.NG + i, xf);
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            if (!((kept >> r) & 1)) continue;
#pragma unroll
                            for (int tap = 0; tap < KK; ++tap) {
                                const float p = fmaf(xf[tap], to_f32(w[r][i * KK + KK - 1 - tap]), v[r]);
                                v[r] = at[tap] >= 0 ? p : v[r];
                            }
                        }
                    }
                }
            } else {
#pragma unroll 1
                for (int32_t z = zb; z < ze && open(); ++z) {
                    const int32_t c = a.I[z];
                    if (c < 0 || c >= a.C) continue;
                    load(c, xf);
#pragma unroll
                    for (int r = 0; r < 4; ++r)
#pragma unroll
                        for (int tap = 0; tap < KK; ++tap)
                            v[r] = fmaf(xf[tap], to_f32(D[(int64_t(z) * N + row0 + r) * KK + tap]), v[r]);
                }
            }
            TY* const yp = static_cast<TY*>(a.y) + int64_t(b) * a.R * HWo + oh * a.Wo + ow;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if ((rows >> r) & 1) put(yp + int64_t(c0 + row0 + r) * HWo, row0 + r, v[r]);
        }
    }
}

// Strip width of a 3x3 tile of TP pixels whose staged positions fit `cap` and
// whose quads of source columns fit `items` (0: none does).  The fewest strips
// that fit: a narrower last strip leaves lanes idle.
int32_t pl_strip(int32_t TP, int32_t cap, int32_t items, const PlArgs& a, int32_t K) {
    if (a.W < 4) return 0;                               // a quad lies in one source row
    const int64_t E = (K - 1) / a.s, PL = std::min(a.s, K);
    for (int32_t k = std::max(1, a.Wo / cap); k <= a.Wo; ++k) {   // (wider strips than `cap` do not fit)
        const int32_t tw = (a.Wo + k - 1) / k;
        if (k > 1 && tw < 8) break;
        int64_t nr = TP % tw == 0 ? TP / tw : (TP - 2) / tw + 2;
        nr = std::min<int64_t>(nr, a.rows);
        const int64_t nimg = std::min<int64_t>(a.batch, nr < 2 ? 1 : (nr - 2) / a.Ho + 2);
        const int64_t rows = PL * (nr + nimg * E);
        const int64_t cols = std::min<int64_t>(a.W, ((tw + E - 1) * a.s + PL + a.dil - 1) / a.dil + (a.dil > 1 ? 1 : 0));
        if (rows * PL * ((tw + E + 3) / 4 * 4) <= cap && rows * ((cols + 3) / 4) <= items) return tw;
    }
    return 0;
}

template <bool kDx, typename TX, typename TY, int N, int K, int NBW, int XCAP, int UQ, bool kS1, bool kQuad,
          bool kEp>
onexn_status launch_plane(const PlArgs& a, hipStream_t stream) {
    hipLaunchKernelGGL((plane_conv<kDx, TX, TY, N, K, NBW, XCAP, UQ, kS1, kQuad, kEp>), dim3(uint32_t(a.total)),
                       dim3(kPlThreads), 0, stream, a);
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return fail(ONEXN_ERR_HIP, "conv2d: launch failed: %s", hipGetErrorString(err));
    return ONEXN_OK;
}

// The 3x3 tiles: pixels and staged positions.  Stride 1: 256 pixels, or 128
// for images whose 256-pixel tiles touch too many rows (below about 9x9) and
// for layers with few workgroups; strided: 128 pixels, of which the four
// parity planes stage up to seven positions each.
constexpr int kPx1 = 256, kCap1 = 528, kPxS = 128, kCapS = 400, kPx2 = 128, kCap2 = 912;

enum PlKind { kPlNone, kPlPoint, kPlPointQuad, kPlS1, kPlS1Small, kPlStrided };

// Sets the launch of tiles of TP pixels in strips of tw columns for blocks of
// `rows` rows; false if there is no such strip (tw = 0) or the grid is out of range.
bool pl_grid(PlArgs& a, int32_t TP, int32_t tw, int32_t rows) {
    if (tw < 1) return false;
    a.tw = tw;
    a.tps = int32_t((int64_t(a.rows) * tw + TP - 1) / TP);
    a.rblocks = (a.R + rows - 1) / rows;
    const int64_t total = int64_t((a.Wo + tw - 1) / tw) * a.tps * a.rblocks;
    if (total < 1 || total > INT32_MAX / kPlThreads) return false;
    a.total = int32_t(total);
    return true;
}

// Chooses the tile of a layer and sets its launch.
PlKind pl_choose(PlArgs& a, int32_t K, int32_t rows) {
    if (a.Ho > kDivMax || (K == 1 && a.Wo > kDivMax)) return kPlNone;   // divided by (3x3 rows: a strip's width)
    if (K == 1) {
        const bool dense = a.s == 1 && a.ph == 0 && a.pw == 0 && int64_t(a.H) * a.W % 4 == 0;
        return !pl_grid(a, kPx1, a.Wo, rows) ? kPlNone : dense ? kPlPointQuad : kPlPoint;
    }
    if (a.s == 1) {
        const int32_t big = pl_strip(kPx1, kCap1, 128, a, K), small = pl_strip(kPxS, kCapS, 128, a, K);
        if (pl_grid(a, kPx1, big, rows) && (!small || a.total > device_cu_count())) return kPlS1;
        return pl_grid(a, kPxS, small, rows) ? kPlS1Small : kPlNone;
    }
    return pl_grid(a, kPx2, pl_strip(kPx2, kCap2, 256, a, K), rows) ? kPlStrided : kPlNone;
}

template <bool kDx, typename TX, typename TY, int N, bool kEp>
onexn_status launch_kind(PlKind kind, const PlArgs& p, hipStream_t s) {
    if (kind == kPlS1) return launch_plane<kDx, TX, TY, N, 3, 2, kCap1, 1, true, true, kEp>(p, s);
    if (kind == kPlS1Small) return launch_plane<kDx, TX, TY, N, 3, 1, kCapS, 1, true, true, kEp>(p, s);
    if constexpr (sizeof(TX) == 2 && !kDx) {
        if (kind == kPlStrided) return launch_plane<kDx, TX, TY, N, 3, 1, kCap2, 2, false, true, kEp>(p, s);
        if (kind == kPlPointQuad) return launch_plane<kDx, TX, TY, N, 1, 2, 1, 1, true, true, kEp>(p, s);
        if (kind == kPlPoint) return launch_plane<kDx, TX, TY, N, 1, 2, 1, 1, false, false, kEp>(p, s);
    }
    return fail(ONEXN_ERR_UNSUPPORTED, "conv2d: no instance for this layer");
}

// Whether the limits that the kernel's 32-bit offsets assume hold.
bool pl_fits(const ConvArgs& a, int32_t batch, int64_t src_img, int es, int64_t dst_px) {
    // A tile of 256 pixels spans at most 257 images.
    if (std::min<int64_t>(batch, 257) * src_img * es >= (int64_t(1) << 31)) return false;
    // (Weights past the last block, never read, are addressed up to 64 blocks on.)
    if ((int64_t(a.t) + 64) * a.N * a.KK * es >= (int64_t(1) << 31)) return false;
    return dst_px < (int64_t(1) << 30);
}

PlArgs pl_args(const ConvArgs& a, int32_t batch) {
    PlArgs p{};
    p.P = a.P;
    p.I = a.I;
    p.D = a.D;
    p.NG = a.N;
    p.G = a.G;
    p.t = a.t;
    p.batch = batch;
    p.ep_scale = a.ep_scale;
    p.ep_bias = a.ep_bias;
    p.ep_act = a.ep_act;
    return p;
}

PlArgs pl_fwd_args(const ConvArgs& a) {
    const int32_t batch = a.npix / a.HWo;
    PlArgs p = pl_args(a, batch);
    p.x = a.x;
    p.y = a.y;
    p.C = a.m;
    p.R = a.n;
    p.H = a.H;
    p.W = a.W;
    p.Ho = a.Ho;
    p.Wo = a.Wo;
    p.s = a.sh;
    p.ph = a.ph;
    p.pw = a.pw;
    p.dil = 1;
    p.rows = batch * a.Ho;
    return p;
}

PlArgs pl_dx_args(const ConvArgs& a, int32_t batch, const void* dy, void* dx) {
    PlArgs p = pl_args(a, batch);
    p.x = dy;
    p.y = dx;
    p.C = a.n;
    p.R = a.m;
    p.H = a.Ho;
    p.W = a.Wo;
    p.Ho = a.H;
    p.Wo = a.W;
    p.s = 1;
    p.dil = a.sh;
    p.ph = a.kh - 1 - a.ph;
    p.pw = a.kw - 1 - a.pw;
    p.rows = batch * a.H;
    return p;
}

// Whether a bf16 1x1 layer is faster here than on the general kernel (tiles of
// 128 pixels, 256 where they are many).  A chunk of 32 kept blocks has little to
// multiply in a layer of few pixels or a short contraction, and a tile that spans
// images of a few pixels loads from as many places as it has images.  us, general and here, p = 0.5, at stride 1:
//   one-pixel images (samples of an FC layer), 2048 -> 1000, N = 32, batch 1:
//     74 and 69, 128: 104 and 122, 512: 105 and 176; 256 -> 256, N = 16, 512:
//     17.5 and 30.2; quads of 2x2 images, 64 -> 64, N = 16, batch 32: 6.6 and 7.1;
//   not quads, N = 16, 64 -> 64: 7x7, batch 1 6.8 and 8.1, 32 7.5 and 8.0; 57x57,
//     batch 8 12.1 and 11.2, 128 124 and 88; 128 -> 128, batch 1: 7x7 8.8 and
//     9.6, 15x15 9.6 and 9.0; 256 -> 256, 5x5, batch 32: 14.9 and 13.7.
// At stride 2, 28x28: 64 -> 256, N = 16, batch 64: 19.4 and 20.1; 128 -> 128,
// batch 32: N = 16 11.5 and 10.4, N = 32 11.3 and 11.2; 256 -> 256, N = 32,
// batch 1 17.1 and 15.7, 32 20.0 and 16.4.
bool pl_point_preferred(const ConvArgs& a, PlKind kind) {
    const double kept = double(a.t) / a.G, macs = double(a.npix) * a.t * a.N;
    if (kind == kPlPointQuad) {
        if (kept < 6 && a.npix <= 8192) return false;    // (3 -> 32 at 56x56, batch 1: 4.7 and 5.3)
        return a.HWo >= 16 || kept >= 56 || a.npix <= 32;
    }
    if (a.HWo < 16) return false;
    if (a.sh == 1) return (kept >= 56 && kept * a.npix >= 6000) || macs >= 5e7;
    return kept >= 112 || macs >= 2e8;
}

}  // namespace

bool planes_fwd_applies(const ConvArgs& a, onexn_dtype xdt, onexn_dtype ydt, onexn_layout layout) {
    if (layout != ONEXN_NCHW || (a.N != 16 && a.N != 32) || a.kh != a.kw || (a.kh != 1 && a.kh != 3)) return false;
    if (a.sh != a.sw) return false;
    const int es = xdt == ONEXN_F32 ? 4 : 2;
    const int32_t batch = a.npix / a.HWo;
    if (!pl_fits(a, batch, a.x_img, es, int64_t(batch) * a.Ho * (a.Wo + 8))) return false;
    if (reinterpret_cast<uintptr_t>(a.D) % (4 * es) != 0) return false;   // quads of weights
    if (xdt == ONEXN_F32 && (ydt != ONEXN_F32 || a.kh != 3 || a.sh != 1)) return false;
    PlArgs p = pl_fwd_args(a);
    const PlKind kind = pl_choose(p, a.kh, a.N);
    if (kind == kPlNone) return false;
    if (tuning(kTuneKernel) == 2) return true;
    if (xdt == ONEXN_BF16) {
        if (a.kh == 1) return pl_point_preferred(a, kind);
        // A chunk is 16 kept blocks, and a strided tile 128 pixels: image inputs of
        // a few channels take less on the general kernel.  us there and here, 3x3
        // stride 2 at 224x224, batch 8: 3 -> 32, N = 32 10.3 and 17.2, N = 16 22.5
        // and 24.2; 6 -> 32, N = 32 12.2 and 17.3, N = 16 36.4 and 24.2; 3 -> 32 at
        // 28x28, batch 64, N = 32: 7.5 and 6.9.
        const bool few = a.m <= 3 || (a.N == 32 && 2 * int64_t(a.t) < 7 * a.G);
        return a.sh == 1 || a.npix <= 2500 || !few;
    }
    // fp32: against the fp32 instruction's kernel, which spreads a layer's
    // chunks over all compute units.  Times in us fitted to layers of 64 to
    // 512 channels at batch 1 to 256, at N = 32: a workgroup alone on its
    // unit takes 6 + 3.4 per chunk of 16 kept blocks, two together 6 + 6.1
    // and more than that 6 + 7 for each two; N = 16: 5 + 3 and 4.5 + 5.4; the
    // other kernel 12 + the multiply-adds at 85 (70) TFLOP/s.  Taken where a
    // fifth faster by these.  256 -> 256 at 14x14, N = 32, batch 1: 32.5 us
    // against 14.4; batch 64: 60 against 92; 32 -> 32 at 112x112, batch 16:
    // 32.6 against 28.1.
    const double wgs = p.total, chunks = double(a.t) / a.G / 16 + 0.5;
    const int64_t cus = device_cu_count();
    const double px = kind == kPlS1 ? 1.0 : 0.7;         // a 128-pixel tile cuts the same weights
    const bool n32 = a.N == 32;
    const double each = wgs <= cus ? (n32 ? 3.4 : 3.0) : wgs <= 2.0 * cus ? (n32 ? 6.1 : 5.4) : (n32 ? 7.0 : 5.4);
    const double here = std::max(1.0, wgs / (2.0 * cus)) * ((n32 ? 6.0 : 4.5) + each * px * chunks);
    const double flops = 2.0 * a.npix * a.N * a.KK * double(a.t);
    return 1.2 * (3 + here) < 12 + flops * 1e-6 / (n32 ? 85 : 70);
}

onexn_status launch_planes_fwd(const ConvArgs& a, onexn_dtype xdt, onexn_dtype ydt, hipStream_t s) {
    PlArgs p = pl_fwd_args(a);
    const PlKind kind = pl_choose(p, a.kh, a.N);
    return with_epilogue(a, [&](auto ep) {
        constexpr bool E = decltype(ep)::value;
        auto by_n = [&](auto tx, auto ty) {
            if (a.N == 32) return launch_kind<false, decltype(tx), decltype(ty), 32, E>(kind, p, s);
            return launch_kind<false, decltype(tx), decltype(ty), 16, E>(kind, p, s);
        };
        if (xdt == ONEXN_F32) return by_n(float{}, float{});
        if (ydt == ONEXN_BF16) return by_n(uint16_t{}, uint16_t{});
        return by_n(uint16_t{}, float{});
    });
}

bool planes_dx_applies(const ConvArgs& a, onexn_dtype wdt, int32_t batch) {
    if (a.N < 8 || a.kh != 3 || a.kw != 3 || a.sh != a.sw || (wdt == ONEXN_F32 && a.sh != 1)) return false;
    const int es = wdt == ONEXN_F32 ? 4 : 2;
    if (!pl_fits(a, batch, int64_t(a.n) * a.HWo, es, int64_t(batch) * a.H * (a.W + 8))) return false;
    if (wdt == ONEXN_F32 && tuning(kTuneKernel) != 2 && bwd_data_pw_applies(a, ONEXN_F32, ONEXN_F32, batch)) {
        // Layers of few channels fill neither the 16-channel chunks nor the tile's
        // 32 rows.  us, fp32 instruction and here, at 56x56, batch 16: 32 -> 8,
        // N = 8 9.9 and 14.6, N = 16 13.5 and 14.9, N = 32 20.9 and 15.2; 144 -> 24,
        // N = 8 45.4 and 51.3, N = 16 39.5 and 51.8, N = 32 64 and 51; 16 -> 16 at
        // 28x28, batch 1, N = 8 11.8 and 10.1; 8 -> 64, N = 8 28.9 and 25.4, N = 16
        // 23.5 and 25.0, N = 32 17.1 and 24.9 (28x28, batch 1: 16.7 and 17.5).
        const bool few_px = int64_t(batch) * a.H * a.W <= (a.n <= 16 ? 20000 : 10000);
        if (a.N < 32 && a.n <= 24 && !(few_px && (a.N == 16 || a.n > 8))) return false;
        if (a.N == 32 && a.m <= 8) return false;
    }
    PlArgs p = pl_dx_args(a, batch, nullptr, nullptr);
    return a.G <= kPlMaxRuns && pl_choose(p, 3, 32) != kPlNone;
}

onexn_status launch_planes_dx(const ConvArgs& a, onexn_dtype wdt, onexn_dtype dxdt, int32_t batch, const void* dy,
                              void* dx, hipStream_t s) {
    PlArgs p = pl_dx_args(a, batch, dy, dx);
    const PlKind kind = pl_choose(p, 3, 32);
    if (wdt == ONEXN_F32) return launch_kind<true, float, float, 32, false>(kind, p, s);
    if (dxdt == ONEXN_BF16) return launch_kind<true, uint16_t, uint16_t, 32, false>(kind, p, s);
    return launch_kind<true, uint16_t, float, 32, false>(kind, p, s);
}

}  // namespace onexn
