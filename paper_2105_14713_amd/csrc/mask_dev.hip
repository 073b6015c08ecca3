// Mask building on the GPU: filter rearrangement, block scoring and the
// per-layer top-(1-p) selection of 1xN pruning, bit-exact with the host's
// onexn_build_mask.
//
// Paper: Lin et al., "1xN Pattern for Pruning Convolutional Neural Networks"
// (arXiv 2105.14713): Sec. 3.3 (filters in decreasing l1 norm), Sec. 3.2 and
// Eq. 4-5 (the l1 norm of each 1xN block), Eq. 1 and Sec. 4.1 (keep the
// 1 - p fraction of blocks with the largest norms, per layer).
//
// Bit-exactness.  The host sums every l1 norm in fp64 in memory order and
// ranks with a strict total order (filters: norm descending, then index
// ascending; blocks: score descending, then row-major index k*G + g
// ascending).  The kernels here add the same fp64 values in the same order
// (no reassociation, no fused multiply-add: the sums are additions of
// |w| only), and select with the same order, so their perm and mask equal
// the host's bit for bit.
//
//   mask_filter_norms  eight filters per wave: chunks of 512 elements come in
//                      coalesced and turn through LDS, and lane f adds filter
//                      f's elements one after another, so the sum is the
//                      sequential one.
//   mask_filter_perm   rank of filter j = filters before it in the order;
//                      perm[rank] = j (the identity without rearrangement).
//   mask_block_scores  one thread per block (k, g), input channel fastest
//                      for coalesced reads; rows of the rearranged layer are
//                      read through perm.
//   selection          The kept blocks are those up to a pivot (score, index)
//                      in the strict order, found by radix selection over the
//                      64-bit score bits (non-negative doubles order like
//                      their bit patterns); mask_write compares every block
//                      with it.  Layers of at most kLdsKeys blocks: one
//                      workgroup with the scores in LDS (mask_select).
//                      Larger ones spread over the chip: the scores kernel
//                      counts the top 10 or 11 key bits, mask_hist the next 11 of
//                      the keys under the pivot's top bits, mask_collect
//                      lists the few keys left, mask_pivot ranks those (or,
//                      with more than its list holds, selects over all scores
//                      as mask_select does).  The list has 1024 entries (256
//                      below 32768 blocks) however large the layer is; equal
//                      scores outnumber it, and for normal weights those that
//                      share the pivot's top 22 bits from some 1.1 million
//                      blocks on at N = 32, 4.3 million at N = 1, and half a
//                      million where a score is one bf16 weight (N = 1, 1x1:
//                      1024 x 1024 4.6 ms; 5.9 before the selection was
//                      spread).  The counts and the list live in the mask's
//                      own bytes until mask_write overwrites them, and the pivot
//                      in the workspace where the norms were, so the
//                      workspace is no larger for it.  (A mask outside device
//                      memory, which need not take atomics, is written once:
//                      mask_pivot then selects over all scores.)
//
// 2048 -> 2048 at N = 32, fp32, rearranged (131072 blocks, 16.8 MB of
// weights): 708 us with one wave per filter, a rank loop over eight
// workgroups and one selecting workgroup (54 + 131 + 19 + 502); 64 us now (21 +
// 10 + 11, then 5 + 6 + 9 + 4 for the selection).
// What bounds it now is the chain of dependent launches and, in the norms,
// the sequential fp64 additions that bit-exactness asks for.
//
// NaN weights, which the host function rejects, give NaN norms and scores;
// here they order above every number, so perm is still a permutation and the
// mask still keeps exactly t blocks.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <mutex>

#include "onexn_internal.h"

// Scratch of the no-allocation entry point (onexn_build_mask_dev_noalloc):
// the workspace of one mask build, 8 MiB, so layers with n + m * G up to about
// a million fit (the 2048 -> 2048 layer at N = 32 needs 1.1 MB).  Every GPU the
// library runs on holds its own copy from the program's load until the
// process ends.  In host code this name stands for the array but is not a
// device address: host code uses the address hipGetSymbolAddress returns.
static __device__ __align__(256) unsigned char scratch[size_t(8) << 20];

namespace onexn {
namespace {

constexpr size_t kScratchBytes = size_t(8) << 20;
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_addr[kMaxDevices] = {};

// Device address of the current device's scratch array, looked up once per
// device (with that device current) and kept.
onexn_status scratch_address(void** out) {
    int dev = 0;
    const hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(ONEXN_ERR_HIP, "build_mask_dev_noalloc: hipGetDevice: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= kMaxDevices)
        return fail(ONEXN_ERR_UNSUPPORTED, "build_mask_dev_noalloc: device %d beyond %d devices", dev, kMaxDevices);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_addr[dev]) {
        void* p = nullptr;
        const hipError_t se = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (se != hipSuccess || !p)
            return fail(ONEXN_ERR_HIP, "build_mask_dev_noalloc: hipGetSymbolAddress(scratch): %s",
                        hipGetErrorString(se));
        g_scratch_addr[dev] = p;
    }
    *out = g_scratch_addr[dev];
    return ONEXN_OK;
}

constexpr int kSelThreads = 1024;
constexpr int kSelBins = 256;
constexpr size_t kWsAlign = 256;
constexpr int kNormFilters = 8;           // filters per wave of mask_filter_norms,
constexpr int kNormLoads = 8;             // 64-element loads of each in flight (64 in all)
constexpr int kNormPitch = 64 * kNormLoads + 1;   // and floats per LDS row of a chunk
constexpr int kRankFilters = 4;           // filters ranked per wave of mask_filter_perm,
constexpr int kRankLoads = 8;             // and 64-norm loads in flight
constexpr int kLdsKeys = 16384;           // most scores one workgroup selects from (128 KB of LDS),
constexpr int kFewKeys = 2048;            // and a smaller variant
constexpr int kFewCand = 512;             // keys select_all ranks instead of going on by digits
constexpr int kDigit2 = 11;               // bits of the second histogram
constexpr int kBins2 = 1 << kDigit2;
constexpr int kHistItems = 4;             // keys per thread of mask_hist and mask_collect

// What the multi-workgroup selection keeps in the mask's bytes until
// mask_write fills them: counts of the keys' first kDigit1 bits (below the
// sign, which is 0) and of the next kDigit2 bits, and the keys left.
template <int kDigit1, int kList>
struct SelScratch {
    static constexpr int kBins1 = 1 << kDigit1, kCand = kList;
    static constexpr int kShift1 = 63 - kDigit1, kShift2 = kShift1 - kDigit2;
    uint32_t hist1[kBins1], hist2[kBins2];
    uint32_t count, pad;
    uint64_t key[kList];
    int32_t index[kList];
};
using SelSmall = SelScratch<10, 256>;     // for kSmallMin blocks and more
using SelLarge = SelScratch<11, 1024>;    // for kLargeMin blocks and more
constexpr int64_t kSmallMin = 16384, kLargeMin = 32768;
static_assert(sizeof(SelSmall) + 8 <= size_t(kSmallMin), "SelSmall lies in the mask's bytes");
static_assert(sizeof(SelLarge) + 8 <= size_t(kLargeMin), "SelLarge lies in the mask's bytes");
static_assert(kSmallMin <= kLdsKeys, "one workgroup holds the scores of every smaller layer");

// The last kept block in the strict order: kept = key above, or equal and index <= index.
struct Pivot {
    uint64_t key;
    int64_t index;
};

__device__ __forceinline__ double abs_elem(const float* w, int64_t e) {
    return fabs(static_cast<double>(w[e]));
}
__device__ __forceinline__ double abs_elem(const uint16_t* w, int64_t e) {
    return fabs(static_cast<double>(__uint_as_float(uint32_t(w[e]) << 16)));
}

// Order key of a non-negative sum: its bit pattern, NaN above +inf.
__device__ __forceinline__ uint64_t order_key(double d) {
    return d != d ? 0x7ff8000000000000ull : static_cast<uint64_t>(__double_as_longlong(d));
}

__device__ __forceinline__ float widen(float v) { return v; }
__device__ __forceinline__ float widen(uint16_t v) { return __uint_as_float(uint32_t(v) << 16); }

template <typename TW>
__global__ void __launch_bounds__(64) mask_filter_norms(const TW* __restrict__ w, int32_t n,
                                                         int64_t filt, double* __restrict__ norm) {
    __shared__ float sw[kNormFilters * kNormPitch];
    constexpr int kChunk = 64 * kNormLoads;
    const int lane = threadIdx.x;
    const int32_t j0 = blockIdx.x * kNormFilters;
    TW v[kNormFilters][kNormLoads];
    auto load = [&](int64_t e0) {                        // past the end: a real element, never added
#pragma unroll
        for (int u = 0; u < kNormLoads; ++u) {
            const int64_t e = min(e0 + 64 * u + lane, filt - 1);
#pragma unroll
            for (int f = 0; f < kNormFilters; ++f) v[f][u] = w[int64_t(min(j0 + f, n - 1)) * filt + e];
        }
    };
    double acc = 0.0;
    load(0);
    for (int64_t e0 = 0; e0 < filt; e0 += kChunk) {
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kNormLoads; ++u)
#pragma unroll
            for (int f = 0; f < kNormFilters; ++f) sw[f * kNormPitch + 64 * u + lane] = fabsf(widen(v[f][u]));
        __syncthreads();
        if (e0 + kChunk < filt) load(e0 + kChunk);
        if (lane < kNormFilters) {
            const float* row = sw + lane * kNormPitch;
            const int cnt = int(min(filt - e0, int64_t(kChunk)));
            int i = 0;
            for (; i + 32 <= cnt; i += 32) {
                float x[32];
#pragma unroll
                for (int u = 0; u < 32; ++u) x[u] = row[i + u];
#pragma unroll
                for (int u = 0; u < 32; ++u) acc += double(x[u]);
            }
            for (; i < cnt; ++i) acc += double(row[i]);
        }
    }
    if (lane < kNormFilters && j0 + lane < n) norm[j0 + lane] = acc;
}

// A wave ranks kRankFilters filters: its lanes take 64 norms at a time and
// the ballot's population counts those before each.  Also clears the
// selection's counts (`clear` words), which later kernels add to.
__global__ void __launch_bounds__(256) mask_filter_perm(const double* __restrict__ norm, int32_t n,
                                                         int32_t rearrange, int32_t* __restrict__ perm,
                                                         uint32_t* __restrict__ counts, int32_t clear) {
    for (int32_t i = blockIdx.x * 256 + threadIdx.x; i < clear; i += gridDim.x * 256) counts[i] = 0;
    const int lane = threadIdx.x & 63;
    const int32_t j0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * kRankFilters;
    if (j0 >= n) return;
    if (!rearrange) {
        if (lane < kRankFilters && j0 + lane < n) perm[j0 + lane] = j0 + lane;
        return;
    }
    uint64_t kj[kRankFilters];
    int32_t rank[kRankFilters];
#pragma unroll
    for (int f = 0; f < kRankFilters; ++f) {
        kj[f] = order_key(norm[min(j0 + f, n - 1)]);
        rank[f] = 0;
    }
    for (int32_t i0 = 0; i0 < n; i0 += 64 * kRankLoads) {
        double v[kRankLoads];
#pragma unroll
        for (int u = 0; u < kRankLoads; ++u) v[u] = norm[min(i0 + 64 * u + lane, n - 1)];
#pragma unroll
        for (int u = 0; u < kRankLoads; ++u) {
            const int32_t i = i0 + 64 * u + lane;
            const uint64_t ki = order_key(v[u]);
#pragma unroll
            for (int f = 0; f < kRankFilters; ++f)
                rank[f] += __popcll(__ballot(i < n && (ki > kj[f] || (ki == kj[f] && i < j0 + f))));
        }
    }
    if (lane == 0) {
#pragma unroll
        for (int f = 0; f < kRankFilters; ++f)
            if (j0 + f < n) perm[rank[f]] = j0 + f;
    }
}

// With kDigit1 > 0 each workgroup also counts its keys' first digit into hist1.
template <typename TW, int kDigit1>
__global__ void __launch_bounds__(256) mask_block_scores(const TW* __restrict__ w, const int32_t* __restrict__ perm,
                                                          int32_t n, int32_t m, int32_t KK, int32_t N,
                                                          int32_t G, double* __restrict__ score,
                                                          uint32_t* __restrict__ hist1) {
    constexpr int kBins1 = 1 << kDigit1;
    __shared__ uint32_t hist[kBins1];
    if constexpr (kDigit1 > 0) {
        for (int b = threadIdx.x; b < kBins1; b += 256) hist[b] = 0;
        __syncthreads();
    }
    const int64_t id = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (id < int64_t(m) * G) {
        const int32_t g = int32_t(id / m), k = int32_t(id - int64_t(g) * m);
        const int64_t filt = int64_t(m) * KK;
        const int32_t rows = min(N, n - g * N);
        double s = 0.0;
        // Eight rows' loads at a time, added in row order.
        int32_t i = 0;
        for (; i + 8 <= rows && KK == 1; i += 8) {
            double v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = abs_elem(w, int64_t(perm[g * N + i + u]) * filt + k);
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
        for (; i < rows; ++i) {
            const int64_t base = int64_t(perm[g * N + i]) * filt + int64_t(k) * KK;
#pragma unroll 9
            for (int32_t e = 0; e < KK; ++e) s += abs_elem(w, base + e);
        }
        score[int64_t(k) * G + g] = s;
        if constexpr (kDigit1 > 0) atomicAdd(&hist[order_key(s) >> (63 - kDigit1)], 1u);
    }
    if constexpr (kDigit1 > 0) {
        __syncthreads();
        for (int b = threadIdx.x; b < kBins1; b += 256)
            if (hist[b]) atomicAdd(&hist1[b], hist[b]);
    }
}

// The bin, from the top, in which the cumulative count of `hist` (kBins
// entries) reaches `need`; *left is what is then still needed of that bin.
// Called by every thread of a 256-thread workgroup.
template <int kBins>
__device__ __forceinline__ int32_t find_bin(const uint32_t* __restrict__ hist, int64_t need, int64_t* left) {
    constexpr int kPer = kBins / 256;
    __shared__ int64_t scan[256];
    __shared__ int32_t sBin;
    __shared__ int64_t sLeft;
    const int tid = threadIdx.x;
    uint32_t c[kPer];
    int64_t sum = 0;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        c[u] = hist[kBins - 1 - (tid * kPer + u)];
        sum += c[u];
    }
    scan[tid] = sum;
    __syncthreads();
    for (int d = 1; d < 256; d <<= 1) {
        const int64_t v = tid >= d ? scan[tid - d] : 0;
        __syncthreads();
        scan[tid] += v;
        __syncthreads();
    }
    int64_t before = scan[tid] - sum;
    if (before < need && scan[tid] >= need) {
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            if (before < need && before + c[u] >= need) {
                sBin = kBins - 1 - (tid * kPer + u);
                sLeft = need - before;
            }
            before += c[u];
        }
    }
    __syncthreads();
    *left = sLeft;
    const int32_t bin = sBin;
    __syncthreads();
    return bin;
}

// Counts the second digit of the keys whose first digit is the pivot's.
template <typename Sel>
__global__ void __launch_bounds__(256) mask_hist(const double* __restrict__ score, int64_t K, int64_t kept,
                                                  Sel* __restrict__ sel) {
    __shared__ uint32_t hist[kBins2];
    for (int b = threadIdx.x; b < kBins2; b += 256) hist[b] = 0;
    int64_t left;
    const uint64_t bin1 = find_bin<Sel::kBins1>(sel->hist1, kept, &left);
    const int64_t i0 = int64_t(blockIdx.x) * (256 * kHistItems) + threadIdx.x;
    double v[kHistItems];
#pragma unroll
    for (int u = 0; u < kHistItems; ++u) v[u] = score[min(i0 + 256 * u, K - 1)];
#pragma unroll
    for (int u = 0; u < kHistItems; ++u) {
        const uint64_t key = order_key(v[u]);
        if (i0 + 256 * u < K && key >> Sel::kShift1 == bin1)
            atomicAdd(&hist[(key >> Sel::kShift2) & (kBins2 - 1)], 1u);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < kBins2; b += 256)
        if (hist[b]) atomicAdd(&sel->hist2[b], hist[b]);
}

// Lists the keys whose first two digits are the pivot's.
template <typename Sel>
__global__ void __launch_bounds__(256) mask_collect(const double* __restrict__ score, int64_t K, int64_t kept,
                                                     Sel* __restrict__ sel) {
    int64_t left;
    const uint64_t bin1 = find_bin<Sel::kBins1>(sel->hist1, kept, &left);
    const uint64_t bin2 = find_bin<kBins2>(sel->hist2, left, &left);
    const uint64_t top = (bin1 << kDigit2) | bin2;
    const int64_t i0 = int64_t(blockIdx.x) * (256 * kHistItems) + threadIdx.x;
    double v[kHistItems];
#pragma unroll
    for (int u = 0; u < kHistItems; ++u) v[u] = score[min(i0 + 256 * u, K - 1)];
#pragma unroll
    for (int u = 0; u < kHistItems; ++u) {
        const int64_t i = i0 + 256 * u;
        const uint64_t key = order_key(v[u]);
        if (i >= K || key >> Sel::kShift2 != top) continue;
        const uint32_t at = atomicAdd(&sel->count, 1u);
        if (at < uint32_t(Sel::kCand)) {
            sel->key[at] = key;
            sel->index[at] = int32_t(i);
        }
    }
}

// Rank of (key, idx) among `count` listed keys in the strict order.
__device__ __forceinline__ int32_t list_rank(const uint64_t* keys, const int32_t* index, int32_t count,
                                             uint64_t key, int32_t idx) {
    int32_t rank = 0, i = 0;
    for (; i + 8 <= count; i += 8) {
        uint64_t k[8];
        int32_t x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            k[u] = keys[i + u];
            x[u] = index[i + u];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) rank += k[u] > key || (k[u] == key && x[u] < idx);
    }
    for (; i < count; ++i) rank += keys[i] > key || (keys[i] == key && index[i] < idx);
    return rank;
}

// The pivot over all K keys, one workgroup: radix selection 8 bits at a time
// from the top until few keys share the pivot's digits, which are then listed
// and ranked; with more than kFewCand keys equal to the pivot's, the last kept
// one of them is counted off in index order.  key_at(i): the key of block i.
template <typename F>
__device__ __forceinline__ Pivot select_all(int64_t K, int64_t kept, F key_at) {
    __shared__ uint64_t sKey[kFewCand];
    __shared__ int32_t sIdx[kFewCand];
    __shared__ uint32_t sCount, sListed;
    __shared__ uint32_t hist[kSelBins];
    __shared__ uint64_t sPrefix;
    __shared__ int64_t sNeed;
    __shared__ int64_t scan[kSelThreads];
    __shared__ int64_t sIndex;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    // After the pass at `shift`, prefix holds the top bits of the kept-th
    // largest key and need the number of keys with those top bits that still
    // have to be kept.
    if (tid == 0) {
        sPrefix = 0;
        sNeed = kept;
        sIndex = 0;
        sListed = 0;
    }
    uint64_t pmask = 0;
    for (int shift = 56; shift >= 0; shift -= 8) {
        for (int b = tid; b < kSelBins; b += kSelThreads) hist[b] = 0;
        __syncthreads();
        const uint64_t prefix = sPrefix;
        const int64_t need = sNeed;
        // Histogram of the next 8 bits of the candidates.  In the first
        // passes most keys share their top bits: when every candidate lane of
        // a wave hits one bin, a single atomic adds their count (same-address
        // atomics of a whole wave would otherwise serialise).
        for (int64_t i0 = 0; i0 < K; i0 += kSelThreads) {
            const int64_t i = i0 + tid;
            uint64_t key = 0;
            if (i < K) key = key_at(i);
            const bool cand = i < K && (key & pmask) == prefix;
            const uint32_t bin = uint32_t(key >> shift) & 0xff;
            const uint64_t active = __ballot(cand);
            if (active) {
                const int leader = __ffsll(static_cast<unsigned long long>(active)) - 1;
                const uint32_t lb = __shfl(bin, leader);
                if (__ballot(cand && bin == lb) == active) {
                    if (lane == leader) atomicAdd(&hist[lb], uint32_t(__popcll(active)));
                } else if (cand) {
                    atomicAdd(&hist[bin], 1u);
                }
            }
        }
        __syncthreads();
        // Counts from the top bin down, one wave, four bins a lane: the bin
        // where they reach `need` holds the need-th key.
        if (tid < 64) {
            uint32_t c[4];
            int64_t sum = 0;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                c[u] = hist[kSelBins - 1 - (4 * lane + u)];
                sum += c[u];
            }
            int64_t upto = sum;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int64_t v = __shfl_up((long long)upto, d);
                if (lane >= d) upto += v;
            }
            int64_t before = upto - sum;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (before < need && before + c[u] >= need) {
                    sNeed = need - before;
                    sPrefix = prefix | (uint64_t(kSelBins - 1 - (4 * lane + u)) << shift);
                    sCount = c[u];
                }
                before += c[u];
            }
        }
        pmask |= uint64_t(0xff) << shift;
        __syncthreads();
        if (sCount <= uint32_t(kFewCand)) {
            const uint64_t top = sPrefix;
            for (int64_t i = tid; i < K; i += kSelThreads) {
                const uint64_t key = key_at(i);
                if ((key & pmask) != top) continue;
                const uint32_t at = atomicAdd(&sListed, 1u);
                sKey[at] = key;
                sIdx[at] = int32_t(i);
            }
            __syncthreads();
            const int32_t count = int32_t(sCount);
            if (tid < count && list_rank(sKey, sIdx, count, sKey[tid], sIdx[tid]) == sNeed - 1) {
                sPrefix = sKey[tid];
                sIndex = sIdx[tid];
            }
            __syncthreads();
            return {sPrefix, sIndex};
        }
    }
    const uint64_t kstar = sPrefix;   // the kept-th largest key
    const int64_t ties = sNeed;       // keys equal to kstar that are kept (the lowest indices)

    // Ties counted in index order: thread tid scans the contiguous slice
    // [tid * per, (tid + 1) * per), and the one whose slice holds the
    // `ties`-th reports its index.
    const int64_t per = (K + kSelThreads - 1) / kSelThreads;
    const int64_t lo = min(K, tid * per), hi = min(K, lo + per);
    int64_t cnt = 0;
    for (int64_t i = lo; i < hi; ++i) cnt += key_at(i) == kstar;
    scan[tid] = cnt;
    __syncthreads();
    for (int d = 1; d < kSelThreads; d <<= 1) {   // inclusive scan
        const int64_t v = tid >= d ? scan[tid - d] : 0;
        __syncthreads();
        scan[tid] += v;
        __syncthreads();
    }
    int64_t before = scan[tid] - cnt;             // ties with a lower index than lo
    if (before < ties && scan[tid] >= ties) {
        for (int64_t i = lo; i < hi; ++i)
            if (key_at(i) == kstar && ++before == ties) sIndex = i;
    }
    __syncthreads();
    return {kstar, sIndex};
}

// Selection and mask of a layer with 0 < kept < K <= kKeys, in one workgroup.
template <int kKeys>
__global__ void __launch_bounds__(kSelThreads) mask_select(const double* __restrict__ score, int32_t K,
                                                            int64_t kept, uint8_t* __restrict__ mask) {
    __shared__ uint64_t keys[kKeys];
    for (int32_t i = threadIdx.x; i < K; i += kSelThreads) keys[i] = order_key(score[i]);
    __syncthreads();
    const Pivot p = select_all(K, kept, [&](int64_t i) { return keys[i]; });
    for (int32_t i = threadIdx.x; i < K; i += kSelThreads)
        mask[i] = keys[i] > p.key || (keys[i] == p.key && i <= p.index);
}

template <typename Sel>
__global__ void __launch_bounds__(kSelThreads) mask_pivot(const double* __restrict__ score, int64_t K, int64_t kept,
                                                           const Sel* __restrict__ sel, Pivot* __restrict__ pivot) {
    __shared__ uint64_t sKey[Sel::kCand];
    __shared__ int32_t sIdx[Sel::kCand];
    __shared__ int64_t sLeft;
    const int tid = threadIdx.x;
    const uint32_t count = sel ? sel->count : 0;
    if (!sel || count > uint32_t(Sel::kCand)) {
        const Pivot p = select_all(K, kept, [&](int64_t i) { return order_key(score[i]); });
        if (tid == 0) *pivot = p;
        return;
    }
    const bool has = tid < int(count);
    const uint64_t key = has ? sel->key[tid] : 0;
    const int32_t idx = has ? sel->index[tid] : 0;
    if (has) {
        sKey[tid] = key;
        sIdx[tid] = idx;
    }
    if (tid == 0) sLeft = kept;
    __syncthreads();
    // What is kept of the listed keys: kept minus the keys in higher bins.
    const uint64_t top = sKey[0] >> Sel::kShift2;  // count >= 1: the pivot itself is listed
    const uint32_t bin1 = uint32_t(top >> kDigit2), bin2 = uint32_t(top) & (kBins2 - 1);
    uint64_t above = 0;
    for (uint32_t b = bin1 + 1 + tid; b < uint32_t(Sel::kBins1); b += kSelThreads) above += sel->hist1[b];
    for (uint32_t b = bin2 + 1 + tid; b < uint32_t(kBins2); b += kSelThreads) above += sel->hist2[b];
    if (above) atomicAdd(reinterpret_cast<unsigned long long*>(&sLeft), 0ull - above);
    __syncthreads();
    if (has && list_rank(sKey, sIdx, int32_t(count), key, idx) == sLeft - 1) *pivot = {key, idx};
}

__global__ void __launch_bounds__(256) mask_write(const double* __restrict__ score, int64_t K,
                                                   const Pivot* __restrict__ pivot, uint8_t* __restrict__ mask) {
    const Pivot p = *pivot;
    const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (i >= K) return;
    const uint64_t key = order_key(score[i]);
    mask[i] = key > p.key || (key == p.key && i <= p.index);
}

__global__ void __launch_bounds__(256) mask_fill(int64_t K, uint8_t v, uint8_t* __restrict__ mask) {
    const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (i < K) mask[i] = v;
}

size_t align_up(size_t v) { return (v + kWsAlign - 1) / kWsAlign * kWsAlign; }

// Workspace: norm[n] then score[m*G], fp64.
size_t workspace_bytes(int64_t n, int64_t K) { return align_up(size_t(n) * 8) + align_up(size_t(K) * 8); }

onexn_status check_mask_args(const void* w, onexn_dtype wdt, int32_t n, int32_t m, int32_t kh,
                             int32_t kw, int32_t N, double p, const int32_t* perm,
                             const uint8_t* mask, const int64_t* t) {
    if (!w || !perm || !mask || !t) return fail(ONEXN_ERR_NULL, "build_mask_dev: NULL pointer argument");
    if (wdt != ONEXN_F32 && wdt != ONEXN_BF16)
        return fail(ONEXN_ERR_DTYPE, "build_mask_dev: unknown weight dtype %d", int(wdt));
    if (n < 1 || m < 1 || kh < 1 || kw < 1)
        return fail(ONEXN_ERR_ARG, "build_mask_dev: layer sizes must be >= 1");
    if (N < 1) return fail(ONEXN_ERR_ARG, "build_mask_dev: block length N must be >= 1");
    if (!(p >= 0.0 && p <= 1.0)) return fail(ONEXN_ERR_ARG, "build_mask_dev: p must lie in [0, 1]");
    const int64_t G = (int64_t(n) + N - 1) / N;
    if (int64_t(n) * m * kh * kw > INT32_MAX || int64_t(m) * G > INT32_MAX ||
        G * N * int64_t(kh) * kw > INT32_MAX)
        return fail(ONEXN_ERR_BUFSIZE, "build_mask_dev: layer too large for int32 indexing");
    return ONEXN_OK;
}

// Scores, pivot and mask of a layer with 0 < kept < K, the selection spread over workgroups.
template <typename Sel, int kDigit1, typename TW>
void launch_multi(const TW* w, const int32_t* perm, int32_t n, int32_t m, int32_t KK, int32_t N, int32_t G, int64_t K,
                  int64_t kept, double* score, Sel* sel, Pivot* pivot, uint8_t* mask, hipStream_t s) {
    const dim3 kgrid(uint32_t((K + 255) / 256)), hgrid(uint32_t((K + 256 * kHistItems - 1) / (256 * kHistItems)));
    hipLaunchKernelGGL((mask_block_scores<TW, kDigit1>), kgrid, dim3(256), 0, s, w, perm, n, m, KK, N, G, score,
                       sel->hist1);
    hipLaunchKernelGGL(mask_hist<Sel>, hgrid, dim3(256), 0, s, score, K, kept, sel);
    hipLaunchKernelGGL(mask_collect<Sel>, hgrid, dim3(256), 0, s, score, K, kept, sel);
    hipLaunchKernelGGL(mask_pivot<Sel>, dim3(1), dim3(kSelThreads), 0, s, score, K, kept, sel, pivot);
    hipLaunchKernelGGL(mask_write, kgrid, dim3(256), 0, s, score, K, pivot, mask);
}

bool in_device_memory(const void* p) {
    hipPointerAttribute_t at{};
    if (hipPointerGetAttributes(&at, p) == hipSuccess) return at.type == hipMemoryTypeDevice;
    (void)hipGetLastError();                       // memory that the runtime does not know
    return false;
}

template <typename TW>
onexn_status launch_mask(const TW* w, int32_t n, int32_t m, int32_t kh, int32_t kw, int32_t N,
                         int64_t kept, int32_t rearrange, int32_t* perm, uint8_t* mask, void* ws,
                         hipStream_t s) {
    const int32_t G = (n + N - 1) / N;
    const int64_t K = int64_t(m) * G;
    double* norm = static_cast<double*>(ws);
    double* score = reinterpret_cast<double*>(static_cast<char*>(ws) + align_up(size_t(n) * 8));
    const int64_t filt = int64_t(m) * kh * kw;
    // Selection spread over workgroups from kSmallMin blocks on, where its
    // scratch fits the mask: about even there (512 x 1024 at N = 32, 16384
    // blocks, rearranged: 37 us; 16368 blocks in one workgroup: 38 us), and the
    // one workgroup's time grows with the blocks.
    const bool all = kept <= 0 || kept >= K, large_layer = !all && K >= kSmallMin;
    const bool multi = large_layer && in_device_memory(mask);
    uint8_t* const aligned = reinterpret_cast<uint8_t*>((reinterpret_cast<uintptr_t>(mask) + 7) & ~uintptr_t(7));
    SelSmall* const small = reinterpret_cast<SelSmall*>(aligned);
    SelLarge* const large = reinterpret_cast<SelLarge*>(aligned);
    Pivot* const pivot = static_cast<Pivot*>(ws);  // the norms are read no more once perm is known
    const int32_t clear = !multi ? 0 : kBins2 + 1 + (K < kLargeMin ? SelSmall::kBins1 : SelLarge::kBins1);
    const dim3 kgrid(uint32_t((K + 255) / 256));
    if (rearrange)
        hipLaunchKernelGGL(mask_filter_norms<TW>, dim3((n + kNormFilters - 1) / kNormFilters), dim3(64), 0, s, w, n,
                           filt, norm);
    hipLaunchKernelGGL(mask_filter_perm, dim3((n + 4 * kRankFilters - 1) / (4 * kRankFilters)), dim3(256), 0, s, norm,
                       n, rearrange, perm, reinterpret_cast<uint32_t*>(aligned), clear);
    if (all) {
        hipLaunchKernelGGL(mask_fill, kgrid, dim3(256), 0, s, K, uint8_t(kept > 0), mask);
    } else if (!multi) {
        hipLaunchKernelGGL((mask_block_scores<TW, 0>), kgrid, dim3(256), 0, s, w, perm, n, m, kh * kw, N, G, score,
                           static_cast<uint32_t*>(nullptr));
        if (large_layer) {
            hipLaunchKernelGGL(mask_pivot<SelLarge>, dim3(1), dim3(kSelThreads), 0, s, score, K, kept,
                               static_cast<const SelLarge*>(nullptr), pivot);
            hipLaunchKernelGGL(mask_write, kgrid, dim3(256), 0, s, score, K, pivot, mask);
        } else if (K <= kFewKeys)
            hipLaunchKernelGGL(mask_select<kFewKeys>, dim3(1), dim3(kSelThreads), 0, s, score, int32_t(K), kept, mask);
        else
            hipLaunchKernelGGL(mask_select<kLdsKeys>, dim3(1), dim3(kSelThreads), 0, s, score, int32_t(K), kept, mask);
    } else if (K < kLargeMin) {
        launch_multi<SelSmall, 10>(w, perm, n, m, kh * kw, N, G, K, kept, score, small, pivot, mask, s);
    } else {
        launch_multi<SelLarge, 11>(w, perm, n, m, kh * kw, N, G, K, kept, score, large, pivot, mask, s);
    }
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return fail(ONEXN_ERR_HIP, "build_mask_dev: launch failed: %s", hipGetErrorString(err));
    return ONEXN_OK;
}

int64_t kept_blocks(int64_t K, double p) {
    double pruned = std::floor(p * double(K) + 0.5);
    pruned = std::min(std::max(pruned, 0.0), double(K));
    return K - int64_t(pruned);
}

onexn_status build_mask_dev(const void* w_dev, onexn_dtype wdt, int32_t n, int32_t m, int32_t kh,
                            int32_t kw, int32_t N, double p, int32_t rearrange, int32_t* perm_dev,
                            uint8_t* mask_dev, int64_t* t, void* ws, size_t ws_bytes,
                            void* stream) {
    const int64_t G = (int64_t(n) + N - 1) / N;
    const int64_t K = int64_t(m) * G;
    const int64_t kept = kept_blocks(K, p);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const onexn_status st =
        wdt == ONEXN_F32
            ? launch_mask(static_cast<const float*>(w_dev), n, m, kh, kw, N, kept, rearrange, perm_dev, mask_dev, ws, s)
            : launch_mask(static_cast<const uint16_t*>(w_dev), n, m, kh, kw, N, kept, rearrange, perm_dev, mask_dev, ws, s);
    (void)ws_bytes;
    if (st == ONEXN_OK) *t = kept;
    return st;
}

}  // namespace
}  // namespace onexn

using namespace onexn;

extern "C" size_t onexn_mask_workspace_bytes(int32_t n, int32_t m, int32_t N) {
    if (n < 1 || m < 1 || N < 1) return 0;
    const int64_t G = (int64_t(n) + N - 1) / N;
    return workspace_bytes(n, int64_t(m) * G);
}

extern "C" onexn_status onexn_build_mask_dev(const void* w_dev, onexn_dtype wdt, int32_t n, int32_t m,
                                             int32_t kh, int32_t kw, int32_t N, double p,
                                             int32_t rearrange, int32_t* perm_dev, uint8_t* mask_dev,
                                             int64_t* t, void* workspace_dev, size_t workspace_bytes_,
                                             void* stream) {
    clear_error();
    if (onexn_status st = check_mask_args(w_dev, wdt, n, m, kh, kw, N, p, perm_dev, mask_dev, t)) return st;
    const int64_t G = (int64_t(n) + N - 1) / N;
    const size_t need = workspace_bytes(n, int64_t(m) * G);
    if (!workspace_dev) return fail(ONEXN_ERR_NULL, "build_mask_dev: NULL workspace");
    if (workspace_bytes_ < need)
        return fail(ONEXN_ERR_BUFSIZE, "build_mask_dev: workspace of %zu bytes, %zu needed", workspace_bytes_, need);
    if (reinterpret_cast<uintptr_t>(workspace_dev) % 8 != 0)
        return fail(ONEXN_ERR_ARG, "build_mask_dev: workspace must be 8-byte aligned");
    return build_mask_dev(w_dev, wdt, n, m, kh, kw, N, p, rearrange, perm_dev, mask_dev, t,
                          workspace_dev, workspace_bytes_, stream);
}

extern "C" onexn_status onexn_build_mask_dev_noalloc(const void* w_dev, onexn_dtype wdt, int32_t n,
                                                     int32_t m, int32_t kh, int32_t kw, int32_t N,
                                                     double p, int32_t rearrange, int32_t* perm_dev,
                                                     uint8_t* mask_dev, int64_t* t, void* stream) {
    clear_error();
    if (onexn_status st = check_mask_args(w_dev, wdt, n, m, kh, kw, N, p, perm_dev, mask_dev, t)) return st;
    const int64_t G = (int64_t(n) + N - 1) / N;
    const size_t need = workspace_bytes(n, int64_t(m) * G);
    if (need > kScratchBytes)
        return fail(ONEXN_ERR_BUFSIZE,
                    "build_mask_dev_noalloc: the layer needs %zu bytes of scratch, the entry point holds "
                    "%zu (use onexn_build_mask_dev with a workspace)", need, kScratchBytes);
    void* ws = nullptr;
    if (onexn_status st = scratch_address(&ws)) return st;
    return build_mask_dev(w_dev, wdt, n, m, kh, kw, N, p, rearrange, perm_dev, mask_dev, t, ws,
                          kScratchBytes, stream);
}
