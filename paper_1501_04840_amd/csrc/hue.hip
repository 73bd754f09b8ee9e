// Hue image pipeline of Sec. 5: hexcone hue of 8-bit RGB pixels, periodic
// hue histogram, strict order of the pixels, and the frame for a target
// density by exact circular histogram specification (the readings are listed
// in ot_hue.h).
//
// Device layout (one caller-owned workspace, carved by ot_hue_create), per
// pixel: the hue FP32, the max and min channel 2 bytes, the rank u32, and for
// the sort the position in the order of the low digit u32, the high digit u16
// and the rank in that order u32; the digit counts per tile int32 [1024][tiles]
// and their totals, the source counts int32 [n]; per frame, the target counts
// and their inclusive cumulative sums int32 [n] and the shift one int64.  The
// strict order is a stable radix sort of 19-bit keys in two passes (below).  Per
// call of F frames: one planning kernel of F blocks (target counts, median
// shift) and one streaming kernel over the pixels in raster order with the
// frames along grid y, four pixels per thread (reads 10 bytes per pixel, writes
// 3 and optionally the 4-byte bin).
#include <hip/hip_runtime.h>

#include <climits>
#include <cstdint>
#include <new>

#include "../../include/ot_hue.h"

namespace {

constexpr int kMaxBins = 4096;
constexpr long long kMaxPix = 1LL << 30;
constexpr int kThreads = 256;
constexpr int kPlanThreads = 1024;
constexpr unsigned kRenderBlocks = 4096;  // 16 blocks per compute unit, per frame
constexpr int kMaxFrames = 65535;         // frames per call (grid y)
constexpr unsigned kConvBlocks = 8192;    // RGB<->HSV grid-stride launches
// radix sort of the 19-bit hue keys over tiles of kSortThreads x kSortItems
constexpr int kSortThreads = 512;
constexpr int kSortItems = 16;
constexpr int kSortTile = kSortThreads * kSortItems;
constexpr int kSortWaves = kSortThreads / 64;
constexpr int kKeyBits = 19;

// Every FP32 step below is one rounded operation in the written order: no
// contraction of a product and a sum into a fused multiply-add.
struct Hue {
    float h;
    int hi, lo;
};

__device__ __forceinline__ Hue hue_of(int r, int g, int b) {
#pragma clang fp contract(off)
    // one division: the sector's signed difference over max - min (selects,
    // not branches, so a wave with mixed sectors divides once)
    Hue o;
    o.hi = max(max(r, g), b);
    o.lo = min(min(r, g), b);
    const bool rs = o.hi == r, gs = !rs && o.hi == g;
    const int num = rs ? g - b : (gs ? b - r : r - g);
    const float d = o.hi > o.lo ? (float)(o.hi - o.lo) : 1.f;
    const float q = (float)num / d;
    float h6 = rs ? (q < 0.f ? q + 6.f : q) : (gs ? q + 2.f : q + 4.f);
    h6 = o.hi > o.lo ? h6 : 0.f;
    float h = h6 / 6.f;
    h = h >= 1.f ? h - 1.f : h;
    o.h = h + 0.f;        // no negative zero in the sort key
    return o;
}

__device__ __forceinline__ int bin_of(float h, int n) {
#pragma clang fp contract(off)
    const float x = h * (float)n;
    return min((int)floorf(x), n - 1);
}

__device__ __forceinline__ unsigned char to_u8(float v) {
#pragma clang fp contract(off)
    float r = floorf(v + 0.5f);
    r = fminf(fmaxf(r, 0.f), 255.f);
    return (unsigned char)(int)r;
}

// HSV of 8-bit RGB: the hexcone hue above, saturation (max - min) / max (0
// for black), value max / 255; float [N][3].
__global__ void __launch_bounds__(kThreads) k_rgb_to_hsv(const unsigned char* __restrict__ rgb,
                                                         long long N, float* hsv) {
#pragma clang fp contract(off)
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x; p < N; p += stride) {
        const unsigned char* c = rgb + 3 * p;
        const Hue u = hue_of(c[0], c[1], c[2]);
        const float hf = (float)u.hi;
        const float d = hf - (float)u.lo;
        hsv[3 * p] = u.h;
        hsv[3 * p + 1] = u.hi > 0 ? d / hf : 0.f;
        hsv[3 * p + 2] = hf / 255.f;
    }
}

// 8-bit RGB of float HSV by the textbook hexcone (h wrapped into [0, 1), s
// and v clamped to [0, 1], non-finite input black), channels rounded to
// nearest.
__global__ void __launch_bounds__(kThreads) k_hsv_to_rgb(const float* __restrict__ hsv,
                                                         long long N, unsigned char* rgb) {
#pragma clang fp contract(off)
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x; p < N; p += stride) {
        float h = hsv[3 * p], s = hsv[3 * p + 1], v = hsv[3 * p + 2];
        const bool bad = !(isfinite(h) && isfinite(s) && isfinite(v));
        h = bad ? 0.f : h;
        s = fminf(fmaxf(bad ? 0.f : s, 0.f), 1.f);
        v = fminf(fmaxf(bad ? 0.f : v, 0.f), 1.f);
        h = h - floorf(h);
        h = h >= 1.f ? h - 1.f : h;
        const float h6 = h * 6.f;
        const int i = min(max((int)floorf(h6), 0), 5);
        const float f = h6 - (float)i;
        const float pp = v * (1.f - s);
        const float sf = s * f;
        const float qq = v * (1.f - sf);
        const float g1 = 1.f - f;
        const float sg = s * g1;
        const float tt = v * (1.f - sg);
        float r, g, b;
        switch (i) {
            case 0: r = v; g = tt; b = pp; break;
            case 1: r = qq; g = v; b = pp; break;
            case 2: r = pp; g = v; b = tt; break;
            case 3: r = pp; g = qq; b = v; break;
            case 4: r = tt; g = pp; b = v; break;
            default: r = v; g = pp; b = qq; break;
        }
        unsigned char* o = rgb + 3 * p;
        o[0] = to_u8(r * 255.f);
        o[1] = to_u8(g * 255.f);
        o[2] = to_u8(b * 255.f);
    }
}

__global__ void k_fill_i32(int* p, int n, int v) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// Sort key: floor(h 2^19), exact (a power-of-two scaling).  Distinct hues of
// 8-bit RGB differ by at least 1 / (6 * 255 * 254) (differences of fractions with
// denominators <= 255, over 6), 1.34 * 2^-19: 2^-19 plus more than the few ulps of
// their FP32 rounding.  Equal hues give equal floats.  So this 19-bit key orders
// pixels exactly as the hue does.
__device__ __forceinline__ unsigned sort_key(float h) {
    return (unsigned)(h * (float)(1u << kKeyBits));
}

// ---- strict order of the pixels: a stable radix sort of the keys in two passes
//
// Tile i holds elements [i T, (i + 1) T) of the current order, T = kSortTile, and
// wave w of its block the w-th eighth, 64 elements a round: the order (wave,
// round, lane) is the element order.  Nothing but the rank of each pixel is
// wanted, so no pixel index is ever moved:
//   k_hue_keys      hues, bin counts, and per tile the counts of the low digit;
//   k_sort_low      each pixel's position pos in the order of the low digit, and the high digits moved there
//                   (2 bytes each, through LDS, in runs of a tile's equal digits);
//   k_sort_hist     per tile of that order the counts of the high digit;
//   k_sort_high     the rank of each element of that order, written there;
//   k_sort_gather   rank[p] = that of position pos[p].
// with k_sort_scan of the counts before k_sort_low and k_sort_high.  A wave counts
// its own digits, so a round needs no barrier; tiles are dealt to the XCDs in
// contiguous eighths, so that one L2 merges the short runs that adjacent tiles
// write side by side.  3840 x 2160: keys 29 us, low 34, hist
// 18, high 34, gather 28, the scans 5 each.  Three 8-bit passes that moved keys
// and indices, with four barriers a round and the last pass's random 4-byte
// writes, took 308 us (the scatters 232) after 47 us of keys.
constexpr int kLowBits = 9, kLow = 1 << kLowBits;
constexpr int kHigh = 1 << (kKeyBits - kLowBits);

// The tile of a block: XCD j (blocks go round-robin) gets the j-th contiguous
// eighth.
__device__ __forceinline__ int tile_of(int hw, int ntiles) {
    const int q = ntiles >> 3, r = ntiles & 7, xcd = hw & 7, slot = hw >> 3;
    return xcd * q + min(xcd, r) + slot;
}

// Hue (FP32) and max and min channel (hilo) in raster order, bin histogram (LDS counts, then one global add per
// bin and block) and the low digit's counts of a tile.  Four pixels per thread
// and step; VEC: the image is 4-byte aligned, so a group of four moves as one
// 12-byte load and one 16- and one 8-byte store (the tail group and unaligned images go
// pixel by pixel).
template <bool VEC>
__global__ void __launch_bounds__(kSortThreads) k_hue_keys(const unsigned char* __restrict__ rgb,
                                                           long long N, int n, int ntiles,
                                                           float* hue, unsigned short* hilo, int* counts,
                                                           int* lhist) {
    extern __shared__ int hist[];              // [n], then [kLow]
    int* const low = hist + n;
    for (int k = threadIdx.x; k < n + kLow; k += kSortThreads) hist[k] = 0;
    __syncthreads();
    const int tile = tile_of(blockIdx.x, ntiles);
    const long long base = (long long)tile * kSortTile;
    auto count = [&](float h) {
        atomicAdd(&hist[bin_of(h, n)], 1);
        atomicAdd(&low[sort_key(h) & (kLow - 1)], 1);
    };
#pragma unroll
    for (int r = 0; r < kSortItems / 4; ++r) {
        const long long p0 = base + 4 * (r * kSortThreads + (int)threadIdx.x);
        if (VEC && p0 + 4 <= N) {
            union { uint3 v; unsigned char b[12]; } in;
            in.v = *reinterpret_cast<const uint3*>(rgb + 3 * p0);
            union { uint2 v; unsigned short u[4]; } m;
            float h[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const Hue u = hue_of(in.b[3 * i], in.b[3 * i + 1], in.b[3 * i + 2]);
                h[i] = u.h;
                m.u[i] = (unsigned short)(u.hi | u.lo << 8);
            }
            *reinterpret_cast<float4*>(hue + p0) = make_float4(h[0], h[1], h[2], h[3]);
            *reinterpret_cast<uint2*>(hilo + p0) = m.v;
#pragma unroll
            for (int i = 0; i < 4; ++i) count(h[i]);
        } else {
            for (long long p = p0; p < p0 + 4 && p < N; ++p) {
                const unsigned char* c = rgb + 3 * p;
                const Hue u = hue_of(c[0], c[1], c[2]);
                hue[p] = u.h;
                hilo[p] = (unsigned short)(u.hi | u.lo << 8);
                count(u.h);
            }
        }
    }
    __syncthreads();
    for (int k = threadIdx.x; k < n; k += kSortThreads)
        if (hist[k]) atomicAdd(&counts[k], hist[k]);
    for (int d = threadIdx.x; d < kLow; d += kSortThreads) lhist[(long long)d * ntiles + tile] = low[d];
}

// hist[d][tile] = number of elements of high digit d in the tile.  Eight
// elements per 16-byte load (the digits' array is 16-byte aligned).
__global__ void __launch_bounds__(kSortThreads) k_sort_hist(const unsigned short* __restrict__ dig,
                                                            long long N, int ntiles, int* hist) {
    __shared__ int cnt[kHigh];
    for (int d = threadIdx.x; d < kHigh; d += kSortThreads) cnt[d] = 0;
    __syncthreads();
    const int tile = tile_of(blockIdx.x, ntiles);
    const long long base = (long long)tile * kSortTile;
#pragma unroll
    for (int r = 0; r < kSortItems / 8; ++r) {
        const long long e = base + 8 * (r * kSortThreads + (int)threadIdx.x);
        if (e + 8 <= N) {
            union { uint4 v; unsigned short u[8]; } x;
            x.v = *reinterpret_cast<const uint4*>(dig + e);
#pragma unroll
            for (int i = 0; i < 8; ++i) atomicAdd(&cnt[x.u[i]], 1);
        } else {
            for (long long q = e; q < e + 8 && q < N; ++q) atomicAdd(&cnt[dig[q]], 1);
        }
    }
    __syncthreads();
    for (int d = threadIdx.x; d < kHigh; d += kSortThreads) hist[(long long)d * ntiles + tile] = cnt[d];
}

// Block d: exclusive prefix sums of hist[d][0..ntiles) in place (the start of
// each tile's run of digit d among all elements of digit d) and totals[d].
constexpr int kScanThreads = 256;

__global__ void __launch_bounds__(kScanThreads) k_sort_scan(int* hist, int ntiles, int* totals) {
    __shared__ int part[kScanThreads];
    const int t = threadIdx.x;
    int* h = hist + (long long)blockIdx.x * ntiles;
    const int per = (ntiles + kScanThreads - 1) / kScanThreads;
    const int i0 = t * per, i1 = min(i0 + per, ntiles);
    int sum = 0;
    for (int i = i0; i < i1; ++i) sum += h[i];
    part[t] = sum;
    __syncthreads();
    for (int off = 1; off < kScanThreads; off <<= 1) {       // inclusive scan of the parts
        const int v = t >= off ? part[t - off] : 0;
        __syncthreads();
        part[t] += v;
        __syncthreads();
    }
    int run = part[t] - sum;
    for (int i = i0; i < i1; ++i) {
        const int v = h[i];
        h[i] = run;
        run += v;
    }
    if (t == kScanThreads - 1) totals[blockIdx.x] = part[t];
}

// Exclusive scan over the block of D values per thread (thread t: entries D t
// + q); sh: one word per wave.
template <int D>
__device__ __forceinline__ void block_scan(int (&v)[D], int* sh) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int own = 0;
#pragma unroll
    for (int q = 0; q < D; ++q) own += v[q];
    int inc = own;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int a = __shfl_up(inc, off, 64);
        inc += lane >= off ? a : 0;
    }
    __syncthreads();                           // (sh may still be read from a scan before)
    if (lane == 63) sh[w] = inc;
    __syncthreads();
    int run = inc - own;
    for (int q = 0; q < w; ++q) run += sh[q];
#pragma unroll
    for (int q = 0; q < D; ++q) {
        const int a = v[q];
        v[q] = run;
        run += a;
    }
}

// The rank of each of the wave's elements among the wave's earlier elements of
// the same digit (rk), and the wave's counts of the digits in cnt (zeros on
// entry).  valid holds for a prefix of the elements.
template <int BITS>
__device__ __forceinline__ void wave_ranks(const int (&dig)[kSortItems], const bool (&valid)[kSortItems],
                                           int* cnt, int (&rk)[kSortItems]) {
    const unsigned long long lt = (1ull << (threadIdx.x & 63)) - 1ull;
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        unsigned long long peers = __ballot(valid[r]);      // lanes of the same digit
#pragma unroll
        for (int b = 0; b < BITS; ++b) {
            const bool bit = (dig[r] >> b) & 1;
            const unsigned long long m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        const int lr = __popcll(peers & lt);
        const int before = cnt[dig[r]];
        rk[r] = before + lr;
        if (valid[r] && lr == 0) cnt[dig[r]] = before + __popcll(peers);
        // the next round's loads see this round's stores (one wave's LDS
        // operations complete in order)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
}

__global__ void __launch_bounds__(kSortThreads) k_sort_low(const float* __restrict__ hue, long long N,
                                                           int ntiles, const int* __restrict__ pre,
                                                           const int* __restrict__ totals,
                                                           unsigned* pos, unsigned short* high) {
    static_assert(kLow == kSortThreads, "a thread per digit");
    __shared__ int cnt[kSortWaves][kLow];      // counts, then in-tile starts, per wave and digit
    __shared__ int gbase[kLow];                // a digit's place in the tile to its global place
    __shared__ int sh[kSortWaves];
    __shared__ unsigned st[kSortTile];         // the tile in order: keys
    const int t = threadIdx.x, w = t >> 6, lane = t & 63;
    const int tile = tile_of(blockIdx.x, ntiles);
    const long long base = (long long)tile * kSortTile;
    int off[1] = {totals[t]};
    const int first = pre[(long long)t * ntiles + tile];
    int dig[kSortItems], rk[kSortItems];
    unsigned key[kSortItems];
    bool valid[kSortItems];
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        const long long e = base + w * (kSortTile / kSortWaves) + r * 64 + lane;
        valid[r] = e < N;
        key[r] = sort_key(hue[valid[r] ? e : 0]);
        dig[r] = key[r] & (kLow - 1);
    }
    for (int i = t; i < kSortWaves * kLow; i += kSortThreads) (&cnt[0][0])[i] = 0;
    block_scan(off, sh);                       // (its barriers order the zeros)
    wave_ranks<kLowBits>(dig, valid, cnt[w], rk);
    __syncthreads();
    {   // digit t
        int run[1] = {0}, c[kSortWaves];
#pragma unroll
        for (int q = 0; q < kSortWaves; ++q) {
            c[q] = cnt[q][t];
            run[0] += c[q];
        }
        block_scan(run, sh);                   // the digit's start in the tile
        gbase[t] = off[0] + first - run[0];
        int s0 = run[0];
#pragma unroll
        for (int q = 0; q < kSortWaves; ++q) {
            cnt[q][t] = s0;
            s0 += c[q];
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        if (!valid[r]) continue;
        const int p = cnt[w][dig[r]] + rk[r];
        st[p] = key[r];
        pos[base + w * (kSortTile / kSortWaves) + r * 64 + lane] = gbase[dig[r]] + p;
    }
    __syncthreads();
    const int nh = (int)min((long long)kSortTile, N - base);
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        const int j = r * kSortThreads + t;
        if (j >= nh) continue;
        const unsigned k = st[j];
        high[gbase[k & (kLow - 1)] + j] = (unsigned short)(k >> kLowBits);
    }
}

__global__ void __launch_bounds__(kSortThreads) k_sort_high(const unsigned short* __restrict__ high,
                                                            long long N, int ntiles,
                                                            const int* __restrict__ pre,
                                                            const int* __restrict__ totals,
                                                            unsigned* rank) {
    constexpr int D = kHigh / kSortThreads;    // digits per thread
    static_assert(D * kSortThreads == kHigh, "whole digits per thread");
    __shared__ int cnt[kSortWaves][kHigh];     // counts, then global starts, per wave and digit
    __shared__ int sh[kSortWaves];
    const int t = threadIdx.x, w = t >> 6, lane = t & 63;
    const int tile = tile_of(blockIdx.x, ntiles);
    const long long base = (long long)tile * kSortTile + w * (kSortTile / kSortWaves) + lane;
    int off[D], first[D];
#pragma unroll
    for (int q = 0; q < D; ++q) {
        off[q] = totals[D * t + q];
        first[q] = pre[(long long)(D * t + q) * ntiles + tile];
    }
    int dig[kSortItems], rk[kSortItems];
    bool valid[kSortItems];
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        valid[r] = base + r * 64 < N;
        dig[r] = high[valid[r] ? base + r * 64 : 0];
    }
    for (int i = t; i < kSortWaves * kHigh; i += kSortThreads) (&cnt[0][0])[i] = 0;
    block_scan(off, sh);                       // (its barriers order the zeros)
    wave_ranks<kKeyBits - kLowBits>(dig, valid, cnt[w], rk);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < D; ++q) {
        int s0 = off[q] + first[q];
#pragma unroll
        for (int i = 0; i < kSortWaves; ++i) {
            const int c = cnt[i][D * t + q];
            cnt[i][D * t + q] = s0;
            s0 += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSortItems; ++r)
        if (valid[r]) rank[base + r * 64] = (unsigned)(cnt[w][dig[r]] + rk[r]);
}

// rank[p] = ranks[pos[p]], four pixels per thread and step (16-byte accesses): a
// tile's reads of ranks are its runs of equal low digits.
__global__ void __launch_bounds__(kSortThreads) k_sort_gather(const unsigned* __restrict__ pos,
                                                              const unsigned* __restrict__ ranks,
                                                              long long N, int ntiles, unsigned* rank) {
    const long long base = (long long)tile_of(blockIdx.x, ntiles) * kSortTile + 4 * threadIdx.x;
    if ((long long)(tile_of(blockIdx.x, ntiles) + 1) * kSortTile <= N) {
        constexpr int Q = kSortItems / 4;
        union { uint4 v; unsigned u[4]; } p[Q], o[Q];
#pragma unroll
        for (int r = 0; r < Q; ++r) p[r].v = *reinterpret_cast<const uint4*>(pos + base + 4 * r * kSortThreads);
#pragma unroll
        for (int r = 0; r < Q; ++r)
#pragma unroll
            for (int i = 0; i < 4; ++i) o[r].u[i] = ranks[p[r].u[i]];
#pragma unroll
        for (int r = 0; r < Q; ++r) *reinterpret_cast<uint4*>(rank + base + 4 * r * kSortThreads) = o[r].v;
    } else {
        for (int r = 0; r < kSortItems / 4; ++r)
            for (long long e = base + 4 * r * kSortThreads, i = 0; i < 4 && e + i < N; ++i)
                rank[e + i] = ranks[pos[e + i]];
    }
}

__global__ void k_hue_density(const int* __restrict__ counts, int n, long long N, float* dens) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) dens[k] = (float)((double)counts[k] * ((double)n / (double)N));
}

// Exclusive prefix sums of two integer arrays of n <= kMaxBins entries held
// kBinsPerThread per thread (Hillis-Steele over the per-thread totals).
constexpr int kBinsPerThread = kMaxBins / kPlanThreads;

__device__ __forceinline__ void block_scan2(int& x, int& y, int* sx, int* sy) {
    const int t = threadIdx.x;
    sx[t] = x;
    sy[t] = y;
    __syncthreads();
    for (int off = 1; off < kPlanThreads; off <<= 1) {
        const int ax = t >= off ? sx[t - off] : 0, ay = t >= off ? sy[t - off] : 0;
        __syncthreads();
        sx[t] += ax;
        sy[t] += ay;
        __syncthreads();
    }
    x = t ? sx[t - 1] : 0;              // exclusive
    y = t ? sy[t - 1] : 0;
    __syncthreads();
}

// One block: target counts by largest remainder, the inclusive cumulative
// target counts, and the shift (lower median of the edge differences).
// The remainder ranks take bins strided over the block (t + 1024 i), the
// prefix sums blocked (kBinsPerThread t + i).  The FP64 mass is summed bin by
// bin in index order (one thread, from LDS); the integer sums and prefix sums
// are exact in any order.
__global__ void __launch_bounds__(kPlanThreads) k_hue_plan(const float* __restrict__ target,
                                                           const int* __restrict__ cs, int n,
                                                           long long N, int* ct_out,
                                                           int* cum_out, long long* shift) {
    {   // block f plans frame f
        const long long f = blockIdx.x;
        target += f * n;
        ct_out += f * n;
        cum_out += f * n;
        shift += f;
    }
    __shared__ double rem[kMaxBins];
    __shared__ int ct[kMaxBins];
    __shared__ int sx[kPlanThreads], sy[kPlanThreads];
    __shared__ double S_sh;
    __shared__ unsigned long long fl_sh;
    int* D = reinterpret_cast<int*>(rem);   // edge differences, once rem is consumed
    const int t = threadIdx.x;
    // the target, negative and non-finite entries as zero, staged in rem
    for (int k = t; k < n; k += blockDim.x) {
        const float v = target[k];
        rem[k] = (isfinite(v) && v > 0.f) ? (double)v : 0.0;
    }
    if (t == 0) fl_sh = 0;
    __syncthreads();
    if (t == 0) {                       // the mass, bin by bin in index order
        double S = 0.0;
#pragma unroll 8
        for (int k = 0; k < n; ++k) S += rem[k];
        S_sh = S;
    }
    __syncthreads();
    const double S = S_sh;
    const bool keep = !(S > 0.0);
    int fsum = 0;
    for (int k = t; k < n; k += blockDim.x) {
        if (keep) {
            ct[k] = cs[k];
            rem[k] = 0.0;
        } else {
            const double x = ((double)N * rem[k]) / S;
            const double c = floor(x);
            ct[k] = (int)c;
            rem[k] = x - c;
        }
        fsum += ct[k];
    }
    atomicAdd(&fl_sh, (unsigned long long)fsum);
    __syncthreads();
    const long long left = keep ? 0 : N - (long long)fl_sh;
    // the `left` largest remainders (ties: lower bin) get one more pixel;
    // bins strided over the block, the rank loop unrolled so that its LDS
    // loads overlap
    int add[kBinsPerThread];
#pragma unroll
    for (int q = 0; q < kBinsPerThread; ++q) {
        const int k = t + q * kPlanThreads;
        add[q] = 0;
        if (k < n && left > 0) {
            const double rk = rem[k];
            int rank = 0;
#pragma unroll 8
            for (int j = 0; j < n; ++j) {
                const double rj = rem[j];
                rank += (rj > rk || (rj == rk && j < k)) ? 1 : 0;
            }
            add[q] = rank < left ? 1 : 0;
        }
    }
    __syncthreads();                    // every read of rem is done
#pragma unroll
    for (int q = 0; q < kBinsPerThread; ++q) {
        const int k = t + q * kPlanThreads;
        if (k < n) ct[k] += add[q];
    }
    __syncthreads();
    int cst[kBinsPerThread], ctt[kBinsPerThread];
    int xs = 0, xt = 0;
#pragma unroll
    for (int q = 0; q < kBinsPerThread; ++q) {
        const int k = kBinsPerThread * t + q;
        cst[q] = k < n ? cs[k] : 0;
        ctt[q] = k < n ? ct[k] : 0;
        xs += cst[q];
        xt += ctt[q];
    }
    block_scan2(xs, xt, sx, sy);
#pragma unroll
    for (int q = 0; q < kBinsPerThread; ++q) {
        const int k = kBinsPerThread * t + q;
        if (k < n) {
            D[k] = xs - xt;             // before bin k
            xs += cst[q];
            xt += ctt[q];
            cum_out[k] = xt;
            ct_out[k] = ctt[q];
        }
    }
    __syncthreads();
    const int m = (n - 1) / 2;          // lower median: the value of rank m
    for (int e = t; e < n; e += blockDim.x) {
        const int de = D[e];
        int rank = 0;
#pragma unroll 8
        for (int j = 0; j < n; ++j) {
            const int dj = D[j];
            rank += (dj < de || (dj == de && j < e)) ? 1 : 0;
        }
        if (rank == m) *shift = de;
    }
}

// Output bins of W pixels of ranks rk: the first bin whose cumulative count
// exceeds q = (rk - s) mod N, i.e. the number of cumulative counts <= q.  cl
// holds the n nondecreasing counts padded with INT_MAX to 2^L entries, so the
// branch-free search needs no bounds test, and its steps are constants: an LDS
// read at a constant offset, a comparison, a select and an add each.  W pixels in
// lockstep so that their LDS loads overlap.
template <int W, int L>
__device__ __forceinline__ void out_bins(const unsigned* rk, int s, int N, const int* cl, int n,
                                         int* lo) {
    // N <= 2^30: rank - s lies in (-2^30, 2^31 - 1), so 32-bit arithmetic
    int q[W];
    const char* at[W];
#pragma unroll
    for (int i = 0; i < W; ++i) {
        q[i] = (int)rk[i] - s;          // rank in [0, N), shift in (-N, N)
        q[i] = q[i] < 0 ? q[i] + N : (q[i] >= N ? q[i] - N : q[i]);
        at[i] = reinterpret_cast<const char*>(cl);
    }
    auto entry = [&](int i, int k) { return *reinterpret_cast<const int*>(at[i] + 4 * k); };
#pragma unroll
    for (int b = L - 1; b >= 0; --b) {
        const int half = 1 << b;
#pragma unroll
        for (int i = 0; i < W; ++i) at[i] += entry(i, half - 1) <= q[i] ? 4 * half : 0;
    }
#pragma unroll
    for (int i = 0; i < W; ++i) {
        const int k = (int)(at[i] - reinterpret_cast<const char*>(cl)) >> 2;
        lo[i] = min(k + (entry(i, 0) <= q[i] ? 1 : 0), n - 1);
    }
}

// What the frames share of a pixel: its hue, the bin of it, and the max and min
// channel (hilo: max in byte 0, min in byte 1).
struct Px {
    float h, bin, hi, lo;
    unsigned hilo;
};

__device__ __forceinline__ Px px_of(unsigned hilo, float h, int n) {
#pragma clang fp contract(off)
    Px p;
    p.h = h;
    p.bin = fminf(floorf(h * (float)n), (float)(n - 1));       // bin_of
    p.hi = (float)(hilo & 255);
    p.lo = (float)(hilo >> 8 & 255);
    p.hilo = hilo & 0xFFFF;
    return p;
}

// A pixel's bytes R, G, B of a frame: its hue moved to the output bin, in the
// hexcone with the max channel hi and the min channel lo kept.  rn = 1 / n.
//   - (kout - bin) / n rounded once, without a division: q = k rn, then one
//     correction by the exact remainder.  The corrected value is within 2^-23 of
//     a unit of the quotient, and for n <= 4096 no quotient k / n lies closer
//     than 2^-13 of a unit to where its rounding changes.
//   - the hue back into [0, 1): h2 - floor(h2) is the wrap by one either way.
//   - one channel is between lo and hi, so only it is rounded; sel gives the
//     bytes (hi, lo, between) their places for each of the six sectors.
__device__ __forceinline__ unsigned paint_px(const Px& p, int kout, float fn, float rn,
                                             const unsigned* sel) {
#pragma clang fp contract(off)
    const float k = (float)kout - p.bin;
    const float q0 = k * rn;
    const float q = fmaf(fmaf(-fn, q0, k), rn, q0);
    float h2 = p.h + q;
    h2 = h2 - floorf(h2);
    h2 = h2 >= 1.f ? h2 - 1.f : h2;
    const float h6 = h2 * 6.f;
    const float sf = fminf(floorf(h6), 5.f);
    const int sector = (int)sf;
    const float x = (p.hi - p.lo) * (h6 - sf);
    const float v = sector & 1 ? p.hi - x : p.lo + x;
    const unsigned between = (unsigned)(v + 0.5f);             // floor: 0 <= v <= 255
    return __builtin_amdgcn_perm(0u, p.hilo | between << 16, sel[sector]);
}

// Frames over the pixels in raster order: blockIdx.y takes FB of the F frames,
// whose cumulative counts are in LDS together, and a thread four pixels in a
// grid-stride loop, read once for all of its frames.  VEC: the output is 4-byte
// aligned (and bins_out 16-byte aligned), so a group of four moves as 8 bytes of max
// and min channels, 16 bytes each of hue, rank and bins, 12 bytes of RGB; the
// tail group and unaligned images go pixel by pixel.  Bound by its vector
// instructions and LDS reads, the search's above all, so its time depends on how far
// apart neighbouring pixels search: 33 frames of 3840 x 2160, 360 bins, of a smooth
// image take 400 us along a path of densities and 487 for 33 unrelated ones (a frame
// alone 24), with random densities 680.  With the pixels read for each frame, a
// division, a rounding per channel and search steps at computed addresses the
// unrelated ones took 834 and a frame 30.
template <bool VEC, int L, int FB>
__global__ void __launch_bounds__(kThreads) k_hue_render(const unsigned short* __restrict__ hilo,
                                                         const float* __restrict__ hue,
                                                         const unsigned* __restrict__ rank,
                                                         const int* __restrict__ cum,
                                                         const long long* __restrict__ shift,
                                                         int F, int n, long long N, unsigned char* out,
                                                         int* bins_out) {
    constexpr int pw = 1 << L;
    __shared__ int cl[FB][pw];         // cumulative counts, INT_MAX padding
    __shared__ unsigned sel[8];
    const int f0 = blockIdx.y * FB, nf = min(FB, F - f0);
    for (int k = threadIdx.x; k < nf * pw; k += blockDim.x) {
        const int f = k >> L, j = k & (pw - 1);
        cl[f][j] = j < n ? cum[(long long)(f0 + f) * n + j] : INT_MAX;
    }
    if (threadIdx.x < 6) {
        // places of R, G, B by sector: hi (0), lo (1) or the channel between (2)
        const unsigned places[6] = {0x010200u, 0x010002u, 0x020001u, 0x000201u, 0x000102u, 0x020100u};
        sel[threadIdx.x] = 0x0C000000u | places[threadIdx.x];  // (0x0C: a zero byte)
    }
    __syncthreads();
    int s32[FB];
#pragma unroll
    for (int f = 0; f < FB; ++f) s32[f] = (int)shift[min(f0 + f, F - 1)];
    const int N32 = (int)N;
    const float fn = (float)n, rn = 1.f / (float)n;
    const long long groups = (N + 3) / 4;
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long gi = (long long)blockIdx.x * blockDim.x + threadIdx.x; gi < groups;
         gi += stride) {
        const long long p0 = 4 * gi;
        if (VEC && p0 + 4 <= N) {
            union { uint4 v; unsigned u[4]; } rk;
            const uint2 m = *reinterpret_cast<const uint2*>(hilo + p0);
            rk.v = *reinterpret_cast<const uint4*>(rank + p0);
            const float4 hv = *reinterpret_cast<const float4*>(hue + p0);
            const Px px[4] = {px_of(m.x, hv.x, n), px_of(m.x >> 16, hv.y, n), px_of(m.y, hv.z, n),
                              px_of(m.y >> 16, hv.w, n)};
#pragma unroll
            for (int f = 0; f < FB; ++f) {
                if (f >= nf) break;            // uniform
                int kb[4];
                unsigned o[4];
                out_bins<4, L>(rk.u, s32[f], N32, cl[f], n, kb);
#pragma unroll
                for (int i = 0; i < 4; ++i) o[i] = paint_px(px[i], kb[i], fn, rn, sel);
                uint3 v;
                v.x = o[0] | o[1] << 24;
                v.y = o[1] >> 8 | o[2] << 16;
                v.z = o[2] >> 16 | o[3] << 8;
                *reinterpret_cast<uint3*>(out + (f0 + f) * 3 * N + 3 * p0) = v;
                if (bins_out)
                    *reinterpret_cast<int4*>(bins_out + (f0 + f) * N + p0) =
                        make_int4(kb[0], kb[1], kb[2], kb[3]);
            }
        } else {
            for (long long p = p0; p < p0 + 4 && p < N; ++p) {
                const unsigned r1 = rank[p];
                const Px px = px_of(hilo[p], hue[p], n);
                for (int f = 0; f < nf; ++f) {
                    int k;
                    out_bins<1, L>(&r1, (int)shift[f0 + f], N32, cl[f], n, &k);
                    const unsigned o = paint_px(px, k, fn, rn, sel);
                    unsigned char* c = out + (f0 + f) * 3 * N + 3 * p;
                    c[0] = (unsigned char)o;
                    c[1] = (unsigned char)(o >> 8);
                    c[2] = (unsigned char)(o >> 16);
                    if (bins_out) bins_out[(f0 + f) * N + p] = k;
                }
            }
        }
    }
}

// Launch for counts padded to 2^L, one frame per block or four.  Four read each
// pixel once for all, but are four serial searches of a block: they pay once the
// frames' blocks still fill the chip in fours (28 a compute unit, pixel by pixel 14),
// and for 1024 counts, where the searches hide more of the reads, only for four times
// that.  Us, one and four: 64 x 64, 360 bins, 5 frames 38 and 43; 640 x 480 x 33 frames
// (39 blocks a unit) 57 and 60, at 64 bins 36 and 32; 1920 x 1080 x 4 (32) 55 and 55, at
// 64 bins 35 and 30; 641 x 479, 9 frames (11) 46 and 49, 17 (20) 56 and 53; 303 x 1605 x 8,
// 300 bins (15) 49 and 47; 3840 x 2160 x 33 526 and 434; 1024 bins: 1280 x 720 x 17 (60) 135
// and 142, 1920 x 1080 x 33 (261) 253 and 240, 1501 x 1001 x 17 (97) 187 and 182, 661 bins
// 147 and 141.  Two frames per block of 2048 counts gained nothing.
template <int L>
void render_launch(bool vec, unsigned blocks, hipStream_t st, const unsigned short* hilo,
                   const float* hue, const unsigned* rank, const int* cum, const long long* shift, int F,
                   int n, long long N, unsigned char* out, int* bins_out) {
    constexpr int FB = L <= 10 ? 4 : 1;
    const long long enough = 256 * (vec ? 28 : 14) * (L == 10 ? 4 : 1);
    const dim3 block(kThreads);
    const int groups = (F + FB - 1) / FB;
    if (F == 1 || FB == 1 || (long long)blocks * F < enough) {
        const dim3 grid(blocks, (unsigned)F);
        if (vec) hipLaunchKernelGGL((k_hue_render<true, L, 1>), grid, block, 0, st, hilo, hue, rank,
                                    cum, shift, F, n, N, out, bins_out);
        else hipLaunchKernelGGL((k_hue_render<false, L, 1>), grid, block, 0, st, hilo, hue, rank,
                                cum, shift, F, n, N, out, bins_out);
        return;
    }
    if constexpr (FB > 1) {
        const dim3 grid(blocks, (unsigned)groups);
        if (vec) hipLaunchKernelGGL((k_hue_render<true, L, FB>), grid, block, 0, st, hilo, hue, rank, cum,
                                    shift, F, n, N, out, bins_out);
        else hipLaunchKernelGGL((k_hue_render<false, L, FB>), grid, block, 0, st, hilo, hue, rank, cum,
                                shift, F, n, N, out, bins_out);
    }
}

unsigned blocks_for(long long n, int t) { return (unsigned)((n + t - 1) / t); }

// Workspace carve of a renderer (256-byte aligned pieces).
struct HueLayout {
    size_t hue, hilo, high, pos, ranks, rank, hist, totals, counts, ct, cum, shift, total;
    int ntiles;
};

HueLayout hue_layout(long long N, int n, int frames) {
    HueLayout L;
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t r = o; o = (o + bytes + 255) / 256 * 256; return r; };
    const size_t w = (size_t)N * sizeof(unsigned);
    L.ntiles = (int)((N + kSortTile - 1) / kSortTile);
    L.hue = take(w);
    L.hilo = take((size_t)N * sizeof(unsigned short));
    L.pos = take(w);
    L.high = take((size_t)N * sizeof(unsigned short));
    L.ranks = take(w);
    L.rank = take(w);
    L.hist = take((size_t)kHigh * L.ntiles * sizeof(int));
    L.totals = take(kHigh * sizeof(int));
    L.counts = take((size_t)n * sizeof(int));
    L.ct = take((size_t)frames * n * sizeof(int));
    L.cum = take((size_t)frames * n * sizeof(int));
    L.shift = take((size_t)frames * sizeof(long long));
    L.total = o;
    return L;
}

int hue_check(long long npix, int nbins, int frames) {
    if (npix < 1 || npix > kMaxPix || nbins < 2 || nbins > kMaxBins || frames < 1 ||
        frames > kMaxFrames)
        return OT_ERR_SHAPE;
    return OT_OK;
}

}  // namespace

struct ot_hue {
    long long N = 0;
    int n = 0;
    int cap = 0;                        // frames the plan arrays hold
    int ntiles = 0;
    hipStream_t st = nullptr;
    // hue, hilo, rank: each pixel's hue, max and min channel and rank (raster
    // order, read by the frames); pos: its position in the order of the low
    // digit; high, ranks: the high digits and ranks in that order
    float* hue = nullptr;
    unsigned short *hilo = nullptr, *high = nullptr;
    unsigned *pos = nullptr, *ranks = nullptr, *rank = nullptr;
    int *hist = nullptr, *totals = nullptr;
    int *counts = nullptr, *ct = nullptr, *cum = nullptr;
    long long* shift = nullptr;
    bool have_source = false;
    int planned = 0;                    // frames of the last plan (0: none)
};

extern "C" {

int ot_hue_workspace_size(long long npix, int nbins, int max_frames, size_t* bytes) {
    if (!bytes) return OT_ERR_PARAM;
    const int st = hue_check(npix, nbins, max_frames);
    if (st != OT_OK) return st;
    *bytes = hue_layout(npix, nbins, max_frames).total;
    return OT_OK;
}

int ot_hue_create(long long npix, int nbins, int max_frames, void* stream, void* workspace,
                  size_t ws_bytes, ot_hue** out) {
    if (!out) return OT_ERR_PARAM;
    *out = nullptr;
    const int st = hue_check(npix, nbins, max_frames);
    if (st != OT_OK) return st;
    const HueLayout L = hue_layout(npix, nbins, max_frames);
    if (!workspace || ws_bytes < L.total || (uintptr_t)workspace % 256 != 0) return OT_ERR_SHAPE;
    ot_hue* h = new (std::nothrow) ot_hue;
    if (!h) return OT_ERR_PARAM;
    char* ws = (char*)workspace;
    h->N = npix;
    h->n = nbins;
    h->cap = max_frames;
    h->ntiles = L.ntiles;
    h->st = (hipStream_t)stream;
    h->hue = (float*)(ws + L.hue);
    h->hilo = (unsigned short*)(ws + L.hilo);
    h->pos = (unsigned*)(ws + L.pos);
    h->high = (unsigned short*)(ws + L.high);
    h->ranks = (unsigned*)(ws + L.ranks);
    h->rank = (unsigned*)(ws + L.rank);
    h->hist = (int*)(ws + L.hist);
    h->totals = (int*)(ws + L.totals);
    h->counts = (int*)(ws + L.counts);
    h->ct = (int*)(ws + L.ct);
    h->cum = (int*)(ws + L.cum);
    h->shift = (long long*)(ws + L.shift);
    *out = h;
    return OT_OK;
}

void ot_hue_destroy(ot_hue* h) {
    if (!h) return;
    (void)hipStreamSynchronize(h->st);
    delete h;
}

int ot_hue_set_source(ot_hue* h, const unsigned char* rgb) {
    if (!h || !rgb) return OT_ERR_PARAM;
    hipLaunchKernelGGL(k_fill_i32, dim3(blocks_for(h->n, kThreads)), dim3(kThreads), 0, h->st,
                       h->counts, h->n, 0);
    const dim3 tiles(h->ntiles), block(kSortThreads);
    const size_t lds = (size_t)(h->n + kLow) * sizeof(int);
    if ((uintptr_t)rgb % 4 == 0)
        hipLaunchKernelGGL(k_hue_keys<true>, tiles, block, lds, h->st, rgb, h->N, h->n, h->ntiles,
                           h->hue, h->hilo, h->counts, h->hist);
    else
        hipLaunchKernelGGL(k_hue_keys<false>, tiles, block, lds, h->st, rgb, h->N, h->n, h->ntiles,
                           h->hue, h->hilo, h->counts, h->hist);
    // stable radix sort of the keys (sort_key): equal hues keep raster order
    hipLaunchKernelGGL(k_sort_scan, dim3(kLow), dim3(kScanThreads), 0, h->st, h->hist, h->ntiles,
                       h->totals);
    hipLaunchKernelGGL(k_sort_low, tiles, block, 0, h->st, h->hue, h->N, h->ntiles, h->hist,
                       h->totals, h->pos, h->high);
    hipLaunchKernelGGL(k_sort_hist, tiles, block, 0, h->st, h->high, h->N, h->ntiles, h->hist);
    hipLaunchKernelGGL(k_sort_scan, dim3(kHigh), dim3(kScanThreads), 0, h->st, h->hist, h->ntiles,
                       h->totals);
    hipLaunchKernelGGL(k_sort_high, tiles, block, 0, h->st, h->high, h->N, h->ntiles, h->hist,
                       h->totals, h->ranks);
    hipLaunchKernelGGL(k_sort_gather, tiles, block, 0, h->st, h->pos, h->ranks, h->N,
                       h->ntiles, h->rank);
    if (hipGetLastError() != hipSuccess) return OT_ERR_HIP;
    h->have_source = true;
    h->planned = 0;
    return OT_OK;
}

int ot_hue_histogram(ot_hue* h, int* counts, float* density) {
    if (!h) return OT_ERR_PARAM;
    if (!h->have_source) return OT_ERR_STATE;
    if (counts &&
        hipMemcpyAsync(counts, h->counts, h->n * sizeof(int), hipMemcpyDeviceToDevice, h->st) !=
            hipSuccess)
        return OT_ERR_HIP;
    if (density)
        hipLaunchKernelGGL(k_hue_density, dim3(blocks_for(h->n, kThreads)), dim3(kThreads), 0,
                           h->st, h->counts, h->n, h->N, density);
    return hipGetLastError() == hipSuccess ? OT_OK : OT_ERR_HIP;
}

int ot_hue_plan(ot_hue* h, const float* targets, int frames) {
    if (!h || !targets || frames < 1 || frames > kMaxFrames) return OT_ERR_PARAM;
    if (!h->have_source) return OT_ERR_STATE;
    if (frames > h->cap) {
        h->planned = 0;
        return OT_ERR_SHAPE;
    }
    hipLaunchKernelGGL(k_hue_plan, dim3(frames), dim3(kPlanThreads), 0, h->st, targets, h->counts,
                       h->n, h->N, h->ct, h->cum, h->shift);
    if (hipGetLastError() != hipSuccess) return OT_ERR_HIP;
    h->planned = frames;
    return OT_OK;
}

int ot_hue_apply(ot_hue* h, unsigned char* rgb_out, int* bins_out) {
    if (!h || !rgb_out) return OT_ERR_PARAM;
    if (!h->planned) return OT_ERR_STATE;
    const int F = h->planned;
    const unsigned gb = blocks_for((h->N + 3) / 4, kThreads);
    const unsigned blocks = gb < kRenderBlocks ? gb : kRenderBlocks;
    // every frame's image 4-byte aligned and bins 16-byte aligned
    const bool vec = ((uintptr_t)rgb_out % 4 == 0) &&
                     ((uintptr_t)bins_out % 16 == 0) &&
                     (F == 1 || ((3 * h->N) % 4 == 0 && (!bins_out || h->N % 4 == 0)));
    switch (32 - __builtin_clz(h->n - 1)) {    // 2 <= n <= kMaxBins
#define OT_HUE_RENDER(L) \
    case L: render_launch<L>(vec, blocks, h->st, h->hilo, h->hue, h->rank, h->cum, h->shift, F, h->n, \
                             h->N, rgb_out, bins_out); break;
        OT_HUE_RENDER(1) OT_HUE_RENDER(2) OT_HUE_RENDER(3) OT_HUE_RENDER(4) OT_HUE_RENDER(5)
        OT_HUE_RENDER(6) OT_HUE_RENDER(7) OT_HUE_RENDER(8) OT_HUE_RENDER(9) OT_HUE_RENDER(10)
        OT_HUE_RENDER(11) OT_HUE_RENDER(12)
#undef OT_HUE_RENDER
    }
    return hipGetLastError() == hipSuccess ? OT_OK : OT_ERR_HIP;
}

int ot_hue_render(ot_hue* h, const float* targets, int frames, unsigned char* rgb_out,
                  int* bins_out) {
    if (!h || !targets || !rgb_out) return OT_ERR_PARAM;
    const int st = ot_hue_plan(h, targets, frames);
    return st != OT_OK ? st : ot_hue_apply(h, rgb_out, bins_out);
}

int ot_hue_plan_info(ot_hue* h, int frame, int* counts, long long* shift) {
    if (!h) return OT_ERR_PARAM;
    if (!h->planned) return OT_ERR_STATE;
    if (frame < 0 || frame >= h->planned) return OT_ERR_PARAM;
    if (counts && hipMemcpyAsync(counts, h->ct + (size_t)frame * h->n, h->n * sizeof(int),
                                 hipMemcpyDeviceToHost, h->st) != hipSuccess)
        return OT_ERR_HIP;
    if (shift && hipMemcpyAsync(shift, h->shift + frame, sizeof(long long),
                                hipMemcpyDeviceToHost, h->st) != hipSuccess)
        return OT_ERR_HIP;
    return hipStreamSynchronize(h->st) == hipSuccess ? OT_OK : OT_ERR_HIP;
}

int ot_hue_rgb_to_hsv(const unsigned char* rgb, long long npix, float* hsv, void* stream) {
    if (npix < 0 || (npix > 0 && (!rgb || !hsv))) return OT_ERR_PARAM;
    if (npix == 0) return OT_OK;
    const unsigned gb = blocks_for(npix, kThreads);
    hipLaunchKernelGGL(k_rgb_to_hsv, dim3(gb < kConvBlocks ? gb : kConvBlocks), dim3(kThreads), 0,
                       (hipStream_t)stream, rgb, npix, hsv);
    return hipGetLastError() == hipSuccess ? OT_OK : OT_ERR_HIP;
}

int ot_hue_hsv_to_rgb(const float* hsv, long long npix, unsigned char* rgb, void* stream) {
    if (npix < 0 || (npix > 0 && (!rgb || !hsv))) return OT_ERR_PARAM;
    if (npix == 0) return OT_OK;
    const unsigned gb = blocks_for(npix, kThreads);
    hipLaunchKernelGGL(k_hsv_to_rgb, dim3(gb < kConvBlocks ? gb : kConvBlocks), dim3(kThreads), 0,
                       (hipStream_t)stream, hsv, npix, rgb);
    return hipGetLastError() == hipSuccess ? OT_OK : OT_ERR_HIP;
}

}  // extern "C"
