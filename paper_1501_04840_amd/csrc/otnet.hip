// Kernels of the warm-start network: convolutions as implicit GEMMs on the
// gfx950 matrix cores (BF16 operands, FP32 accumulation) and the pooling,
// upsampling, loss, optimiser and layout pieces around them.
#include <algorithm>

#include "net_common.h"

namespace otn {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int kThreads = 256;

// Round to nearest even (finite inputs).
__device__ inline bf16_t f2bf(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (bf16_t)(u >> 16);
}
__device__ inline float bf2f(bf16_t h) { return __uint_as_float((uint32_t)h << 16); }

__device__ inline void unpack8(const uint4& v, float* f) {
    const bf16_t* h = reinterpret_cast<const bf16_t*>(&v);
#pragma unroll
    for (int q = 0; q < 8; ++q) f[q] = bf2f(h[q]);
}
__device__ inline uint4 pack8(const float* f) {
    uint4 v;
    bf16_t* h = reinterpret_cast<bf16_t*>(&v);
#pragma unroll
    for (int q = 0; q < 8; ++q) h[q] = f2bf(f[q]);
    return v;
}

// ---- convolutions and input gradients --------------------------------------
//
// out[p][n] = sum_k A[p][k] W[n][k], k = (tap, c).  A block owns 64 pixels (TI
// images x TH rows x TW columns, or 64 consecutive pixels of a 1x1 layer) and
// 32 WN outputs.  Its pixels with the one-pixel border, all channels, are
// staged in LDS once and serve every tap, so the K loop has no barrier: a wave
// reads its pixel fragments from LDS and its weights, stored in fragment order
// (one contiguous KB per fragment and 16 K entries), straight from L2, AHEAD
// steps ahead.  With 64 x 64 block tiles that gathered both operands into LDS
// for every 32 K entries, the address divisions and the two barriers per stage
// held the 64 x 64 network's forward pass of 32 images to 108 TFLOP/s (548 us
// in 15 launches); this form takes 270 us (219 TFLOP/s): 48 us (315 TFLOP/s)
// for the widest layer, 7-20 us for the others, where few fragments are left
// per compute unit and a wave's serial K loop and the launch count, 39 us for
// the FP32 head, bound by its 99 MB.  The sum over k runs in the same steps of
// 16 in the same order, so results are the same bit for bit.
//
// Lane l of a wave holds K entries 8 (l / 32) + 0..7 of row l mod 32 of each
// operand; accumulator entry r of lane l is row 8 (r / 4) + 4 (l / 32) + r mod
// 4, column l mod 32.  BF16 outputs take the weights as rows and the pixels as
// columns (a lane then owns 16 outputs of one pixel, stored as 16-byte
// pieces); the FP32 head takes the pixels as rows (its unaligned rows are
// stored one float per lane, 32 consecutive outputs together).
//
// LDS layout: 16-byte units of eight channels; a pixel is `pu` units (odd, so
// that eight neighbours fall in distinct bank groups), a row of the staged tile
// `ru` units (8 mod 16: the next row takes the other eight groups).
// Weight fragments in flight: 16 (at 8 the weights' latency still showed:
// their first reader fetches them from beyond its L2), 4 for fewer steps.
constexpr int kConvAhead = kConvPad / 512;
constexpr size_t kConvLds = 156 * 1024;             // staged tiles up to this size

struct ConvGeom {
    int th_log, tw_log;        // tile rows and columns (3x3 layers)
    int bw, bh;                // staged columns and rows of one image
    int ntx, nty;              // tiles along x and y
    int nc8;                   // units of 8 channels per pixel
    int pu, ru, iu;            // LDS units per pixel, row, image
    unsigned mc, mw, mh;       // reciprocals of nc8, bw and bh (e / d = mulhi(e, m), e < 2^16)
    int entries;               // units to stage
};

// Steps of the offset table: whole groups and one more.
__host__ __device__ inline int conv_table(int nsteps, int ahead) {
    return (nsteps + ahead - 1) / ahead * ahead + ahead;
}

template <int PF, int WP, int WN, int AHEAD, bool STAGED, int EPI>
__global__ void __launch_bounds__(64 * WP * WN) k_conv(ConvArgs a, ConvGeom g) {
    static_assert(PF * WP == 2, "64 pixels per block");
    constexpr bool SWAP = EPI != EPI_F32;
    extern __shared__ __attribute__((aligned(16))) uint4 tile[];
    const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wp = wave % WP, wn = wave / WP;
    constexpr int NT = 64 * WP * WN;
    // tile origin: image b0 and (y0, x0), or the linear pixel m0 of a 1x1 layer
    const int tl = blockIdx.x;
    const bool one = a.taps == 1;
    int b0 = 0, y0 = 0, x0 = 0;
    const int ti = 64 >> (g.th_log + g.tw_log);
    if (!one) {
        const int per = g.ntx * g.nty, bi = tl / per, r = tl - bi * per;
        b0 = bi * ti;
        y0 = (r / g.ntx) << g.th_log;
        x0 = (r % g.ntx) << g.tw_log;
    }
    if (STAGED) {
        // Every unit of the tile and its border, zeros outside the image.  The
        // loads are unconditional (outside: the tensor's first unit), eight in
        // flight per thread: a load under a condition was waited for before the
        // next one, which was most of the kernel's time.
        constexpr int Q = 8;
        for (int e0 = threadIdx.x; e0 < g.entries; e0 += Q * NT) {
            uint4 v[Q];
            int at[Q];
            bool in[Q];
#pragma unroll
            for (int j = 0; j < Q; ++j) {
                const int e = e0 + j * NT;
                const int px = g.nc8 == 1 ? e : (int)__umulhi(e, g.mc), u = e - px * g.nc8;
                long long q;
                if (one) {
                    q = 64ll * tl + px;
                    in[j] = e < g.entries && q < a.M;
                    at[j] = (px >> 3) * g.ru + (px & 7) * g.pu + u;
                } else {
                    const int row = __umulhi(px, g.mw), hx = px - row * g.bw;
                    const int im = __umulhi(row, g.mh), hy = row - im * g.bh;
                    const int b = b0 + im, y = y0 + hy - 1, x = x0 + hx - 1;
                    in[j] = e < g.entries && b < a.nb && (unsigned)y < (unsigned)a.H &&
                            (unsigned)x < (unsigned)a.W;
                    q = (long long)(b * a.H + y) * a.W + x;
                    at[j] = im * g.iu + hy * g.ru + hx * g.pu + u;
                }
                v[j] = *reinterpret_cast<const uint4*>(a.src + (in[j] ? q * a.src_ld + 8 * u : 0));
            }
#pragma unroll
            for (int j = 0; j < Q; ++j)
                if (e0 + j * NT < g.entries) tile[at[j]] = in[j] ? v[j] : make_uint4(0, 0, 0, 0);
        }
    }
    // Where each step's K entries lie in the staged tile, relative to a pixel's
    // first unit: the byte offset of unit k8 = 2 s + half at steps[half][s], for
    // nsteps rounded up to whole groups and one group more (those read the
    // pixel's own first unit).  The K loop reads a group's offsets with a few
    // 16-byte LDS loads instead of walking taps and channels.
    const int nk8 = a.K >> 3, nsteps = (nk8 + 1) >> 1, tab = conv_table(nsteps, AHEAD);
    int* const steps = reinterpret_cast<int*>(tile + (STAGED ? ti * g.iu : 0));
    if (STAGED)
        for (int e = threadIdx.x; e < 2 * tab; e += NT) {
            const int h = e >= tab ? 1 : 0, k8 = 2 * (e - h * tab) + h;
            int o = 0;
            if (k8 < nk8) {
                const int tap = g.nc8 == 1 ? k8 : (int)__umulhi(k8, g.mc), cu = k8 - tap * g.nc8;
                const int dy = tap / 3, dx = tap - 3 * dy;
                o = 16 * (dy * g.ru + dx * g.pu + cu);
            }
            steps[e] = o;
        }
    // An unstaged source has no table (its length would grow with the channels):
    // the loads come in the order of the steps and walk the unit and the tap of
    // this half's next step (past K: a unit of the image that no product uses).
    int wc = half, wt = 0;
    auto walk = [&](int n) {
        wc += n;
#pragma unroll
        for (int q = 0; q < 2; ++q)                      // (one channel unit: two taps a step)
            if (wc >= g.nc8) {
                wc -= g.nc8;
                ++wt;
            }
    };
    walk(0);
    // this lane's pixel of each fragment
    int base[PF], row0[PF], col0[PF];
    long long pix[PF];                                   // pixel index, -1 outside
#pragma unroll
    for (int f = 0; f < PF; ++f) {
        const int q = (wp * PF + f) * 32 + l32;
        if (one) {
            const int m = 64 * tl + q;
            base[f] = (q >> 3) * g.ru + (q & 7) * g.pu;
            pix[f] = m < a.M ? m : -1;
            row0[f] = col0[f] = 0;
        } else {
            const int tx = q & ((1 << g.tw_log) - 1), ty = (q >> g.tw_log) & ((1 << g.th_log) - 1);
            const int im = q >> (g.tw_log + g.th_log), b = b0 + im, y = y0 + ty, x = x0 + tx;
            base[f] = im * g.iu + ty * g.ru + tx * g.pu;
            pix[f] = b < a.nb && y < a.H && x < a.W ? (long long)(b * a.H + y) * a.W + x : -1;
            row0[f] = y;
            col0[f] = x;
        }
    }
    if (STAGED)
#pragma unroll
        for (int f = 0; f < PF; ++f) base[f] *= 16;
    auto load_a = [&](bf16x8 (&fa)[PF], int o) {
        if (STAGED) {
#pragma unroll
            for (int f = 0; f < PF; ++f)
                fa[f] = *reinterpret_cast<const bf16x8*>(reinterpret_cast<const char*>(tile) + base[f] + o);
        } else {
            const int dy = wt / 3 - 1, dx = wt - 3 * (wt / 3) - 1;
#pragma unroll
            for (int f = 0; f < PF; ++f) {
                uint4 v = make_uint4(0, 0, 0, 0);
                const int y = one ? 0 : row0[f] + dy, x = one ? 0 : col0[f] + dx;
                const bool in = pix[f] >= 0 &&
                                (one || ((unsigned)y < (unsigned)a.H && (unsigned)x < (unsigned)a.W));
                const long long q = one ? pix[f] : pix[f] + (long long)dy * a.W + dx;
                if (in) v = *reinterpret_cast<const uint4*>(a.src + q * a.src_ld + 8 * wc);
                fa[f] = *reinterpret_cast<const bf16x8*>(&v);
            }
            walk(2);
        }
    };
    const int nf = blockIdx.y * WN + wn, n0 = nf * 32;
    const bool live = n0 < a.N;                          // wave-uniform
    // weight fragments of steps s .. s + AHEAD - 1 (reads past the last
    // step stay inside the padded weight buffer)
    const bf16x8* wq = reinterpret_cast<const bf16x8*>(a.wmat) + (long long)(live ? nf : 0) * nsteps * 64;
    bf16x8 wb[AHEAD];
#pragma unroll
    for (int j = 0; j < AHEAD; ++j) wb[j] = wq[j * 64 + lane];
    floatx16 acc[PF];
#pragma unroll
    for (int f = 0; f < PF; ++f)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[f][r] = 0.f;
    __syncthreads();
    if (!live) return;
    auto mma = [&](const bf16x8& w, const bf16x8 (&fa)[PF]) {
#pragma unroll
        for (int f = 0; f < PF; ++f)
            acc[f] = SWAP ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(w, fa[f], acc[f], 0, 0, 0)
                          : __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[f], w, acc[f], 0, 0, 0);
    };
    // Groups of AHEAD steps, straight-line: the next step's pixels are
    // read and the weights AHEAD steps on are requested before a step's
    // products (the scheduling barriers keep them there).
    const int4* so = reinterpret_cast<const int4*>(steps + half * tab);
    constexpr int G4 = AHEAD / 4;
    int4 on[G4] = {};
    int oc[AHEAD];
    bf16x8 fa[2][PF];
    auto request = [&] {                                 // a group's offsets
        if (STAGED)
#pragma unroll
            for (int q = 0; q < G4; ++q) on[q] = so[q];
    };
    request();
    load_a(fa[0], on[0].x);
    int s = 0;
    auto take = [&] {                                    // this group's offsets; the next one's loads
#pragma unroll
        for (int q = 0; q < G4; ++q) {
            oc[4 * q] = on[q].x;
            oc[4 * q + 1] = on[q].y;
            oc[4 * q + 2] = on[q].z;
            oc[4 * q + 3] = on[q].w;
        }
        so += G4;
        request();
    };
    const int whole = nk8 >> 1;                          // steps wholly inside K
    for (; s + AHEAD <= whole; s += AHEAD) {
        take();
        wq += AHEAD * 64;
#pragma unroll
        for (int j = 0; j < AHEAD; ++j) {
            load_a(fa[(j + 1) & 1], j + 1 < AHEAD ? oc[j + 1] : on[0].x);
            const bf16x8 w = wb[j];
            wb[j] = wq[j * 64 + lane];
            __builtin_amdgcn_sched_barrier(0);
            mma(w, fa[j & 1]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    take();
#pragma unroll
    for (int j = 0; j < AHEAD; ++j) {
        if (s + j >= nsteps) break;                      // uniform
        if (j + 1 < AHEAD) load_a(fa[(j + 1) & 1], oc[j + 1]);
        if (s + j >= whole && half)                      // the upper half is past K
#pragma unroll
            for (int f = 0; f < PF; ++f) fa[j & 1][f] = bf16x8{};
        mma(wb[j], fa[j & 1]);
    }
    if (!SWAP) {
        const int col = n0 + l32;
#pragma unroll
        for (int f = 0; f < PF; ++f)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                // the pixel of accumulator row r is held by lane `row`
                const int row = (r >> 2) * 8 + half * 4 + (r & 3);
                const int m = __shfl((int)pix[f], row, 64);
                if (m < 0 || col >= a.dst_n) continue;
                reinterpret_cast<float*>(a.dst)[(long long)m * a.dst_ld + a.dst_off + col] = acc[f][r] + a.bias[col];
            }
        return;
    }
#pragma unroll
    for (int f = 0; f < PF; ++f) {
        unsigned h[8];                                   // outputs 8 (q / 2) + 4 half + 2 (q mod 2) + 0, 1
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int n = n0 + 8 * (q >> 1) + 4 * half + 2 * (q & 1);
            float v0 = acc[f][2 * q], v1 = acc[f][2 * q + 1];
            if (EPI == EPI_RELU) {
                v0 = fmaxf(v0 + (n < a.N ? a.bias[n] : 0.f), 0.f);
                v1 = fmaxf(v1 + (n < a.N ? a.bias[n + 1] : 0.f), 0.f);
            }
            h[q] = (unsigned)f2bf(v0) | ((unsigned)f2bf(v1) << 16);
        }
        // lanes l and l + 32 exchange so that each holds eight consecutive outputs
#pragma unroll
        for (int q = 0; q < 8; q += 4) {
            const auto s0 = __builtin_amdgcn_permlane32_swap(h[q], h[q + 2], false, false);
            const auto s1 = __builtin_amdgcn_permlane32_swap(h[q + 1], h[q + 3], false, false);
            const int n = n0 + 8 * (q >> 1) + 8 * half;
            if (pix[f] < 0 || n >= a.dst_n) continue;
            uint4 v = make_uint4(s0[0], s1[0], s0[1], s1[1]);
            if (EPI == EPI_MASK) {
                const uint4 mk = *reinterpret_cast<const uint4*>(a.mask + pix[f] * a.mask_ld + n);
                float m[8];
                unpack8(mk, m);
                bf16_t* o = reinterpret_cast<bf16_t*>(&v);
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = m[e] > 0.f ? o[e] : (bf16_t)0;
            }
            *reinterpret_cast<uint4*>(reinterpret_cast<bf16_t*>(a.dst) + pix[f] * a.dst_ld + a.dst_off + n) = v;
        }
    }
}

ConvGeom conv_geom(const ConvArgs& a) {
    ConvGeom g{};
    g.nc8 = a.cin / 8;
    if (a.taps == 1) {
        g.th_log = g.tw_log = 3;
        g.bw = g.bh = 8;
        g.ntx = (a.M + 63) / 64;
        g.nty = 1;
    } else {
        // small images share a tile: the least power of two that holds a side
        auto lg = [](int n) { return n > 4 ? 3 : n > 2 ? 2 : n > 1 ? 1 : 0; };
        g.th_log = lg(a.H);
        g.tw_log = lg(a.W);
        g.bw = (1 << g.tw_log) + 2;
        g.bh = (1 << g.th_log) + 2;
        g.ntx = (a.W + (1 << g.tw_log) - 1) >> g.tw_log;
        g.nty = (a.H + (1 << g.th_log) - 1) >> g.th_log;
    }
    g.pu = g.nc8 | 1;
    g.ru = g.bw * g.pu;
    g.ru += (24 - (g.ru & 15)) & 15;
    g.iu = g.bh * g.ru;
    const int ti = 64 >> (g.th_log + g.tw_log);
    g.entries = ti * g.bh * g.bw * g.nc8;
    auto rec = [](int d) { return (unsigned)(((1ull << 32) + d - 1) / d); };
    g.mc = rec(g.nc8);
    g.mw = rec(g.bw);
    g.mh = rec(g.bh);
    return g;
}

template <int PF, int WP, int WN, int AHEAD, int EPI>
void conv_launch_a(const ConvArgs& a, const ConvGeom& g, hipStream_t st) {
    const int ti = 64 >> (g.th_log + g.tw_log);
    const size_t tab = 8 * (size_t)conv_table((a.K + 15) / 16, AHEAD), lds = 16 * (size_t)ti * g.iu + tab;
    const unsigned tiles = a.taps == 1 ? g.ntx : (unsigned)((a.nb + ti - 1) / ti * g.ntx * g.nty);
    const dim3 grid(tiles, ((a.N + 31) / 32 + WN - 1) / WN), block(64 * WP * WN);
    // (the reciprocals need e < 2^16)
    if (lds <= kConvLds && g.entries < 65536)
        hipLaunchKernelGGL((k_conv<PF, WP, WN, AHEAD, true, EPI>), grid, block, lds, st, a, g);
    else
        hipLaunchKernelGGL((k_conv<PF, WP, WN, AHEAD, false, EPI>), grid, block, 0, st, a, g);
}

template <int PF, int WP, int WN, int EPI>
void conv_launch(const ConvArgs& a, const ConvGeom& g, hipStream_t st) {
    if (a.K >= 16 * kConvAhead) conv_launch_a<PF, WP, WN, kConvAhead, EPI>(a, g, st);
    else conv_launch_a<PF, WP, WN, 4, EPI>(a, g, st);
}

template <int EPI>
void conv_dispatch(const ConvArgs& a, hipStream_t st) {
    const ConvGeom g = conv_geom(a);
    const int ti = 64 >> (g.th_log + g.tw_log), nf = (a.N + 31) / 32;
    const long long tiles = a.taps == 1 ? g.ntx : (long long)((a.nb + ti - 1) / ti) * g.ntx * g.nty;
    // Few fragments: a wave each (half the serial K loop per wave); many: two
    // pixel fragments per wave (a weight fragment loaded serves both).  Waves
    // along the outputs share the staged tile, as long as blocks remain for
    // every compute unit.
    if (tiles * nf < 1024 || nf == 1) {
        if (nf >= 2 && tiles * nf >= 512) conv_launch<1, 2, 2, EPI>(a, g, st);
        else conv_launch<1, 2, 1, EPI>(a, g, st);
    } else if (nf >= 4 && tiles * nf >= 2048) {
        conv_launch<2, 1, 4, EPI>(a, g, st);
    } else {
        conv_launch<2, 1, 2, EPI>(a, g, st);
    }
}

// ---- weight gradients ------------------------------------------------------
//
// dW[(tap, c)][n] = sum over pixels q of src[q + tap][c] dz[q][n]: the
// contraction runs over pixels, while both tensors hold channels together.  A
// block walks tiles of 64 pixels (as k_conv's); it stages the tile with its
// border (the channels its rows need) and the tile's dz in LDS as they are and
// reads both operands with transposing LDS loads (four pixels x 16 channels per
// 16 lanes), so every tap reads the one staged tile.  Its 32 x 32 fragments of
// dW, MW x NW per wave, stay in registers over all of its tiles, and the next
// tile's loads are in flight during a tile's products.  Gathering each of the
// nine taps' pixels and writing them to LDS transposed element by element took
// 880 us for the 64 x 64 network and 32 images (67 TFLOP/s); this form 385 us
// (152 TFLOP/s): 64 us for the widest layer, 15-43 us for the others, of which
// the first tile's decoding and loads and the partial's stores are 8-10 us.
//
// Rows of dW are numbered i = (c / 32) taps + tap (fragments of 32 channels);
// the bias gradient is a product with a row of ones, on the last wave of the
// first row group.  NWAVE: the waves split the outputs instead of the rows
// (1x1 layers: one or two row fragments, many outputs).
typedef short short4v __attribute__((ext_vector_type(4)));
typedef short short8v __attribute__((ext_vector_type(8)));

struct WgradGeom {
    int th_log, tw_log, ti;    // tile rows, columns and images (3x3 layers)
    int bw, bh;                // staged columns and rows of one image
    int ntx, nty, tiles;       // tiles along x and y, in all
    unsigned mw, mh;           // reciprocals of bw and bh
    int cf, mf;                // fragments of 32 channels, of 32 rows (cf taps)
    int per_wave, group;       // row fragments per wave and block
    int per_split;             // tiles per split
};

// Channel units of 8 staged by row group gy, and the first fragment's channel
// fragment.
__host__ __device__ inline int wgrad_units(const WgradGeom& g, int taps, int cin, int gy, int* cb0) {
    const int f0 = gy * g.group, f1 = f0 + g.group < g.mf ? f0 + g.group : g.mf;
    *cb0 = f0 / taps;
    const int c1 = 32 * ((f1 - 1) / taps + 1);
    return (c1 < cin ? c1 : cin) / 8 - 4 * *cb0;
}
// LDS pitch of a pixel of n units: 4 mod 8 units (64 bytes times an odd
// number), so that the four pixels a transposing read takes from 32 lanes, 64
// bytes each, fall in distinct banks, and at least n rounded up to whole
// fragments of 4 units.
__host__ __device__ inline int wgrad_pitch(int n) { return (n + 3) / 8 * 8 + 4; }

__device__ __forceinline__ bf16x8 tr_read(const char* lds, int at0, int at1) {
    typedef __attribute__((address_space(3))) short4v lds_short4;
    const short4v x = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)(lds + at0));
    const short4v y = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)(lds + at1));
    const short8v v = __builtin_shufflevector(x, y, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, v);
}

// Q: units of a tile in flight per thread.  Where the accumulators leave room,
// two waves share a SIMD.
template <int MW, int NW, bool NWAVE, int Q>
__global__ void __launch_bounds__(kThreads, Q < 12 && 16 * (MW + 1) * NW + 8 * Q <= 160 ? 2 : 1) k_wgrad(ConvArgs a, WgradGeom g) {
    extern __shared__ __attribute__((aligned(16))) uint4 tile[];
    constexpr int NB = NWAVE ? 4 * NW : NW;              // output fragments per block
    const int lane = threadIdx.x & 63, half = lane >> 5, i16 = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool one = a.taps == 1;
    const int gy = blockIdx.y, n0 = blockIdx.z * NB * 32;
    int cb0;
    const int nu = wgrad_units(g, a.taps, a.cin, gy, &cb0);
    const int pu = wgrad_pitch(nu), ru = g.bw * pu, iu = g.bh * ru;
    const int nd = min(a.N - n0, NB * 32) / 8, du = wgrad_pitch(nd);
    const int dz0 = g.ti * iu;
    const int es = g.ti * g.bh * g.bw * nu, ed = 64 * nd, entries = es + ed;
    const unsigned mu = 0xFFFFFFFFu / nu + 1, md = 0xFFFFFFFFu / nd + 1;
    const int t0 = blockIdx.x * g.per_split, t1 = min(t0 + g.per_split, g.tiles);

    // A thread's units of a tile, decoded once: LDS place (14 bits), border
    // column (7), border row (4), image (6) and tensor (1: dz) in one word, and
    // the element offset from the tile's origin.  A 1x1 layer is one image of
    // one row of K pixels.
    const int W = one ? a.K : a.W, H = one ? 1 : a.H;
    unsigned pk[Q];
    int rel[Q];
    uint4 v[Q];
    auto decode = [&](int e0) {
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            const int e = min(e0 + j * kThreads + (int)threadIdx.x, entries - 1);
            int at, hx, hy, im, u;
            const bool d = e >= es;
            if (!d) {
                const int px = nu == 1 ? e : (int)__umulhi(e, mu);
                u = e - px * nu;
                const int row = __umulhi(px, g.mw), col = px - row * g.bw;
                im = one ? 0 : (int)__umulhi(row, g.mh);
                hy = one ? 1 : row - im * g.bh;
                hx = one ? px + 1 : col;
                at = im * iu + (one ? row : hy) * ru + col * pu + u;
            } else {
                const int f = e - es, px = nd == 1 ? f : (int)__umulhi(f, md);
                u = f - px * nd;
                im = one ? 0 : px >> (g.tw_log + g.th_log);
                hy = one ? 1 : ((px >> g.tw_log) & ((1 << g.th_log) - 1)) + 1;
                hx = one ? px + 1 : (px & ((1 << g.tw_log) - 1)) + 1;
                at = dz0 + px * du + u;
            }
            // images past the tile's (their pixels are zero) read no image
            if (im >= g.ti) hx = 127;
            pk[j] = (unsigned)at | (unsigned)hx << 14 | (unsigned)hy << 21 | (unsigned)im << 25 | (d ? 1u << 31 : 0u);
            const int q = (im * H + hy - 1) * W + hx - 1;
            rel[j] = q * (d ? a.dz_ld : a.src_ld) + 8 * u + (d ? n0 : 32 * cb0);
        }
    };
    unsigned inside = 0;
    auto load = [&](int t) {
        int b0 = 0, y0 = 0, x0 = 64 * t;
        if (!one) {
            const int per = g.ntx * g.nty, bi = t / per, r = t - bi * per;
            b0 = bi * g.ti;
            y0 = (r / g.ntx) << g.th_log;
            x0 = (r % g.ntx) << g.tw_log;
        }
        const long long q0 = (long long)(b0 * H + y0) * W + x0;
        const bf16_t* const s0 = a.src + q0 * a.src_ld;
        const bf16_t* const d0 = a.dz + q0 * a.dz_ld;
        const int nim = one ? 1 : a.nb - b0;
        inside = 0;
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            const int hx = pk[j] >> 14 & 127, hy = pk[j] >> 21 & 15, im = pk[j] >> 25 & 63;
            const bool in = hx != 127 && im < nim && (unsigned)(y0 + hy - 1) < (unsigned)H &&
                            (unsigned)(x0 + hx - 1) < (unsigned)W;
            const bf16_t* s = (int)pk[j] < 0 ? d0 : s0;
            v[j] = *reinterpret_cast<const uint4*>(in ? s + rel[j] : a.src);
            inside |= in ? 1u << j : 0u;
        }
    };
    auto store = [&](int e0) {
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            if (e0 + j * kThreads + (int)threadIdx.x < entries)
                tile[pk[j] & 16383] = inside >> j & 1 ? v[j] : make_uint4(0, 0, 0, 0);
        }
    };

    // this lane's place in the transposing reads: pixel 16 ks + 8 half + 4 j +
    // i16 / 4 of the tile, channels 16 ((lane / 16) mod 2) + 4 (i16 mod 4)
    const int lch = 32 * ((lane >> 4) & 1) + 8 * (i16 & 3);   // bytes
    int px[4][2];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int p = 16 * ks + 8 * half + 4 * j + (i16 >> 2);
            int at;
            if (one) {
                at = (p >> 3) * ru + (p & 7) * pu;
            } else {
                const int tx = p & ((1 << g.tw_log) - 1), ty = (p >> g.tw_log) & ((1 << g.th_log) - 1);
                const int im = p >> (g.tw_log + g.th_log);
                at = im < g.ti ? im * iu + ty * ru + tx * pu : 0;
            }
            px[ks][j] = 16 * at + lch;
        }
    const int dzl = 16 * (dz0 + (8 * half + (i16 >> 2)) * du) + lch;
    // byte offset of each row fragment: its tap and channels (past the last:
    // some fragment's, not stored)
    const int f0 = gy * g.group + (NWAVE ? 0 : wave * g.per_wave);
    const int fend = min(min(f0 + g.per_wave, (gy + 1) * g.group), g.mf);
    int foff[MW];
#pragma unroll
    for (int i = 0; i < MW; ++i) {
        const int f = f0 + i < fend ? f0 + i : gy * g.group, cb = f / a.taps, tap = f - cb * a.taps;
        foff[i] = 16 * ((tap / 3) * ru + (tap % 3) * pu + 4 * (cb - cb0));
    }
    const int nb0 = NWAVE ? wave * NW : 0;               // this wave's first output fragment
    const int nlast = (nd + 3) / 4 - 1;                  // the block's last one with outputs
    const bool bias = gy == 0 && (NWAVE || wave == 3);
    floatx16 acc[MW][NW], accb[NW];
#pragma unroll
    for (int j = 0; j < NW; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            accb[j][r] = 0.f;
#pragma unroll
            for (int i = 0; i < MW; ++i) acc[i][j][r] = 0.f;
        }
    const __bf16 w1 = (lane & 31) == 0 ? (__bf16)1.f : (__bf16)0.f;
    const bf16x8 ones = {w1, w1, w1, w1, w1, w1, w1, w1};
    const char* const lds = reinterpret_cast<const char*>(tile);

    const bool ahead = entries <= Q * kThreads;          // a tile's units all fit in registers
    if (ahead) {
        decode(0);
        load(t0);
    }
    for (int t = t0; t < t1; ++t) {
        if (t > t0) __syncthreads();                     // the last tile's reads are done
        if (ahead) {
            store(0);
        } else {
            for (int e0 = 0; e0 < entries; e0 += Q * kThreads) {
                decode(e0);
                load(t);
                store(e0);
            }
        }
        __syncthreads();
        if (ahead && t + 1 < t1) load(t + 1);
        // Steps n = ks MW + i; row fragments are read AH steps ahead and output
        // fragments one ks ahead of their products (the scheduling barriers
        // keep them there: left alone, every product waited for its own read).
        constexpr int AH = 3;
        bf16x8 fb[2][NW], fa[AH + 1];
        auto read_b = [&](int ks) {
#pragma unroll
            for (int j = 0; j < NW; ++j) {
                const int at = dzl + 64 * min(nb0 + j, nlast) + 256 * ks * du;
                fb[ks & 1][j] = tr_read(lds, at, at + 64 * du);
            }
        };
        auto read_a = [&](int n) {
            const int ks = n / MW, i = n % MW;
            fa[n % (AH + 1)] = tr_read(lds, px[ks][0] + foff[i], px[ks][1] + foff[i]);
        };
        read_b(0);
#pragma unroll
        for (int n = 0; n < AH; ++n) read_a(n);
#pragma unroll
        for (int n = 0; n < 4 * MW; ++n) {
            const int ks = n / MW, i = n % MW;
            if (i == 0 && ks < 3) read_b(ks + 1);
            if (n + AH < 4 * MW) read_a(n + AH);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < NW; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[n % (AH + 1)], fb[ks & 1][j], acc[i][j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (i == MW - 1 && bias)
#pragma unroll
                for (int j = 0; j < NW; ++j)
                    accb[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ones, fb[ks & 1][j], accb[j], 0, 0, 0);
        }
    }
    // partial of this split: rows tap cin + c, then the bias row
    float* const out = reinterpret_cast<float*>(a.dst) + (long long)blockIdx.x * a.M * a.N;
#pragma unroll
    for (int j = 0; j < NW; ++j) {
        const int col = n0 + 32 * (nb0 + j) + (lane & 31);
        if (col >= a.N) continue;
#pragma unroll
        for (int i = 0; i < MW; ++i) {
            if (f0 + i >= fend) continue;
            const int f = f0 + i, cb = f / a.taps, tap = f - cb * a.taps;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int c = 32 * cb + (r >> 2) * 8 + half * 4 + (r & 3);
                if (c < a.cin) out[(long long)(tap * a.cin + c) * a.N + col] = acc[i][j][r];
            }
        }
        if (bias && half == 0) out[(long long)(a.M - 1) * a.N + col] = accb[j][0];
    }
}

// The wave tile of a layer: rows x outputs of 32 x 32 fragments.  Narrow
// layers (32 outputs) keep up to 16 row fragments per wave, wider ones share
// each row fragment read between two or four outputs; the row groups are
// evened out, so that a block's waves all have work.
struct WgradTile {
    int mw, nw;
    bool nwave;
};
WgradTile wgrad_tile(int taps, int cin, int cout) {
    const int nf = (cout + 31) / 32, mf = taps * ((cin + 31) / 32);
    if (taps == 1) return {1, 2, true};
    if (nf == 1) return {mf <= 12 ? 3 : mf <= 28 ? 7 : 16, 1, false};
    if (nf < 4) return {mf <= 12 ? 3 : mf <= 20 ? 5 : 7, 2, false};
    return {3, 4, false};
}

WgradGeom wgrad_geom(int taps, int cin, int cout, int nb, int H, int W, int* row_groups,
                     int* col_groups, size_t* lds) {
    const WgradTile w = wgrad_tile(taps, cin, cout);
    WgradGeom g{};
    g.cf = (cin + 31) / 32;
    g.mf = taps * g.cf;
    const int cap = w.nwave ? w.mw : 4 * w.mw, ngr = (g.mf + cap - 1) / cap;
    g.group = (g.mf + ngr - 1) / ngr;
    g.per_wave = w.nwave ? g.group : (g.group + 3) / 4;
    *row_groups = (g.mf + g.group - 1) / g.group;
    const int NB = w.nwave ? 4 * w.nw : w.nw;
    *col_groups = ((cout + 31) / 32 + NB - 1) / NB;
    ConvArgs a{};
    a.taps = taps; a.cin = cin; a.nb = nb; a.H = H; a.W = W; a.M = nb * H * W;
    const ConvGeom c = conv_geom(a);
    g.th_log = c.th_log; g.tw_log = c.tw_log; g.bw = c.bw; g.bh = c.bh;
    g.ntx = c.ntx; g.nty = c.nty; g.mw = c.mw; g.mh = c.mh;
    g.ti = taps == 1 ? 1 : 64 >> (g.th_log + g.tw_log);
    const int nd = std::min((cout + 7) / 8, 4 * NB);
    for (;;) {           // tiny images: as many per tile as LDS holds
        size_t most = 0;
        for (int gy = 0; gy < *row_groups; ++gy) {
            int cb0;
            const int nu = wgrad_units(g, taps, cin, gy, &cb0);
            most = std::max(most, (size_t)g.ti * g.bh * g.bw * wgrad_pitch(nu));
        }
        *lds = 16 * (most + 64 * (size_t)wgrad_pitch(nd));
        if (*lds <= kConvLds || g.ti == 1) break;
        g.ti /= 2;
    }
    g.tiles = taps == 1 ? c.ntx : (nb + g.ti - 1) / g.ti * c.ntx * c.nty;
    return g;
}

// Sum of the splits' partials: 64 consecutive entries per block, each wave
// every fourth split with eight loads in flight (a thread per entry waiting on
// its chain of up to 342 loads took 430 us over the layers of the 64 x 64
// network; now 146).
__global__ void __launch_bounds__(kThreads) k_wgrad_reduce(const float* __restrict__ part, int splits,
                                                          long long mn, float* out) {
    __shared__ float red[kThreads / 64][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    constexpr int NWV = kThreads / 64, U = 8;
    const long long i = (long long)blockIdx.x * 64 + lane;
    const float* s = part + (i < mn ? i : 0);
    float acc = 0.f;
    for (int z = w; z < splits; z += NWV * U) {
        float v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = z + NWV * u < splits ? s[(z + NWV * u) * mn] : 0.f;
#pragma unroll
        for (int u = 0; u < U; ++u) acc += v[u];
    }
    red[w][lane] = acc;
    __syncthreads();
    if (w == 0 && i < mn) {
        float t = red[0][lane];
#pragma unroll
        for (int q = 1; q < NWV; ++q) t += red[q][lane];
        out[i] = t;
    }
}

// BF16 copy of the FP32 input, channels padded to ld (a multiple of 8) with
// zeros: eight output channels per thread, one 16-byte store.  Bound by HBM
// (4 bytes read, 2 written per channel): 131072 pixels of 195 channels take
// 26 us (5.9 TB/s) against 59 us with one channel and one 64-bit division per
// thread.
template <typename I>
__global__ void __launch_bounds__(kThreads) k_pack_input(const float* __restrict__ x, int in_ch,
                                                        long long npix, bf16_t* __restrict__ out,
                                                        int ld) {
    const I l8 = (I)(ld / 8);
    const I i = (I)blockIdx.x * kThreads + threadIdx.x;
    if (i >= (I)npix * l8) return;
    const I p = i / l8;
    const int c = (int)(i - p * l8) * 8;
    const float* s = x + (long long)p * in_ch + c;
    float f[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) f[q] = c + q < in_ch ? s[q] : 0.f;
    *reinterpret_cast<uint4*>(out + (long long)i * 8) = pack8(f);
}

// dst[b][y][x][c] = mean of the 2x2 source block (8 channels per thread).
__global__ void __launch_bounds__(kThreads) k_pool(View src, int C, int nb, int H, int W,
                                                  bf16_t* dst) {
    const int h = H / 2, w = W / 2, c8 = C / 8;
    const long long n = (long long)nb * h * w * c8;
    const long long i = (long long)blockIdx.x * kThreads + threadIdx.x;
    if (i >= n) return;
    const int c = (int)(i % c8) * 8;
    const long long p = i / c8;
    const int x = (int)(p % w), y = (int)((p / w) % h), b = (int)(p / ((long long)w * h));
    float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int dy = 0; dy < 2; ++dy)
        for (int dx = 0; dx < 2; ++dx) {
            const long long q = ((long long)(b * H + 2 * y + dy) * W + 2 * x + dx);
            float f[8];
            unpack8(*reinterpret_cast<const uint4*>(src.ptr + q * src.ld + c), f);
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e] += f[e];
        }
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] *= 0.25f;
    *reinterpret_cast<uint4*>(dst + p * C + c) = pack8(acc);
}

// dst (2h x 2w, channels [0, C)) = nearest upsampling of src (h x w x C).
__global__ void __launch_bounds__(kThreads) k_upsample(const bf16_t* src, int C, int nb, int h,
                                                      int w, View dst) {
    const int H = 2 * h, W = 2 * w, c8 = C / 8;
    const long long n = (long long)nb * H * W * c8;
    const long long i = (long long)blockIdx.x * kThreads + threadIdx.x;
    if (i >= n) return;
    const int c = (int)(i % c8) * 8;
    const long long p = i / c8;
    const int x = (int)(p % W), y = (int)((p / W) % H), b = (int)(p / ((long long)W * H));
    const long long q = (long long)(b * h + y / 2) * w + x / 2;
    *reinterpret_cast<uint4*>(dst.ptr + p * dst.ld + c) =
        *reinterpret_cast<const uint4*>(src + q * C + c);
}

// out (h x w x C) = (sum of the 2x2 block of g's channels [0, C)) masked by
// hlow > 0: the gradient through upsampling into the ReLU that fed it.
__global__ void __launch_bounds__(kThreads) k_up_bwd(View g, int C, int nb, int h, int w,
                                                    const bf16_t* hlow, bf16_t* out) {
    const int W = 2 * w, c8 = C / 8;
    const long long n = (long long)nb * h * w * c8;
    const long long i = (long long)blockIdx.x * kThreads + threadIdx.x;
    if (i >= n) return;
    const int c = (int)(i % c8) * 8;
    const long long p = i / c8;
    const int x = (int)(p % w), y = (int)((p / w) % h), b = (int)(p / ((long long)w * h));
    float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int dy = 0; dy < 2; ++dy)
        for (int dx = 0; dx < 2; ++dx) {
            const long long q = (long long)(b * 2 * h + 2 * y + dy) * W + 2 * x + dx;
            float f[8];
            unpack8(*reinterpret_cast<const uint4*>(g.ptr + q * g.ld + c), f);
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e] += f[e];
        }
    float m[8];
    unpack8(*reinterpret_cast<const uint4*>(hlow + p * C + c), m);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = m[e] > 0.f ? acc[e] : 0.f;
    *reinterpret_cast<uint4*>(out + p * C + c) = pack8(acc);
}

// out (H x W x C) = (gpool at the pooled pixel / 4 + gcat) masked by cat > 0:
// the two gradient paths into an encoder level's output, through its ReLU.
__global__ void __launch_bounds__(kThreads) k_merge(const bf16_t* gpool, View gcat, View cat, int C,
                                                   int nb, int H, int W, bf16_t* out) {
    const int c8 = C / 8;
    const long long n = (long long)nb * H * W * c8;
    const long long i = (long long)blockIdx.x * kThreads + threadIdx.x;
    if (i >= n) return;
    const int c = (int)(i % c8) * 8;
    const long long p = i / c8;
    const int x = (int)(p % W), y = (int)((p / W) % H), b = (int)(p / ((long long)W * H));
    const long long q = (long long)(b * (H / 2) + y / 2) * (W / 2) + x / 2;
    float a[8], g[8], m[8];
    unpack8(*reinterpret_cast<const uint4*>(gpool + q * C + c), a);
    unpack8(*reinterpret_cast<const uint4*>(gcat.ptr + p * gcat.ld + c), g);
    unpack8(*reinterpret_cast<const uint4*>(cat.ptr + p * cat.ld + c), m);
#pragma unroll
    for (int e = 0; e < 8; ++e) a[e] = m[e] > 0.f ? 0.25f * a[e] + g[e] : 0.f;
    *reinterpret_cast<uint4*>(out + p * C + c) = pack8(a);
}

__device__ inline double block_sum_d(double v) {
    __shared__ double red[kThreads / 64];
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) red[w] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0)
        for (int q = 0; q < kThreads / 64; ++q) s += red[q];
    return s;
}

constexpr int kLossPer = 16;    // elements per thread of the loss kernel

// dy = d loss / d y (BF16, padded channels 0) and the loss per block (FP64).  A
// thread's loads are clamped, not skipped, so that eight elements' are in flight;
// waited for one element at a time, with 64-bit divisions, 32 targets of 64 x 64 x
// 189 took 60 us, now 40.
template <typename I>
__global__ void __launch_bounds__(kThreads) k_loss(const float* y, const float* t, const float* cw,
                                                  int out_ch, int out_p, long long npix,
                                                  bf16_t* dy, double* part) {
    constexpr int U = 8;
    const I n = (I)(npix * out_p), base = (I)blockIdx.x * kThreads * kLossPer + threadIdx.x;
    const double inv = 1.0 / (double)npix;
    double s = 0.0;
    for (int h = 0; h < kLossPer / U; ++h) {
        float yv[U], tv[U], w[U];
        bool in[U];                            // a channel of the target, not padding
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const I i = base + (I)(h * U + u) * kThreads;
            const I p = i / (I)out_p;
            const int c = (int)(i - p * (I)out_p);
            in[u] = i < n && c < out_ch;
            const long long o = in[u] ? (long long)p * out_ch + c : 0;
            yv[u] = y[o];
            tv[u] = t[o];
            w[u] = cw[in[u] ? c : 0];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const I i = base + (I)(h * U + u) * kThreads;
            if (i >= n) break;
            float g = 0.f;
            if (in[u]) {
                const float d = yv[u] - tv[u];
                s += (double)w[u] * (double)d * (double)d * inv;
                g = (float)(2.0 * w[u] * inv) * d;
            }
            dy[i] = f2bf(g);
        }
    }
    s = block_sum_d(s);
    if (threadIdx.x == 0) part[blockIdx.x] = s;
}

__global__ void __launch_bounds__(kThreads) k_sum(const double* part, int n, double* out) {
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += kThreads) s += part[i];
    s = block_sum_d(s);
    if (threadIdx.x == 0) *out = s;
}

__global__ void __launch_bounds__(kThreads) k_adam(float* p, float* m, float* v, const float* g,
                                                  long long n, float lr, float b1, float b2,
                                                  float eps, float c1, float c2) {
    const long long i = (long long)blockIdx.x * kThreads + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// BF16 copies of one layer's weights w[tap][ci][co] in the fragment order of
// k_conv: fragment (output group of 32, step of 16 K entries) is 64 lanes x 8
// entries, lane l holding K entries 8 (l / 32) + 0..7 of output l mod 32; zeros
// past the outputs and past K.  wf for the forward GEMM (outputs co, K = (tap,
// ci)), wb for the input gradient (outputs ci, K = (flipped tap, co)).
__global__ void __launch_bounds__(kThreads) k_export(const float* w, int taps, int cin, int cout,
                                                    bf16_t* wf, bf16_t* wb) {
    const long long nff = frag_elems(cout, taps * cin), nfb = frag_elems(cin, taps * cout);
    long long i = (long long)blockIdx.x * kThreads + threadIdx.x;
    const bool back = i >= nff;
    if (back) i -= nff;
    if (back && i >= nfb) return;
    const int N = back ? cin : cout, kc = back ? cout : cin, K = taps * kc;
    const int nsteps = (K + 15) / 16;
    const int e = (int)(i & 7), l = (int)(i >> 3) & 63;
    const int fs = (int)(i >> 9), f = fs / nsteps, s = fs - f * nsteps;
    const int n = 32 * f + (l & 31), k = 16 * s + 8 * (l >> 5) + e;
    bf16_t h = 0;
    if (n < N && k < K) {
        const int tap = k / kc, c = k - tap * kc;
        const int ci = back ? n : c, co = back ? c : n, t = back ? taps - 1 - tap : tap;
        h = f2bf(w[((long long)t * cin + ci) * cout + co]);
    }
    (back ? wb : wf)[i] = h;
}

// Layers between the flat exchange layout (cin_o, cout_o) and the padded device
// layout (cin_p, cout_p), blockIdx.y the layer; padded entries read as 0.  (A
// launch per layer: 20 of 3 us for the network of the 64 x 64 problems.)
__global__ void __launch_bounds__(kThreads) k_param_map(ParamMaps q, int to_padded) {
    const ParamMap& l = q.l[blockIdx.y];
    const unsigned cin_p = l.cin_p, cout_p = l.cout_p;
    const long long nw = (long long)l.taps * cin_p * cout_p, np = nw + cout_p;
    for (long long i = (long long)blockIdx.x * kThreads + threadIdx.x; i < np;
         i += (long long)gridDim.x * kThreads) {
        long long o = -1;
        if (i < nw) {
            const bool small = nw < (1LL << 32);          // 32-bit divisions
            const long long row = small ? (long long)((unsigned)i / cout_p) : i / cout_p;
            const int co = (int)(i - row * cout_p);
            const int tap = (int)(small ? (unsigned)row / cin_p : row / cin_p);
            const int ci = (int)(row - (long long)tap * cin_p);
            if (co < l.cout_o && ci < l.cin_o) o = ((long long)tap * l.cin_o + ci) * l.cout_o + co;
        } else {
            const int co = (int)(i - nw);
            if (co < l.cout_o) o = (long long)l.taps * l.cin_o * l.cout_o + co;
        }
        if (to_padded)
            l.dst[i] = o >= 0 ? l.src[o] : 0.f;
        else if (o >= 0)
            l.dst[o] = l.src[i];
    }
}

// ---- solver glue ----------------------------------------------------------

// x[b][y][x] = (f0 channels, f1 channels, then base channels if base is given):
// four consecutive output floats per thread (one 16-byte store; a group may
// run over a pixel's end).  A thread per pixel, each lane writing its own row,
// moved a 64-byte sector per 4-byte store: 262144 pixels of 195 channels took
// 1590 us; consecutive outputs take 122 us.
template <typename I>
__global__ void __launch_bounds__(kThreads) k_warm_inputs(WarmGeom g, int nb,
                                                         const float* __restrict__ f0,
                                                         const float* __restrict__ f1,
                                                         const float* __restrict__ base,
                                                         float* __restrict__ x) {
    const I plane = (I)g.X * g.Y;
    const int nch = g.C * (g.P - 1) + 3 * g.C * g.P;
    const int in_ch = 2 * g.C + (base ? nch : 0);
    const I n = (I)nb * plane * in_ch;
    const I e0 = 4 * ((I)blockIdx.x * kThreads + threadIdx.x);
    if (e0 >= n) return;
    I i = e0 / in_ch;                                  // pixel (over the batch)
    int ch = (int)(e0 - i * in_ch);
    float v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (ch >= 2 * g.C) {
            v[q] = i < (I)nb * plane ? base[(long long)i * nch + ch - 2 * g.C] : 0.f;
        } else if (i < (I)nb * plane) {
            const I b = i / plane, p = i - b * plane;
            const float* f = ch < g.C ? f0 : f1;
            v[q] = f[((long long)b * g.C + (ch < g.C ? ch : ch - g.C)) * plane + p];
        } else {
            v[q] = 0.f;
        }
        if (++ch == in_ch) { ch = 0; ++i; }
    }
    if (e0 + 4 <= n && ((uintptr_t)x & 15) == 0) {
        *reinterpret_cast<float4*>(x + e0) = make_float4(v[0], v[1], v[2], v[3]);
    } else {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (e0 + q < n) x[e0 + q] = v[q];
    }
}

// Between the planar solver state and the channels-last network layout: mode 0
// writes the target (state minus base) from the state, mode 1 the state from a
// network output (plus base).  A block maps 64 consecutive pixels (a lane
// each on the planar side) x 64 channels (a lane each on the channels-last
// side) through LDS, so both sides move 256-byte runs.  With a thread per
// pixel walking its channels, each lane of the channels-last side was on a
// line of its own: 64 problems of 64 x 64 x 3 x 16 took 820 us (mode 0, no
// base) and 1440 us (mode 1 with base); now 96 and 165 us (4.1 and 3.6 TB/s of 4-byte lanes).
constexpr int kMapPix = 64, kMapCh = 64, kMapPitch = kMapCh + 1;

// One channel of the network layout in the planar state: q < 0 a density
// slice with its interpolation weight s, else the momentum component q; off
// the offset k slice + c plane of its time step and colour.
struct MapChan {
    long long off;
    int q, c;
    float s;
};

template <int MODE>
__global__ void __launch_bounds__(kThreads) k_warm_map(WarmGeom g, int nb,
                                                      const float* __restrict__ f0,
                                                      const float* __restrict__ f1, const float* Fr, float* Fw,
                                                      long long sF, const float* Mxr,
                                                      const float* Myr, const float* Mcr,
                                                      float* Mxw, float* Myw, float* Mcw,
                                                      long long sM, const float* yr,
                                                      const float* base, float* tw) {
    __shared__ float tb[kMapPix * kMapPitch];                        // base, then (mode 0) the target
    __shared__ float ty[MODE == 1 ? kMapPix * kMapPitch : 1];        // network output
    // the tile's channels, decoded once: their divisions in every wave and
    // channel were half of the instructions
    __shared__ MapChan chan[kMapCh];
    const long long plane = (long long)g.X * g.Y;
    const long long slice = plane * g.C, npix = nb * plane;
    const int P = g.P, C = g.C;
    const int o0 = C * (P - 1), nch = o0 + 3 * C * P;
    const int cl = threadIdx.x % kMapCh, pl = threadIdx.x % kMapPix;      // channel, pixel of a thread
    const int cr = threadIdx.x / kMapCh, pr = __builtin_amdgcn_readfirstlane(threadIdx.x / kMapPix);
    constexpr int CR = kThreads / kMapCh, PR = kThreads / kMapPix;        // pixels, channels per round
    const long long i0 = (long long)blockIdx.x * kMapPix;
    const int np = (int)min((long long)kMapPix, npix - i0);
    // the channel tiles in turn (their runs of a pixel's row share cache lines;
    // as blocks of their own, on other XCDs, they fetched those lines twice)
    for (int ch0 = 0; ch0 < nch; ch0 += kMapCh) {
        const int nc = min(kMapCh, nch - ch0);
        if (ch0) __syncthreads();
        if ((int)threadIdx.x < nc) {
            const int ch = ch0 + threadIdx.x;
            MapChan h;
            int k;
            if (ch < o0) {
                k = 1 + ch / C;
                h.q = -1;
                h.c = ch % C;
            } else {
                const int kc = (ch - o0) % (P * C);
                k = kc / C;
                h.q = (ch - o0) / (P * C);
                h.c = kc % C;
            }
            h.s = (float)k / (float)P;
            h.off = k * slice + (long long)h.c * plane;
            chan[threadIdx.x] = h;
        }
        // channels-last side: a lane per channel; every load in flight (outside
        // the tile: its first entry) before the first LDS store
        {
            constexpr int R = kMapPix / CR;
            float vb[R], vy[R];
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const int q = cr + j * CR;
                const long long e = i0 * nch + (q < np && cl < nc ? q * nch + ch0 + cl : 0);
                vb[j] = base ? base[e] : 0.f;
                vy[j] = MODE == 1 ? yr[e] : 0.f;
            }
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const int l = (cr + j * CR) * kMapPitch + cl;
                tb[l] = vb[j];
                if (MODE == 1) ty[l] = vy[j];
            }
        }
        __syncthreads();
        // planar side: a lane per pixel
        const long long i = i0 + pl;
        if (pl < np) {
            const long long b = i / plane, p = i - b * plane;
            const int x = (int)(p % g.X), y = (int)(p / g.X);
            const bool wx = !g.perx && x == 0, wy = !g.pery && y == 0;
            const long long bF = b * sF + p, bM = b * sM + p, bf = b * slice + p;
            constexpr int R = kMapCh / PR, Q = 8;
            const bool dens = ch0 < o0;                      // the tile has density channels
#pragma unroll 1
            for (int j0 = 0; j0 < R; j0 += Q) {
                // the state (mode 0) and the end densities of Q channels in flight
                // (past the tile: its first channel)
                float v[Q], a0[Q], a1[Q];
#pragma unroll
                for (int j = 0; j < Q; ++j) {
                    const int cc = pr + (j0 + j) * PR;
                    const MapChan h = chan[cc < nc ? cc : 0];
                    if (MODE == 0)
                        v[j] = h.q < 0 ? Fr[bF + h.off] : (h.q == 0 ? Mxr : h.q == 1 ? Myr : Mcr)[bM + h.off];
                    a0[j] = dens ? f0[bf + h.c * plane] : 0.f;
                    a1[j] = dens ? f1[bf + h.c * plane] : 0.f;
                }
#pragma unroll
                for (int j = 0; j < Q; ++j) {
                    const int cc = pr + (j0 + j) * PR, l = pl * kMapPitch + cc;
                    if (cc >= nc) break;
                    const MapChan h = chan[cc];
                    const float bs = tb[l];
                    if (h.q < 0) {
                        // (1 - s) f0 + s f1, the second product rounded
                        const float lin = fmaf(1.f - h.s, a0[j], h.s * a1[j]);
                        if (MODE == 0)
                            tb[l] = v[j] - lin - bs;
                        else
                            Fw[bF + h.off] = lin + ty[l] + bs;
                    } else {
                        const bool wall = (h.q == 0 && wx) || (h.q == 1 && wy) ||
                                          (h.q == 2 && !g.perc && h.c == 0);
                        if (MODE == 0)
                            tb[l] = wall ? 0.f : v[j] - bs;
                        else
                            (h.q == 0 ? Mxw : h.q == 1 ? Myw : Mcw)[bM + h.off] = wall ? 0.f : ty[l] + bs;
                    }
                }
            }
        }
        if (MODE == 0) {
            __syncthreads();
            if (cl < nc)
#pragma unroll 4
                for (int q = cr; q < np; q += CR)
                    tw[(i0 + q) * nch + ch0 + cl] = tb[q * kMapPitch + cl];
        }
    }
}

// fc = 2 x 2 block means of f (coarse X, Y of gc; the fine grid is twice as
// wide and high).
__global__ void __launch_bounds__(kThreads) k_restrict(WarmGeom gc, int nb, const float* f,
                                                      float* fc) {
    const long long pc = (long long)gc.X * gc.Y;
    const long long n = nb * gc.C * pc;
    const long long i = (long long)blockIdx.x * kThreads + threadIdx.x;
    if (i >= n) return;
    const long long bc = i / pc, p = i - bc * pc;
    const int x = (int)(p % gc.X), y = (int)(p / gc.X);
    const int X = 2 * gc.X;
    const float* s = f + bc * 4 * pc + (long long)(2 * y) * X + 2 * x;
    fc[i] = 0.25f * (s[0] + s[1] + s[X] + s[X + 1]);
}

// Linear interpolation weight and the two neighbours of position u on an
// axis of n samples at integer positions (clamped at the ends, or wrapped).
struct Lerp {
    int a, b;
    float w;
};
__device__ inline Lerp lerp_at(float u, int n, int periodic) {
    int i0 = (int)floorf(u);
    Lerp r;
    r.w = u - (float)i0;
    if (periodic) {
        r.a = ((i0 % n) + n) % n;
        r.b = (r.a + 1) % n;
    } else {
        r.a = min(max(i0, 0), n - 1);
        r.b = min(max(i0 + 1, 0), n - 1);
    }
    return r;
}

// Prolong a coarse state (X/2, Y/2, same C, P_c steps) to the fine grid:
// bilinear in space for cell-centred values, linear between faces for the
// staggered momenta (walls read as 0), linear in time.  Writes the unknown
// slices of F and every slot of Mx, My, Mc.  A block per 256 pixels and time
// step (blockIdx.y): a thread walking every step of its pixel left the chip
// waiting on its chain of loads (170 us for 64 problems of 64 x 64 x 3 x 16;
// now 155 us).
__global__ void __launch_bounds__(kThreads) k_prolong(WarmGeom gc, WarmGeom gf, int nb,
                                                     const float* Fc, long long sFc,
                                                     const float* Mxc, const float* Myc,
                                                     const float* Mcc, long long sMc, float* F,
                                                     long long sF, float* Mx, float* My,
                                                     float* Mc, long long sM) {
    const long long plane = (long long)gf.X * gf.Y;
    const long long i = (long long)blockIdx.x * kThreads + threadIdx.x;
    if (i >= nb * plane) return;
    const long long b = i / plane, p = i - b * plane;
    const int x = (int)(p % gf.X), y = (int)(p / gf.X);
    const long long pc = (long long)gc.X * gc.Y, slc = pc * gc.C, slf = plane * gf.C;
    const float rt = (float)gc.P / (float)gf.P;
    // cell-centred positions of this fine cell on the coarse grid
    const Lerp cx = lerp_at(0.5f * x - 0.25f, gc.X, gf.perx);
    const Lerp cy = lerp_at(0.5f * y - 0.25f, gc.Y, gf.pery);
    auto centred = [&](const float* A, long long off) -> float {
        const float* r0 = A + off + (long long)cy.a * gc.X;
        const float* r1 = A + off + (long long)cy.b * gc.X;
        const float v0 = (1.f - cx.w) * r0[cx.a] + cx.w * r0[cx.b];
        const float v1 = (1.f - cx.w) * r1[cx.a] + cx.w * r1[cx.b];
        return (1.f - cy.w) * v0 + cy.w * v1;
    };
    // coarse face value along an axis: slot j of n faces, walls at 0 and n
    auto face = [&](const float* row, int j, int n, int stride, int periodic) -> float {
        if (periodic) return row[(long long)(((j % n) + n) % n) * stride];
        return (j <= 0 || j >= n) ? 0.f : row[(long long)j * stride];
    };
    for (int k = blockIdx.y; k < gf.P; k += gridDim.y) {
        if (k > 0) {
            float s = k * rt;
            int j0 = min((int)floorf(s), gc.P - 1);
            const float a = s - (float)j0;
            for (int c = 0; c < gf.C; ++c) {
                const long long o0 = b * sFc + j0 * slc + (long long)c * pc;
                const float v = (1.f - a) * centred(Fc, o0) + a * centred(Fc, o0 + slc);
                F[b * sF + k * slf + (long long)c * plane + p] = v;
            }
        }
        {
            const Lerp ct = lerp_at((k + 0.5f) * rt - 0.5f, gc.P, 0);
            for (int c = 0; c < gf.C; ++c) {
                const long long mi = b * sM + k * slf + (long long)c * plane + p;
                float vt[3] = {0.f, 0.f, 0.f};
                for (int h = 0; h < 2; ++h) {
                    const int kc = h ? ct.b : ct.a;
                    const float wt = h ? ct.w : 1.f - ct.w;
                    const long long oc = b * sMc + kc * slc + (long long)c * pc;
                    // x faces: fine slot x sits at coarse face position x / 2
                    {
                        const int j0 = x >> 1;
                        const float w = (x & 1) ? 0.5f : 0.f;
                        const float* r0 = Mxc + oc + (long long)cy.a * gc.X;
                        const float* r1 = Mxc + oc + (long long)cy.b * gc.X;
                        const float v0 = (1.f - w) * face(r0, j0, gc.X, 1, gf.perx) + w * face(r0, j0 + 1, gc.X, 1, gf.perx);
                        const float v1 = (1.f - w) * face(r1, j0, gc.X, 1, gf.perx) + w * face(r1, j0 + 1, gc.X, 1, gf.perx);
                        vt[0] += wt * ((1.f - cy.w) * v0 + cy.w * v1);
                    }
                    {
                        const int j0 = y >> 1;
                        const float w = (y & 1) ? 0.5f : 0.f;
                        const float* c0 = Myc + oc + cx.a;
                        const float* c1 = Myc + oc + cx.b;
                        const float v0 = (1.f - w) * face(c0, j0, gc.Y, gc.X, gf.pery) + w * face(c0, j0 + 1, gc.Y, gc.X, gf.pery);
                        const float v1 = (1.f - w) * face(c1, j0, gc.Y, gc.X, gf.pery) + w * face(c1, j0 + 1, gc.Y, gc.X, gf.pery);
                        vt[1] += wt * ((1.f - cx.w) * v0 + cx.w * v1);
                    }
                    vt[2] += wt * centred(Mcc, oc);
                }
                const bool wx = !gf.perx && x == 0, wy = !gf.pery && y == 0, wc = !gf.perc && c == 0;
                Mx[mi] = wx ? 0.f : vt[0];
                My[mi] = wy ? 0.f : vt[1];
                Mc[mi] = wc ? 0.f : vt[2];
            }
        }
    }
}

dim3 map_grid(const WarmGeom& g, int nb) {
    return dim3((unsigned)(((long long)nb * g.X * g.Y + kMapPix - 1) / kMapPix));
}

inline unsigned blocks(long long n) { return (unsigned)((n + kThreads - 1) / kThreads); }

}  // namespace

void launch_conv(const ConvArgs& a, int epi, hipStream_t st) {
    switch (epi) {
        case EPI_RELU: conv_dispatch<EPI_RELU>(a, st); break;
        case EPI_F32: conv_dispatch<EPI_F32>(a, st); break;
        case EPI_PLAIN: conv_dispatch<EPI_PLAIN>(a, st); break;
        default: conv_dispatch<EPI_MASK>(a, st); break;
    }
}

// Most splits of a layer's pixels: a block per compute unit where a wave's
// fragments fill its registers, else two.
int wgrad_splits(int taps, int cin, int cout, int nb, int H, int W) {
    int rows, cols;
    size_t lds;
    const WgradGeom g = wgrad_geom(taps, cin, cout, nb, H, W, &rows, &cols, &lds);
    const WgradTile w = wgrad_tile(taps, cin, cout);
    const int most = std::max(1, (w.mw * w.nw > 8 ? 256 : 512) / (rows * cols));
    return std::min(most, g.tiles);
}

// The tiles go to the splits in equal shares, and only splits that have tiles are
// launched and summed (360 tiles over 256 splits are 180 of two; the other 76 wrote
// zeros that were read and summed: gradient of 9 images of 64 x 64 802 us, now 781).
int launch_wgrad(const ConvArgs& a, hipStream_t st) {
    int rows, cols;
    size_t lds;
    WgradGeom g = wgrad_geom(a.taps, a.cin, a.N, a.nb, a.H, a.W, &rows, &cols, &lds);
    const int most_splits = wgrad_splits(a.taps, a.cin, a.N, a.nb, a.H, a.W);
    g.per_split = (g.tiles + most_splits - 1) / most_splits;
    const int splits = (g.tiles + g.per_split - 1) / g.per_split;
    const WgradTile w = wgrad_tile(a.taps, a.cin, a.N);
    const dim3 grid(splits, rows, cols), block(kThreads);
    // units of the largest tile per thread: the variant that keeps them all in
    // flight with the fewest idle loads
    int most = 0;
    for (int gy = 0; gy < rows; ++gy) {
        int cb0;
        most = std::max(most, g.ti * g.bh * g.bw * wgrad_units(g, a.taps, a.cin, gy, &cb0));
    }
    most += 64 * std::min(a.N / 8, 4 * (w.nwave ? 4 * w.nw : w.nw));
#define OTN_WG(MW, NW, NWAVE, Q)                                                                  \
    if (w.mw == MW && w.nw == NW && (most <= Q * kThreads || Q == 12)) {                          \
        hipLaunchKernelGGL((k_wgrad<MW, NW, NWAVE, Q>), grid, block, lds, st, a, g);              \
        return splits;                                                                            \
    }
    OTN_WG(1, 2, true, 8) OTN_WG(1, 2, true, 12)
    OTN_WG(3, 1, false, 4) OTN_WG(3, 1, false, 12)
    OTN_WG(7, 1, false, 8) OTN_WG(7, 1, false, 12)
    OTN_WG(16, 1, false, 12)
    OTN_WG(3, 2, false, 4) OTN_WG(3, 2, false, 12)
    OTN_WG(5, 2, false, 8) OTN_WG(5, 2, false, 12)
    OTN_WG(7, 2, false, 8) OTN_WG(7, 2, false, 12)
    OTN_WG(3, 4, false, 8) OTN_WG(3, 4, false, 12)
#undef OTN_WG
    return splits;
}

void launch_wgrad_reduce(const float* part, int splits, int M, int N, float* out, hipStream_t st) {
    const long long mn = (long long)M * N;
    hipLaunchKernelGGL(k_wgrad_reduce, dim3((unsigned)((mn + 63) / 64)), dim3(kThreads), 0, st, part, splits, mn, out);
}

void launch_pack_input(const float* x, int in_ch, long long npix, bf16_t* out, int ld,
                       hipStream_t st) {
    // 32-bit indices (one cheap division) where every one fits
    const long long n = npix * (ld / 8);
    if (n < (1LL << 31))
        hipLaunchKernelGGL(k_pack_input<unsigned>, dim3(blocks(n)), dim3(kThreads), 0, st, x, in_ch,
                           npix, out, ld);
    else
        hipLaunchKernelGGL(k_pack_input<long long>, dim3(blocks(n)), dim3(kThreads), 0, st, x, in_ch,
                           npix, out, ld);
}

void launch_pool(View src, int C, int nb, int H, int W, bf16_t* dst, hipStream_t st) {
    const long long n = (long long)nb * (H / 2) * (W / 2) * (C / 8);
    hipLaunchKernelGGL(k_pool, dim3(blocks(n)), dim3(kThreads), 0, st, src, C, nb, H, W, dst);
}

void launch_upsample(const bf16_t* src, int C, int nb, int h, int w, View dst, hipStream_t st) {
    const long long n = (long long)nb * 4 * h * w * (C / 8);
    hipLaunchKernelGGL(k_upsample, dim3(blocks(n)), dim3(kThreads), 0, st, src, C, nb, h, w, dst);
}

void launch_up_bwd(View g, int C, int nb, int h, int w, const bf16_t* hlow, bf16_t* out,
                   hipStream_t st) {
    const long long n = (long long)nb * h * w * (C / 8);
    hipLaunchKernelGGL(k_up_bwd, dim3(blocks(n)), dim3(kThreads), 0, st, g, C, nb, h, w, hlow, out);
}

void launch_merge(const bf16_t* gpool, View gcat, View cat, int C, int nb, int H, int W,
                  bf16_t* out, hipStream_t st) {
    const long long n = (long long)nb * H * W * (C / 8);
    hipLaunchKernelGGL(k_merge, dim3(blocks(n)), dim3(kThreads), 0, st, gpool, gcat, cat, C, nb, H,
                       W, out);
}

int loss_blocks(long long n) { return (int)((n + kThreads * kLossPer - 1) / (kThreads * kLossPer)); }

void launch_loss(const float* y, const float* t, const float* cw, int out_ch, int out_p,
                 long long npix, bf16_t* dy, double* part, hipStream_t st) {
    const long long n = npix * out_p;
    if (n < (1LL << 31) - kThreads * kLossPer)
        hipLaunchKernelGGL(k_loss<unsigned>, dim3(loss_blocks(n)), dim3(kThreads), 0, st, y, t, cw, out_ch,
                           out_p, npix, dy, part);
    else
        hipLaunchKernelGGL(k_loss<long long>, dim3(loss_blocks(n)), dim3(kThreads), 0, st, y, t, cw,
                           out_ch, out_p, npix, dy, part);
}

void launch_sum(const double* part, int n, double* out, hipStream_t st) {
    hipLaunchKernelGGL(k_sum, dim3(1), dim3(kThreads), 0, st, part, n, out);
}

void launch_adam(float* p, float* m, float* v, const float* g, long long n, float lr, float b1,
                 float b2, float eps, float c1, float c2, hipStream_t st) {
    hipLaunchKernelGGL(k_adam, dim3(blocks(n)), dim3(kThreads), 0, st, p, m, v, g, n, lr, b1, b2,
                       eps, c1, c2);
}

void launch_export(const float* w, int taps, int cin, int cout, bf16_t* wf, bf16_t* wb,
                   hipStream_t st) {
    const long long n = frag_elems(cout, taps * cin) + frag_elems(cin, taps * cout);
    hipLaunchKernelGGL(k_export, dim3(blocks(n)), dim3(kThreads), 0, st, w, taps, cin, cout, wf, wb);
}

void launch_param_maps(const ParamMaps& q, int to_padded, hipStream_t st) {
    hipLaunchKernelGGL(k_param_map, dim3(256, q.n), dim3(kThreads), 0, st, q, to_padded);
}

void launch_warm_inputs(const WarmGeom& g, int nb, const float* f0, const float* f1,
                        const float* base, float* x, hipStream_t st) {
    const int in_ch = 2 * g.C + (base ? g.C * (g.P - 1) + 3 * g.C * g.P : 0);
    const long long n = (long long)nb * g.X * g.Y * in_ch;
    const dim3 grid(blocks((n + 3) / 4));
    if (n < (1LL << 31) - 4 * kThreads)
        hipLaunchKernelGGL(k_warm_inputs<unsigned>, grid, dim3(kThreads), 0, st, g, nb, f0, f1, base, x);
    else
        hipLaunchKernelGGL(k_warm_inputs<long long>, grid, dim3(kThreads), 0, st, g, nb, f0, f1, base, x);
}

void launch_warm_targets(const WarmGeom& g, int nb, const float* f0, const float* f1,
                         const float* F, long long sF, const float* Mx, const float* My,
                         const float* Mc, long long sM, const float* base, float* t,
                         hipStream_t st) {
    hipLaunchKernelGGL(k_warm_map<0>, map_grid(g, nb), dim3(kThreads), 0, st, g, nb, f0, f1, F,
                       (float*)nullptr, sF, Mx, My, Mc, (float*)nullptr, (float*)nullptr,
                       (float*)nullptr, sM, (const float*)nullptr, base, t);
}

void launch_warm_state(const WarmGeom& g, int nb, const float* f0, const float* f1,
                       const float* y, const float* base, float* F, long long sF, float* Mx,
                       float* My, float* Mc, long long sM, hipStream_t st) {
    hipLaunchKernelGGL(k_warm_map<1>, map_grid(g, nb), dim3(kThreads), 0, st, g, nb, f0, f1,
                       (const float*)nullptr, F, sF, (const float*)nullptr, (const float*)nullptr,
                       (const float*)nullptr, Mx, My, Mc, sM, y, base, (float*)nullptr);
}

void launch_restrict(const WarmGeom& gc, int nb, const float* f, float* fc, hipStream_t st) {
    const long long n = (long long)nb * gc.C * gc.X * gc.Y;
    hipLaunchKernelGGL(k_restrict, dim3(blocks(n)), dim3(kThreads), 0, st, gc, nb, f, fc);
}

void launch_prolong(const WarmGeom& gc, const WarmGeom& gf, int nb, const float* Fc,
                    long long sFc, const float* Mxc, const float* Myc, const float* Mcc,
                    long long sMc, float* F, long long sF, float* Mx, float* My, float* Mc,
                    long long sM, hipStream_t st) {
    const long long n = (long long)nb * gf.X * gf.Y;
    hipLaunchKernelGGL(k_prolong, dim3(blocks(n), (unsigned)std::min(gf.P, 65535)), dim3(kThreads), 0, st, gc, gf, nb, Fc, sFc, Mxc,
                       Myc, Mcc, sMc, F, sF, Mx, My, Mc, sM);
}

}  // namespace otn
