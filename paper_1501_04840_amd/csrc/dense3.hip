// Three-pass Poisson solve with dense transforms, for x and y of any length up to
// 512: the counterpart of the fused passes of transform.hip (power-of-two Neumann
// axes, P in {8, 16, 32}) for other shapes: image sides like 173 x 131, small
// problems, odd numbers of time steps.
//
//   k_dx (forward)  a block owns some times of every colour of one row y: rows of
//                   length X, transformed along x and written to the transposed
//                   scratch Rt[b][jx][c][y][t];
//   k_dyt           a block owns some lines (frequency jx, colour mode): Y P
//                   values of a line are one contiguous run; transform along y, along t, division by the eigenvalues of
//                   A A^T, the inverses, back in place;
//   k_dx (inverse)  the mirror of the first, with the inverse colour transform.
//
// r arrives in colour modes (StepArgs::cmix).  The transforms are products with
// the axis matrices on the matrix cores (MFMA 16x16x4 FP32).  The DCT-II matrix
// is even or odd about the axis's middle by the parity of its row, so a Neumann
// axis is folded (x[k] +- x[n - 1 - k]) and its even and odd frequencies are two
// products of half the length; a periodic axis is one product.  The matrices
// are stored in fragment order (one contiguous KB per 16 outputs and 16 inputs,
// zeros past the ends), loaded from L2 three groups ahead, and each fragment
// serves up to 64 rows.  Tiles stay in LDS between the steps of a pass.
//
// They replace five passes (rows, columns, colour and time, columns, rows) whose
// kernels waited for their staging loads one by one, read the matrices with no
// load ahead and did the products along t one scalar load per term: at 173 x 131
// x 3 x 12 an iteration took 128 us, 102 of them in the solve; now 77.  What bounds
// a pass at such sizes: launch and the latency of one block's loads, then the
// products (unfolded they were 85 us).  A few problems of 16 x 16 x 3 x 8: 45 us
// per iteration, now 28.
//
// The spatial-DC line (jx, jy) = (0, 0) is solved in FP64 from the plane sums
// of r, which extra blocks of the first pass reduce, by the jx = 0 blocks of the
// second, as in the other paths.
#include <algorithm>

#include "otd_common.h"

#pragma clang fp contract(on)   // as in fft_common.h

namespace otd {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kDThreads = 1024;            // at most
constexpr int kDMaxL = 512;                // longest axis
constexpr int kDMaxP = 64;                 // most times
constexpr size_t kDLds = 152 * 1024;

struct DenseArgs {
    Geom g;
    float* R;
    float* Rt;
    AxisTab tx, ty, tc, tt;
    DenseAxis ax, ay;
    const double* tc64;
    const double* tt64;
    double* part;              // FP64 plane partials of r, plane stride nbx
    int nbx;
    const float* frz;          // per problem: nonzero = frozen, skipped (or null)
    int nsb;                   // plane-sum blocks of the forward x pass (a multiple of 8)
    int nrg, tb;               // x passes: time groups of a row y, times in each
    int lpb;                   // y and time pass: lines (jx, colour mode) per block
};

// e / d for e < 2^16 by a reciprocal (rcp_of).
__device__ __forceinline__ unsigned rcp_of(int d) { return 0xFFFFFFFFu / d + 1; }
__device__ __forceinline__ int div_by(int e, unsigned m, int d) { return d == 1 ? e : (int)__umulhi(e, m); }

// Position of a frequency (folded: even ones, then odd ones from H on), and
// whether a position holds one.
__device__ __forceinline__ int pos_of(const DenseAxis& x, int j) { return x.fold ? (j & 1) * x.H + (j >> 1) : j; }
__device__ __forceinline__ int freq_of(const DenseAxis& x, int p) {
    return x.fold ? (p < x.H ? 2 * p : 2 * (p - x.H) + 1) : p;
}

// A ring of groups of 16 inputs of NC tiles of 16 outputs, whose loads run
// kAhead groups ahead (the table is padded behind its last fragment).
constexpr int kAhead = 3, kRing = kAhead + 1;
static_assert(kRing % 2 == 0, "a ring keeps the data fragments' parity");
static_assert(kAhead <= kDenseAxisPad, "loads ahead stay inside the table");

template <int NC>
struct MatrixRing {
    f32x4 v[kRing][NC];
    const f32x4* p[NC];
    __device__ __forceinline__ void next(int slot) {
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            v[slot][i] = *p[i];
            p[i] += 64;
        }
    }
};

// The waves of a block over an axis's output tiles: wave w of W takes tiles
// tl = w / nb + i W / nb (i < MI) of block w mod nb (folded: nb = 2, even and odd
// outputs).  W is a multiple of nb.
template <int MI>
struct TileShare {
    int b, tl0, step, T;
    __device__ __forceinline__ explicit TileShare(const DenseAxis& x) {
        const int nb = x.fold ? 2 : 1, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        b = x.fold ? w & 1 : 0;
        tl0 = x.fold ? w >> 1 : w;
        step = (blockDim.x >> 6) / nb;
        T = x.H / 16;
    }
    __device__ __forceinline__ void start(MatrixRing<MI>& m, const float* table) const {
#pragma unroll
        for (int i = 0; i < MI; ++i)
            m.p[i] = reinterpret_cast<const f32x4*>(table) +
                     (long long)(b * T + min(tl0 + i * step, T - 1)) * T * 64 + (threadIdx.x & 63);
#pragma unroll
        for (int s = 0; s < kAhead; ++s) m.next(s);
    }
};

// tile[n][p] -> sum over the block's positions k of table[p][k] tile[n][k], 16
// RT rows n, in place.  Lane l of a wave takes k = 16 s + 4 (l / 16) + q of group
// s in product q, from both operands; the next group's data and the matrix
// entries kAhead groups on are requested before a group's products, and the
// scheduling barriers keep them there.
template <int RT, int MI>
__device__ __forceinline__ void product(float* tile, int pitch, const DenseAxis& ax, const TileShare<MI>& sh,
                                        MatrixRing<MI>& m) {
    const int lane = threadIdx.x & 63, row = lane & 15, g = lane >> 4, groups = sh.T;
    f32x4 acc[MI][RT];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int r = 0; r < RT; ++r) acc[i][r] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (sh.tl0 < sh.T) {
        const float* const x = tile + row * pitch + sh.b * ax.H + 4 * g;
        f32x4 a[2][RT];
        auto read = [&](int s, f32x4 (&v)[RT]) {           // past the last group: the last
            const float* p = x + 16 * min(s, groups - 1);
#pragma unroll
            for (int r = 0; r < RT; ++r) v[r] = *reinterpret_cast<const f32x4*>(p + 16 * r * pitch);
        };
        auto mma = [&](int u, const f32x4 (&v)[RT]) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int i = 0; i < MI; ++i)
#pragma unroll
                    for (int r = 0; r < RT; ++r)
                        acc[i][r] = __builtin_amdgcn_mfma_f32_16x16x4f32(m.v[u][i][q], v[r][q], acc[i][r], 0, 0, 0);
        };
        read(0, a[0]);
        int s = 0;
        for (; s + kRing <= groups; s += kRing) {
#pragma unroll
            for (int u = 0; u < kRing; ++u) {
                read(s + u + 1, a[(u + 1) & 1]);
                m.next((u + kAhead) % kRing);
                __builtin_amdgcn_sched_barrier(0);
                mma(u, a[u & 1]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int u = 0; u < kRing - 1; ++u) {
            if (s + u >= groups) break;                    // uniform
            read(s + u + 1, a[(u + 1) & 1]);
            mma(u, a[u & 1]);
        }
    }
    __syncthreads();                           // every wave has read the tile
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const int tl = sh.tl0 + i * sh.step;
        if (tl >= sh.T) continue;
#pragma unroll
        for (int r = 0; r < RT; ++r)
            *reinterpret_cast<f32x4*>(tile + (16 * r + row) * pitch + sh.b * ax.H + 16 * tl + 4 * g) = acc[i][r];
    }
    __syncthreads();
}

// One x pass of a row index y and a group of times (rows n = c tb + t - t0, 16 RT
// of them).  Blocks go to the XCDs round-robin: each XCD takes a contiguous
// eighth of the (row y, time group) items, times fastest, so that the pieces of
// the transposed scratch one L2 holds are longer runs.  (The plane-sum blocks
// ahead of them are a multiple of eight, the same shift for every XCD.)  With the
// time groups of a row on XCDs of their own 173 x 131 x 3 x 12 took 79.6 us an
// iteration, now 76.8; 128 x 128 x 3 x 12 55.3 and 53.0; from 400 x 400 on 1%.
template <int RT, int MI, bool INV>
__global__ void __launch_bounds__(kDThreads) k_dx(DenseArgs a) {
    extern __shared__ __attribute__((aligned(16))) float xs[];
    if (!INV && (int)blockIdx.x < a.nsb) {
        if (threadIdx.x < 256)
            plane_sums_block(PlaneSums{a.part, (long long)a.g.B * a.g.P * a.g.C, a.nbx}, blockIdx.x);
        return;
    }
    const Geom& g = a.g;
    const DenseAxis ax = a.ax;
    const int X = g.X, P = g.P, C = g.C, H = ax.H, width = ax.fold ? 2 * H : H, pitch = width + 4;
    const int h = ax.fold ? (X + 1) / 2 : X, nth = blockDim.x, W = nth >> 6;
    const int blk = blockIdx.x - (INV ? 0 : a.nsb), items = g.Y * g.B * a.nrg;
    const int xcd = blk & 7, item = xcd * (items >> 3) + min(xcd, items & 7) + (blk >> 3);
    const int yb = item / a.nrg, tg = item - yb * a.nrg, b = yb / g.Y, y = yb - b * g.Y;
    if (a.frz && a.frz[b] != 0.f) return;      // block-uniform
    const int t0 = tg * a.tb, nt = min(a.tb, P - t0), nr = C * nt;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    float* const Rb = a.R + (long long)b * g.nc + (long long)t0 * g.slice + (long long)y * X;
    float* const Tb = a.Rt + (long long)b * g.nc + (long long)y * P + t0;
    const int YP = g.Y * P;
    // the matrix entries are on their way while the rows are staged
    const TileShare<MI> sh(ax);
    MatrixRing<MI> ring;
    sh.start(ring, INV ? ax.inv : ax.fwd);
    const unsigned mnr = rcp_of(nr), mnt = rcp_of(nt);
    constexpr int U = 8;                       // pieces in flight per thread (folded: two loads each)
    if (!INV) {
        // the waves take (row, 64 columns) pieces in turn; rows without a time
        // and columns past the end are zeros
        const int cols = (H + 63) / 64, pieces = 16 * RT * cols;
        for (int q0 = wave; q0 < pieces; q0 += U * W) {
            float v[U], w[U];
#pragma unroll
            for (int j = 0; j < U; ++j) {
                const int q = q0 + j * W, r = q / cols, k = 64 * (q - r * cols) + lane;
                const int c = r / a.tb, t = r - c * a.tb;
                const bool in = q < pieces && c < C && t < nt && k < h;
                const long long o = in ? (long long)t * g.slice + (long long)c * g.plane : 0;
                v[j] = Rb[o + (in ? k : 0)];
                w[j] = ax.fold ? Rb[o + (in ? X - 1 - k : 0)] : 0.f;
                v[j] = in ? v[j] : 0.f;
                w[j] = in && 2 * k + 1 != X ? w[j] : 0.f;    // (the middle of an odd axis counts once)
            }
#pragma unroll
            for (int j = 0; j < U; ++j) {
                const int q = q0 + j * W, r = q / cols, k = 64 * (q - r * cols) + lane;
                if (q >= pieces || k >= H) continue;
                xs[r * pitch + k] = v[j] + w[j];
                if (ax.fold) xs[r * pitch + H + k] = 2 * k + 1 != X ? v[j] - w[j] : 0.f;
            }
        }
    } else {
        // the transposed scratch: consecutive lanes along t, then c, then jx
        const int tot = nr * X;
        for (int e0 = threadIdx.x; e0 < tot; e0 += 2 * U * nth) {
            float v[2 * U];
#pragma unroll
            for (int j = 0; j < 2 * U; ++j) {
                const int e = min(e0 + j * nth, tot - 1);
                const int jx = div_by(e, mnr, nr), nl = e - jx * nr, c = div_by(nl, mnt, nt), t = nl - c * nt;
                v[j] = Tb[(long long)(jx * C + c) * YP + t];
            }
#pragma unroll
            for (int j = 0; j < 2 * U; ++j) {
                const int e = min(e0 + j * nth, tot - 1);
                const int jx = div_by(e, mnr, nr), nl = e - jx * nr, c = div_by(nl, mnt, nt), t = nl - c * nt;
                xs[(c * a.tb + t) * pitch + pos_of(ax, jx)] = v[j];
            }
        }
        // zeros where there is no frequency or no time
        for (int r = wave; r < 16 * RT; r += W) {
            const bool row = r < C * a.tb && r % a.tb < nt;
            for (int p = lane; p < width; p += 64)
                if (!row || freq_of(ax, p) >= X) xs[r * pitch + p] = 0.f;
        }
        if (C > 1) {                           // inverse colour transform
            __syncthreads();
            const float* const Uc = a.tc.mat + C * C;    // Uc[jc C + c] = M_c[jc][c]
            for (int e = threadIdx.x; e < nt * width; e += nth) {
                const int t = e / width, p = e - t * width;
                float v[4];
#pragma unroll
                for (int jc = 0; jc < 4; ++jc) v[jc] = jc < C ? xs[(jc * a.tb + t) * pitch + p] : 0.f;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    if (c >= C) break;
                    float s = 0.f;
#pragma unroll
                    for (int jc = 0; jc < 4; ++jc)
                        if (jc < C) s = fmaf(Uc[jc * C + c], v[jc], s);
                    xs[(c * a.tb + t) * pitch + p] = s;
                }
            }
        }
    }
    __syncthreads();
    product<RT, MI>(xs, pitch, ax, sh, ring);
    if (!INV) {
        for (int e = threadIdx.x; e < nr * X; e += nth) {
            const int jx = div_by(e, mnr, nr), nl = e - jx * nr, c = div_by(nl, mnt, nt), t = nl - c * nt;
            Tb[(long long)(jx * C + c) * YP + t] = xs[(c * a.tb + t) * pitch + pos_of(ax, jx)];
        }
        return;
    }
    for (int r = wave; r < 16 * RT; r += W) {
        const int c = r / a.tb, t = r - c * a.tb;
        if (c >= C || t >= nt) continue;       // uniform
        float* const o = Rb + (long long)t * g.slice + (long long)c * g.plane;
        for (int k = lane; k < h; k += 64) {
            const float e = xs[r * pitch + k];
            if (!ax.fold) {
                o[k] = e;
            } else {
                const float d = xs[r * pitch + H + k];
                o[k] = e + d;
                if (2 * k + 1 != X) o[X - 1 - k] = e - d;
            }
        }
    }
}

// Time transform of columns p0 .. p0 + 15, in place: x[jt][p] = sum over t of
// T[t][jt] x[t][p] for rows x, with the division by the eigenvalues (DIVIDE).
// The wave owns these entries.  PT > 0: P <= 16 PT and the matrix is held in
// registers, else it is read from T.
template <int PT>
struct TimeMatrix {
    float v[PT > 0 ? PT : 1][PT > 0 ? 4 * PT : 1];
    __device__ __forceinline__ void load(const float* T, int P) {
        const int lane = threadIdx.x & 63, col = lane & 15, g = lane >> 4;
        if constexpr (PT > 0)
#pragma unroll
            for (int m = 0; m < PT; ++m)
#pragma unroll
                for (int s = 0; s < 4 * PT; ++s) {
                    const int k = 4 * s + g, jt = 16 * m + col;
                    const float w = T[min(k, P - 1) * P + min(jt, P - 1)];
                    v[m][s] = k < P && jt < P ? w : 0.f;
                }
    }
};

template <int PT, bool DIVIDE>
__device__ __forceinline__ void t_product(float* rows, int pitch, int P, const TimeMatrix<PT>& tm,
                                          const float* T, int p0, float lc, const float* lamt) {
    const int lane = threadIdx.x & 63, col = lane & 15, g = lane >> 4;
    float* const x = rows + p0 + col;
    constexpr int MT = PT > 0 ? PT : kDMaxP / 16;
    f32x4 acc[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) acc[m] = f32x4{0.f, 0.f, 0.f, 0.f};
    if constexpr (PT > 0) {
        float b[4 * PT];
#pragma unroll
        for (int s = 0; s < 4 * PT; ++s) {
            const int k = 4 * s + g;
            const float w = x[min(k, P - 1) * pitch];
            b[s] = k < P ? w : 0.f;
        }
#pragma unroll
        for (int s = 0; s < 4 * PT; ++s)
#pragma unroll
            for (int m = 0; m < PT; ++m)
                acc[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(tm.v[m][s], b[s], acc[m], 0, 0, 0);
    } else {
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            if (16 * m >= P) break;
            const int jt = 16 * m + col;
            for (int s0 = 0; 4 * s0 < P; s0 += 4) {
                float av[4], bv[4];
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const int k = 4 * (s0 + s) + g;
                    const bool in = k < P;
                    av[s] = in && jt < P ? T[k * P + jt] : 0.f;
                    bv[s] = in ? x[k * pitch] : 0.f;
                }
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    acc[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[s], bv[s], acc[m], 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        if (16 * m >= P) break;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int jt = 16 * m + 4 * g + q;
            if (jt >= P) continue;
            float v = acc[m][q];
            if (DIVIDE) {
                const float lam = lc + lamt[jt];
                v = lam > 0.f ? v / lam : 0.f;
            }
            x[jt * pitch] = v;
        }
    }
    // the wave's later reads see its writes
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int RT, int MI, int PT>
__global__ void __launch_bounds__(kDThreads) k_dyt(DenseArgs a) {
    extern __shared__ __attribute__((aligned(16))) float tile[];
    __shared__ double d1[4 * kDMaxP], d2[4 * kDMaxP];
    __shared__ float dcl[4 * kDMaxP], lamt[kDMaxP];
    const Geom& g = a.g;
    const DenseAxis ay = a.ay;
    const int Y = g.Y, P = g.P, C = g.C, H = ay.H, width = ay.fold ? 2 * H : H, pitch = width + 4;
    const int h = ay.fold ? (Y + 1) / 2 : Y, nth = blockDim.x, W = nth >> 6;
    const int b = blockIdx.y, q0 = blockIdx.x * a.lpb, nq = min(a.lpb, g.X * C - q0);   // lines q = jx C + c
    if (a.frz && a.frz[b] != 0.f) return;      // block-uniform
    const int NR = nq * P, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    float* const base = a.Rt + (long long)b * g.nc + (long long)q0 * Y * P;
    const int mt = width / 16, ndc = max(min(q0 + nq, C) - q0, 0) * P;   // (ndc: rows of spatial-DC lines)
    const TileShare<MI> sh(ay);
    MatrixRing<MI> ring;
    sh.start(ring, ay.fwd);
    TimeMatrix<PT> tf, ti;
    if (wave < nq * mt) {
        tf.load(a.tt.mat, P);
        ti.load(a.tt.mat + P * P, P);
    }
    // entries (c, y, t), t fastest, y < h (folded: with their mirror images)
    const int tot = NR * h;
    const unsigned mp = rcp_of(P), mh = rcp_of(h);
    constexpr int U = 4;
    for (int e0 = threadIdx.x; e0 < tot; e0 += U * nth) {
        float v[U], w[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int e = min(e0 + j * nth, tot - 1);
            const int q = div_by(e, mp, P), t = e - q * P, c = div_by(q, mh, h), y = q - c * h;
            const float* s = base + (long long)c * Y * P + t;
            v[j] = s[y * P];
            w[j] = ay.fold ? s[(Y - 1 - y) * P] : 0.f;
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int e = min(e0 + j * nth, tot - 1);
            const int q = div_by(e, mp, P), t = e - q * P, c = div_by(q, mh, h), y = q - c * h;
            float* const o = tile + (c * P + t) * pitch + y;
            const bool mid = 2 * y + 1 == Y;   // the middle of an odd axis counts once
            o[0] = ay.fold && !mid ? v[j] + w[j] : v[j];
            if (ay.fold) o[H] = mid ? 0.f : v[j] - w[j];
        }
    }
    for (int r = wave; r < 16 * RT; r += W)    // zeros past the axis and past the rows
        for (int p = lane; p < width; p += 64)
            if (r >= NR || (p >= h && p < H) || p >= H + h) tile[r * pitch + p] = 0.f;
    for (int e = threadIdx.x; e < P; e += nth) lamt[e] = a.tt.lam[e];
    if (ndc)
        for (int e = threadIdx.x; e < C * P; e += nth) d1[e] = a.part[((long long)b * C * P + e) * a.nbx];
    __syncthreads();
    if (ndc) {
        // FP64 (colour, time) problem of the spatial-DC line for this block's
        // modes: the plane sums to colour modes, then each time product over
        // eight lanes
        const int l = threadIdx.x & 7;
        const double* lt = a.tt64 + P * P;
        const double* lamc = a.tc64 + C * C;
        for (int e = threadIdx.x; e < ndc; e += nth) {
            const int jc = q0 + e / P, k = e % P;
            double s = 0.0;
            for (int c = 0; c < C; ++c) s += a.tc64[jc * C + c] * d1[k * C + c];
            d2[e] = s;
        }
        __syncthreads();
        for (int o = threadIdx.x >> 3; o < ndc; o += nth / 8) {
            const int r = o / P, jt = o - r * P;
            double s = 0.0;
            for (int k = l; k < P; k += 8) s += a.tt64[jt * P + k] * d2[r * P + k];
            s += __shfl_xor(s, 4, 8);
            s += __shfl_xor(s, 2, 8);
            s += __shfl_xor(s, 1, 8);
            const double lam = lamc[q0 + r] + lt[jt];
            if (l == 0) d1[o] = lam > 0.0 ? s / lam : 0.0;
        }
        __syncthreads();
        for (int o = threadIdx.x >> 3; o < ndc; o += nth / 8) {
            const int r = o / P, k = o - r * P;
            double s = 0.0;
            for (int jt = l; jt < P; jt += 8) s += a.tt64[jt * P + k] * d1[r * P + jt];
            s += __shfl_xor(s, 4, 8);
            s += __shfl_xor(s, 2, 8);
            s += __shfl_xor(s, 1, 8);
            if (l == 0) dcl[o] = (float)(s / sqrt((double)g.plane));
        }
    }
    product<RT, MI>(tile, pitch, ay, sh, ring);
    sh.start(ring, ay.inv);                    // for the way back
    {
        for (int task = wave; task < nq * mt; task += W) {
            const int c = task / mt, p0 = 16 * (task - c * mt), jx = (q0 + c) / C;
            const float lc = a.tx.lam[jx] + a.tc.lam[q0 + c - jx * C] + a.ty.lam[min(freq_of(ay, p0 + (lane & 15)), Y - 1)];
            float* const rows = tile + (long long)c * P * pitch;
            t_product<PT, true>(rows, pitch, P, tf, a.tt.mat, p0, lc, lamt);
            t_product<PT, false>(rows, pitch, P, ti, a.tt.mat + P * P, p0, 0.f, nullptr);
        }
    }
    __syncthreads();
    if (ndc) {
        for (int e = threadIdx.x; e < ndc; e += nth) tile[e * pitch] = dcl[e];
        __syncthreads();
    }
    product<RT, MI>(tile, pitch, ay, sh, ring);
    for (int e = threadIdx.x; e < tot; e += nth) {
        const int q = div_by(e, mp, P), t = e - q * P, c = div_by(q, mh, h), y = q - c * h;
        const float* const o = tile + (c * P + t) * pitch + y;
        float* const s = base + (long long)c * Y * P + t;
        const float ev = o[0];
        if (!ay.fold) {
            s[y * P] = ev;
        } else {
            const float od = o[H];
            s[y * P] = ev + od;
            if (2 * y + 1 != Y) s[(Y - 1 - y) * P] = ev - od;
        }
    }
}

// Output tiles of an axis, and its waves: two tiles per wave past 16.
int axis_tiles(int n, int periodic) { return (dense_fold(n, periodic) ? 2 : 1) * dense_width(n, periodic) / 16; }
int axis_mi(int tiles) { return tiles <= 16 ? 1 : 2; }
int axis_waves(int tiles, int nb) {
    const int w = (tiles + axis_mi(tiles) - 1) / axis_mi(tiles);
    return std::max((w + nb - 1) / nb * nb, 4);
}
size_t axis_lds(int n, int periodic, int rt) { return 16 * (size_t)rt * (16 * axis_tiles(n, periodic) + 4) * 4; }

// Times per row group of the x passes: as many rows as keep two blocks per
// compute unit (a matrix entry loaded serves them all), evened out.
int dx_groups(const Geom& g, int* rt) {
    const int nyb = g.Y * g.B;
    int best = g.P;                            // one time per group
    for (int r = 4; r >= 1; --r) {
        const int cap = 16 * r / g.C, groups = (g.P + cap - 1) / cap;
        if (axis_lds(g.X, g.perx, r) > kDLds / 2 && r > 1) continue;
        best = groups;
        if ((long long)nyb * groups >= 512) break;
    }
    const int tb = (g.P + best - 1) / best;
    *rt = (g.C * tb + 15) / 16;
    return (g.P + tb - 1) / tb;
}

// Lines (jx, colour mode) per block of the y and time pass: as many as leave two
// blocks per compute unit, up to 64 rows (they share the matrix loads).
int dyt_lines(const Geom& g) {
    const long long lines = (long long)g.X * g.C * g.B;
    return (int)std::max(1ll, std::min<long long>(kDMaxP / g.P, lines / 512));
}

template <int RT, bool INV>
void dx_launch(const DenseArgs& a, unsigned blocks, size_t lds, hipStream_t st) {
    const int tiles = axis_tiles(a.g.X, a.g.perx);
    const dim3 grid(blocks), block(64 * axis_waves(tiles, a.ax.fold ? 2 : 1));
    if (axis_mi(tiles) == 1) hipLaunchKernelGGL((k_dx<RT, 1, INV>), grid, block, lds, st, a);
    else hipLaunchKernelGGL((k_dx<RT, 2, INV>), grid, block, lds, st, a);
}

template <bool INV>
void dx_dispatch(const DenseArgs& a, int rt, unsigned blocks, size_t lds, hipStream_t st) {
    if (rt == 1) dx_launch<1, INV>(a, blocks, lds, st);
    else if (rt == 2) dx_launch<2, INV>(a, blocks, lds, st);
    else if (rt == 3) dx_launch<3, INV>(a, blocks, lds, st);
    else dx_launch<4, INV>(a, blocks, lds, st);
}

template <int RT, int MI>
void dyt_launch_mi(const DenseArgs& a, dim3 grid, dim3 block, size_t lds, hipStream_t st) {
    if (a.g.P <= 16) hipLaunchKernelGGL((k_dyt<RT, MI, 1>), grid, block, lds, st, a);
    else if (a.g.P <= 32 && (RT < 3 || MI == 1))   // (past that the registers do not hold both matrices)
        hipLaunchKernelGGL((k_dyt<RT, MI, RT < 3 || MI == 1 ? 2 : 0>), grid, block, lds, st, a);
    else hipLaunchKernelGGL((k_dyt<RT, MI, 0>), grid, block, lds, st, a);
}

template <int RT>
void dyt_launch(const DenseArgs& a, hipStream_t st) {
    const int tiles = axis_tiles(a.g.Y, a.g.pery);
    const dim3 grid((a.g.X * a.g.C + a.lpb - 1) / a.lpb, a.g.B), block(64 * axis_waves(tiles, a.ay.fold ? 2 : 1));
    const size_t lds = axis_lds(a.g.Y, a.g.pery, RT);
    if (axis_mi(tiles) == 1) dyt_launch_mi<RT, 1>(a, grid, block, lds, st);
    else dyt_launch_mi<RT, 2>(a, grid, block, lds, st);
}

}  // namespace

bool dense_fold(int n, int periodic) { return !periodic && n > 16; }
int dense_width(int n, int periodic) { return ((dense_fold(n, periodic) ? (n + 1) / 2 : n) + 15) / 16 * 16; }

size_t dense_axis_floats(int n, int periodic) {
    const size_t H = dense_width(n, periodic), nb = dense_fold(n, periodic) ? 2 : 1;
    return 2 * nb * H * H + 256 * (size_t)kDenseAxisPad;
}

void dense_axis_fill(int n, int periodic, const double* M, float* out) {
    const int H = dense_width(n, periodic), T = H / 16;
    const bool fold = dense_fold(n, periodic);
    const int nb = fold ? 2 : 1, h = fold ? (n + 1) / 2 : n;
    std::fill(out, out + dense_axis_floats(n, periodic), 0.f);
    for (int inv = 0; inv < 2; ++inv)
        for (int b = 0; b < nb; ++b)
            for (int o = 0; o < H; ++o)            // output and input position of block b
                for (int i = 0; i < H; ++i) {
                    const int fp = inv ? i : o, x = inv ? o : i, j = fold ? 2 * fp + b : fp;
                    if (j >= n || x >= h || (b == 1 && 2 * x + 1 == n)) continue;
                    const size_t frag = ((size_t)(inv * nb + b) * T + o / 16) * T + i / 16;
                    const int lane = o % 16 + 16 * (i % 16 / 4);
                    out[(frag * 64 + lane) * 4 + i % 4] = (float)M[(size_t)j * n + x];
                }
}

DenseAxis dense_axis(int n, int periodic, const float* dev) {
    DenseAxis a;
    a.H = dense_width(n, periodic);
    a.fold = dense_fold(n, periodic);
    a.fwd = dev;
    a.inv = dev + (size_t)(a.fold ? 2 : 1) * a.H * a.H;
    return a;
}

bool dense3_ok(const Geom& g) {
    if (!rows_ok(g) || g.P > kDMaxP || g.X > kDMaxL || g.Y > kDMaxL || g.B > 65535) return false;
    const int m = dyt_lines(g), rt = (g.P * m + 15) / 16;
    int rx;
    dx_groups(g, &rx);
    // (entries of a tile are divided by reciprocals, exact below 2^16)
    return axis_lds(g.Y, g.pery, rt) <= kDLds && axis_lds(g.X, g.perx, rx) <= kDLds &&
           (long long)m * g.P * g.Y < 65536 && 64ll * g.X < 65536;
}

void launch_dense3(const Geom& g, float* R, float* Rt, const AxisTab& tx, const AxisTab& ty,
                   const AxisTab& tc, const AxisTab& tt, const DenseAxis& ax, const DenseAxis& ay,
                   const double* tc64, const double* tt64, double* part_slice, int nbx, int pass,
                   const float* frz, hipStream_t st) {
    DenseArgs a{};
    a.g = g; a.R = R; a.Rt = Rt; a.tx = tx; a.ty = ty; a.tc = tc; a.tt = tt; a.ax = ax; a.ay = ay;
    a.tc64 = tc64; a.tt64 = tt64; a.part = part_slice; a.nbx = nbx; a.frz = frz;
    if (pass == 1) {
        a.lpb = dyt_lines(g);
        switch ((g.P * a.lpb + 15) / 16) {
            case 1: dyt_launch<1>(a, st); break;
            case 2: dyt_launch<2>(a, st); break;
            case 3: dyt_launch<3>(a, st); break;
            default: dyt_launch<4>(a, st); break;
        }
        return;
    }
    int rt;
    a.nrg = dx_groups(g, &rt);
    a.tb = (g.P + a.nrg - 1) / a.nrg;
    const long long planes = (long long)g.B * g.P * g.C, per8 = 8 * kSumPlanesPerBlock;
    a.nsb = pass == 0 ? (int)((planes + per8 - 1) / per8 * 8) : 0;
    const unsigned blocks = (unsigned)(a.nsb + (long long)g.Y * g.B * a.nrg);
    const size_t lds = axis_lds(g.X, g.perx, rt);
    if (pass == 0) dx_dispatch<false>(a, rt, blocks, lds, st);
    else dx_dispatch<true>(a, rt, blocks, lds, st);
}

}  // namespace otd
