// k_gather_colifft.hip -- step P5 (polar -> Cartesian interpolation in the
// frequency domain, Section 2) fused with the first half of P6 (the inverse
// DFT along k_y) and the row part of P7/P8 (shift and crop).
//
// A block owns F neighbouring Cartesian columns k_x = a*dk (a in [0, G/2))
// and all G rows k_y = b*dk of each, b in FFT order; thread t works on column
// t mod F, so the lanes of a wave cover F neighbouring columns times 64/F
// neighbouring rows, and their polar reads fall on few cache lines (the same
// angle row, consecutive radii). Columns go to XCDs in contiguous ranges so
// neighbouring columns share an L2.
//
// With linear radial taps the polar spectra of Q = 2 consecutive slices are
// stored interleaved, sample by sample, in cache-line tiles of 2 angles x 4
// samples (PolarTiles): one tap of one point reads both slices' values of a
// sample as 16 contiguous bytes, and the four samples of a point's two angle
// rows mostly share one or two lines (simulated over the 2048 x 4096 gather
// points of N = 2048 with two columns per block: 7.9 distinct 128-byte lines
// per wave and slice, against 9.9 for interleaved rows and 16.4 for one
// slice per row). A block therefore gathers both slices of a group at once;
// their column transforms run one after the other. Cubic taps keep one slice
// per group in plain rows (Q = 1), and uneven batches too (their slices differ
// in V).
//
// A thread gathers the points its transform starts from, so gathered values
// stay in its registers (16 points per thread at two waves per SIMD from G =
// 2048 on, which takes one LDS exchange fewer than 8 points at four). The polar
// reads (64 slices of 2048^2: 1.28 ms on their own, bound by the latency of L1
// misses), the transforms (0.87 ms, vector ALU) and the grid stores (0.4 ms)
// ran one after the other, 2.2 ms; a block that walks several groups now reads
// the next group's points between the butterflies of the current one, a pair's
// first slice waiting in LDS: 2.02 ms (cubic taps at P_c = 1: 1.28 -> 1.11).
// Blocks of one group keep nothing in LDS but the transforms and overlap
// through several blocks per compute unit: 8 slices of 256^2 42.8 -> 13.2 us,
// 2 of 2048^2 89 -> 66, one of 256^2 16.7 -> 10.2 (the coordinates' part of
// that below).
//
// Each thread keeps the interpolation coordinates of its E points in
// three registers each and reuses them for every slice of its chunk. They
// are exact to FP32 rounding although radius and angle indices reach a few
// thousand (gather_point.h):
//   radius index r = |(a,b)| P_r/P_c: m = floor(r) corrected by exact integers,
//   its fraction by Newton steps on the integer r^2 - m^2;
//   angle index: a polynomial arctangent picks the interval [theta_j0,
//   theta_j0+1), then the offset inside it is the arcsine of the cross product
//   of the point direction with (cos theta_j0, sin theta_j0), which come from
//   a table as FP32 pairs; the products' rounding errors are carried along, so
//   the fraction carries no cancellation (non-uniform angles: cross products in
//   FP64).
// Bound by vector ALU issue: about 100 FP32 operations and one 16-byte table
// read per point, the reads of a thread's points in flight together. The
// coordinates of a 2048^2 slice take 20 us of the whole GPU per chunk of
// slices where every point's are formed (34 us with an FP64 square root, FP64
// cross products and the library arctangent, one point after the other); at N =
// 4096 and two slices the kernel went from 400 to 315 us, 96 uneven sinograms
// from 4.9 to 4.3 ms.
// Per slice, the column is inverse-transformed along b, and only the N rows
// that survive the crop are written, to a grid laid out [N/8][GT][8]
// (complex, GT >= G/2 columns per tile row): the 8 rows of a tile and
// neighbouring columns form contiguous runs, and the row kernel reads each
// 8-row tile contiguously.
//
// Gather rules (bilinear in (r, q)):
//   b >= 0: theta = atan2(b, a), sample as stored; b < 0: theta + pi, conjugate
//   (y(t, theta + pi) = y(-t, theta)); the angle neighbour past theta_{V-1}
//   is theta_0 with the conjugation flipped; radial samples m >= M/2 are zero.
//   Origin (0,0): dc_scale * sum_j dt*Y_j[0] (mean for FBP, kappa/dk * mean
//   for plain B).
#include "bst_internal.h"
#include "bst_check.h"
#include "fft_lds.h"

namespace bst {

// Points (transform values) per thread: 16 from G = 2048 on, at two waves per
// SIMD, 8 below, at four. It fixes the transform's arithmetic, so it depends on
// G alone: a slice's result is the same in every batch.
constexpr int gather_points(int G) { return G >= 2048 ? 16 : 8; }
// Threads per block (the columns per block follow). PIPE: blocks that walk
// several groups, each group's gather overlapped with the previous one's
// transforms (G >= 2048). The others overlap through several blocks per compute
// unit. (256-thread blocks of one column at G = 4096 lose the shared lines: 2.57 ms
// against 2.03 for 64 slices of 2048^2; 128-thread ones at G = 1024 and 2048
// gather 1.1 to 1.3 times slower, 512-thread ones up to 1.3 times.)
constexpr int gather_threads(int G, bool pipe) { return pipe && G >= 4096 ? 512 : (G <= 512 ? 128 : 256); }
// Threads that add up a slice's origin terms: the ordinary kernels' block, at most
// 256.
constexpr int gather_sum_threads(int G) {
    const int all = G / 2 * (G / gather_points(G)), most = gather_threads(G, false);
    return all < most ? all : most;
}
// arithmetic instructions between two polar reads of the overlapped gather
// (64 slices of 2048^2: 2.17 ms with 8, 2.06 with 14, 2.04 with 20, 2.07 with 28)
constexpr int kReadSpacing = 20;

// Word 3 of a CDNA buffer resource for plain dword data (32-bit data format,
// no swizzle, raw offsets).
constexpr int kBufferWord3 = 0x00020000;

// One slice group's polar block as a buffer resource: loads take a 32-bit
// byte offset in one VGPR against a base held in SGPRs, and read 0 past the
// end. The block holds at most 16384 x 4101 x 32 bytes (< 2^32). The base and
// size, the same in every lane, are read from the first one: where the
// compiler loses sight of that it serialises every load over the lanes.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t polar_rsrc(const float2* base, unsigned bytes) {
    const unsigned long long p = (unsigned long long)base;
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)p), hi = __builtin_amdgcn_readfirstlane((unsigned)(p >> 32));
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<float2*>(((unsigned long long)hi << 32) | lo), 0,
                                             __builtin_amdgcn_readfirstlane((int)bytes), kBufferWord3);
}

__device__ __forceinline__ float4 load16(__amdgpu_buffer_rsrc_t r, unsigned off) {
    const auto q = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
    return make_float4(__uint_as_float(q[0]), __uint_as_float(q[1]), __uint_as_float(q[2]), __uint_as_float(q[3]));
}

template <int LOGG, int QV, int CAP, bool PIPE>
struct GatherCfg {
    static constexpr int G = 1 << LOGG;
    static constexpr int Q = QV;                         // slices per polar group
    static constexpr int E = gather_points(G);           // points (values) per thread
    static constexpr int T = G / E;
    static constexpr int WAVES = E == 16 ? 2 : 4;        // per SIMD, for the registers
    static constexpr int F1 = CAP > T ? CAP / T : 1;     // columns per block:
    static constexpr int F = F1 < G / 2 ? F1 : G / 2;    // no more than exist
    static constexpr int WG = F * T;
    // transform stride in LDS (float2; a power of two, the columns' lanes
    // interleaved and their positions told apart by region_xor)
    static constexpr int STRIDE = G;
    static constexpr int REGION = F * STRIDE;            // one slice's F transforms
    static constexpr bool PARK = PIPE && Q == 2;         // a second region: a pair's parked slice
    static constexpr int NREG = PARK ? 2 : 1;
};

// f(integral_constant<int, i>) for i = 0 .. N - 1
template <int N, int I = 0, class F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<N, I + 1>(f);
    }
}

// Sums of Q values over the block, in a fixed order: each wave's lanes, then the
// waves. red: Q floats per wave.
template <int WG, int Q>
__device__ __forceinline__ void block_sums(float (&x)[Q], float* red) {
    constexpr int NW = (WG + 63) / 64;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
#pragma unroll
        for (int k = 0; k < Q; ++k) x[k] += __shfl_xor(x[k], o, 64);
    }
#pragma unroll
    for (int k = 0; k < Q; ++k)
        if ((threadIdx.x & 63) == 0) red[k * NW + (threadIdx.x >> 6)] = x[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < Q; ++k) {
        x[k] = 0.f;
#pragma unroll
        for (int i = 0; i < NW; ++i) x[k] += red[k * NW + i];
    }
    __syncthreads();
}

// Interpolation stencil of one Cartesian point, fixed for all slices:
//   o0      sample index (one unit is the Q slices' values of one sample,
//           8 Q bytes) of the first radial tap of angle j0; the taps of j1
//           are one polar row further, or, when j1 wraps to angle 0, (V-1)
//           rows back. In the tiled layout of two slices (PolarTiles) bit 29
//           says the second radial tap starts the next tile (m0 = 3 mod 4) and
//           bit 30 that j0 is odd (j1 in the next tile row). Bit 31 flips the conjugation of the j0 taps
//           (non-uniform angles, below theta_0, where the j0 neighbour is the
//           image theta_{V-1} - pi);
//   g       radial fraction, its sign bit set when j1 wraps;
//   w1      angular weight f of the j1 taps, negative when they are
//           conjugated. The j0 taps have weight 1 - f and are conjugated for
//           the lower half-plane b < 0 (known at compile time from the
//           point's slot in the thread), unless bit 31 of o0 flips it.
// Points outside the radial data (and the origin, which the DC rule sets
// afterwards) point at the zero slots that end rows 0 and 1, so every point
// runs the same branch-free code.
struct Stencil {
    unsigned o0;
    float g, w1;
};
constexpr unsigned kOffsetMask = 0x7FFFFFFFu;
constexpr unsigned kSampleMask = 0x1FFFFFFFu;  // o0 without its flag bits
constexpr int kSeriesAngles = 16;              // fewer angles: the library arctangent

// Uniform angles of a slice: the plan's table, or (uneven batches, a count per
// slice) the slice's own (split_direction of j pi / V); V / pi as an FP32 pair.
struct AngleView {
    int V;
    float vpi_f, vpi_lo;
    const float4* dir;
};

// Arctangent of y / x, y >= 0, to 1e-5 (Abramowitz and Stegun 4.4.49): picks
// the angle interval only (V <= 16384: within a tenth of a step), the offset in
// it is exact.
__device__ __forceinline__ float coarse_angle(float x, float y) {
    const float ax = fabsf(x);
    const float t = fminf(ax, y) * __builtin_amdgcn_rcpf(fmaxf(ax, y));
    const float u = t * t;
    float th = fmaf(u, 0.0208351f, -0.0851330f);
    th = fmaf(u, th, 0.1801410f);
    th = fmaf(u, th, -0.3302995f);
    th = t * fmaf(u, th, 0.9998660f);
    if (y > ax) th = 1.57079633f - th;
    return x < 0.f ? 3.14159265f - th : th;
}

// conjugation of the j0 taps of point e: the lower half-plane, flipped by bit
// e of `flips` (bit 31 of the point's o0, collected once per block)
template <bool NU>
__device__ __forceinline__ bool lower_j0(unsigned flips, int e, bool lower) {
    if constexpr (NU) return lower != (((flips >> e) & 1u) != 0u);
    return lower;
}

// First guess of a point's angle index, at most one off.
__device__ __forceinline__ int angle_guess(int col, int bs, const AngleView& av) {
    const float x = bs < 0 ? -(float)col : (float)col;
    const int j = (int)(coarse_angle(x, fmaxf(fabsf((float)bs), 1e-20f)) * av.vpi_f);  // (0, 0): any index
    return min(max(j, 0), av.V - 1);
}

// Stencil of Cartesian point (col, bs); bs signed. NU: non-uniform angles.
// SERIES: uniform, at least kSeriesAngles angles. guess, cs: the angle index
// from angle_guess and its table entry (uniform angles). mirror: also the
// stencil of (col, -bs) (SERIES, bs >= 0, not the tent rule's wide points).
// TENT: a wide point of the tent rule (|bs| <= B_col) gets bit 31 of o0 and
// its patch slot in the low bits; its polar reads go to the zero slots.
template <bool TILED>
__device__ __forceinline__ unsigned sample_code(const GatherArgs& a, int j, int m) {
    // 32-bit: a group has at most 16384 x 4104 samples
    if constexpr (TILED)
        return (__umul24((unsigned)j >> 1, (unsigned)((a.S + 3) >> 2)) + ((unsigned)m >> 2)) * 8u +
               (unsigned)((j & 1) * 4 + (m & 3)) + ((unsigned)((m & 3) == 3) << 29) + ((unsigned)(j & 1) << 30);
    else
        return __umul24((unsigned)j, (unsigned)a.S) + (unsigned)m;
}

template <bool NU, bool TENT, bool TILED, bool SERIES>
__device__ __forceinline__ Stencil point_stencil(int col, int bs, const GatherArgs& a, const AngleView& av,
                                                 int guess, float4 cs, Stencil* mirror = nullptr) {
    // points without a stencil of their own: the origin, radii past the data
    Stencil none;
    none.o0 = sample_code<TILED>(a, 0, a.zero_slot);
    none.g = none.w1 = 0.f;
    const int n = max(col * col + bs * bs, 1);
    const int up = a.radius.shift > 0 ? 2 * a.radius.shift : 0, down = a.radius.shift < 0 ? -2 * a.radius.shift : 0;
    bool empty = (col == 0 && bs == 0) ||
                 (n << up) >= (int)(__umul24((unsigned)a.zero_slot, (unsigned)a.zero_slot) << down);
    if constexpr (TENT) {
        const int2 tc = a.tent_cols[col];
        if (!(col == 0 && bs == 0) && bs >= -tc.y && bs <= tc.y) {
            none.o0 = (unsigned)(tc.x + bs + tc.y) | 0x80000000u;
            empty = true;
        }
    }
    // the series variant runs on to the end with every point, so that the
    // table reads of a thread's points overlap
    if (!SERIES && empty) return none;
    const RadialIndex rad = radial_index(n, __builtin_amdgcn_rsqf((float)n), a.radius);
    const int m0 = rad.m;
    const float g = rad.g;

    // direction of the point on [0, pi): (x, y) with y >= 0
    const bool lower = bs < 0;
    const int x = lower ? -col : col;
    const int y = lower ? -bs : bs;
    int j0;
    float f;
    bool flip0 = false;
    if constexpr (!NU) {
        const float xf = (float)x, yf = (float)y;
        if constexpr (SERIES) {
            f = angle_offset(xf, yf, cs, rad, av.vpi_f, av.vpi_lo);
        } else {
            const double c = (double)cs.x + (double)cs.y, sn = (double)cs.z + (double)cs.w;
            const float cross = (float)((double)y * c - (double)x * sn), dot = (float)((double)x * c + (double)y * sn);
            f = atan2f(cross, dot) * av.vpi_f;
        }
        // the interval next to the guessed one, where there is one
        j0 = min(max(guess + (int)floorf(f), 0), av.V - 1);
        f = fminf(fmaxf(f - (float)(j0 - guess), 0.f), 1.f);
    } else {
        // theta_j <= theta exactly when the cross product e_j x u is >= 0 (both
        // directions in [0, pi)): binary search for the last such j, between
        // the angles below the bucket edges that enclose theta (the coarse
        // angle is within 2e-5 of it). For V = 377 golden-angle projections
        // that takes one probe where the whole range took nine, each a
        // dependent 16-byte read: 5 slices of 512^2 gather in 22 us, 29 before.
        auto at_or_before = [&](int jj) {
            const double2 e = a.ang[jj];
            return (double)y * e.x - (double)x * e.y >= 0.0;
        };
        const float th = coarse_angle((float)x, (float)y), scale = (float)a.ang_buckets * 0.318309886f;
        const int k0 = min(max((int)floorf((th - 3e-5f) * scale), 0), a.ang_buckets);
        const int k1 = min(max((int)floorf((th + 3e-5f) * scale) + 1, 0), a.ang_buckets);
        int lo = k0 > 0 ? a.ang_below[k0] - 1 : -1, hi = k1 < a.ang_buckets ? a.ang_below[k1] : a.V;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (at_or_before(mid)) lo = mid; else hi = mid;
        }
        double ex, ey;  // direction of the lower neighbour
        if (lo < 0) {
            j0 = a.V - 1;  // below theta_0: the image theta_{V-1} - pi, conjugated
            flip0 = true;
            ex = -a.ang[j0].x;
            ey = -a.ang[j0].y;
        } else {
            j0 = lo;
            ex = a.ang[j0].x;
            ey = a.ang[j0].y;
        }
        const double cross = (double)y * ex - (double)x * ey;
        const double dot = (double)x * ex + (double)y * ey;
        f = fminf(fmaxf(atan2f((float)cross, (float)dot) * a.inv_gap[j0], 0.f), 1.f);
    }
    // past theta_{V-1} the neighbour is theta_0 + pi: conjugated (both
    // neighbours of a point below theta_0 are already in place)
    const bool wrap = (j0 + 1 == av.V);
    const bool conj1 = lower != (wrap && !flip0);
    Stencil st;
    st.o0 = sample_code<TILED>(a, j0, m0) | ((unsigned)flip0 << 31);
    st.g = __uint_as_float(__float_as_uint(g) | ((unsigned)wrap << 31));
    st.w1 = conj1 ? -f : f;
    if (mirror) {
        // (a, -b), b > 0: direction pi - theta, between the angles V - 1 - j0
        // and V - j0 at fraction 1 - f, all of it conjugated but the image past
        // theta_{V-1}
        const bool mwrap = j0 == 0;
        mirror->o0 = sample_code<TILED>(a, av.V - 1 - j0, m0);
        mirror->g = __uint_as_float(__float_as_uint(g) | ((unsigned)mwrap << 31));
        mirror->w1 = mwrap ? 1.f - f : f - 1.f;
        if (empty) *mirror = none;
    }
    return empty ? none : st;
}

// Grid stores are non-temporal: the row kernel reads them only after this
// kernel ends, and 2 GB of them per 64 slices would otherwise evict the polar
// lines the gather reuses.
__device__ __forceinline__ void store_streaming(float2* p, float2 v) {
    typedef float f2v __attribute__((ext_vector_type(2)));
    const f2v t = {v.x, v.y};
    __builtin_nontemporal_store(t, reinterpret_cast<f2v*>(p));
}

// Column `col`'s rows of one slice that survive the crop, those of points e <
// KEEP and e >= E - KEEP, to the slice's grid D (8-row tiles [N/8][GT][8]).
// From T = 8 on the rows of a thread differ by whole tiles: one 32-bit lane
// offset (a slice has at most 2^27 bytes) against a base per point.
template <int LOGG, int E, int KEEP>
__device__ __forceinline__ void store_rows(const float2 (&v)[E], float2* D, const GatherArgs& a, int j, int col) {
    constexpr int G = 1 << LOGG, T = G / E;
    constexpr int N = G * 2 * KEEP / E;
    [[maybe_unused]] const unsigned elems = (unsigned)N * (unsigned)a.GT;
    const unsigned lane = (((unsigned)j >> 3) * (unsigned)a.GT + (unsigned)col) * 8u + ((unsigned)j & 7u);
#pragma unroll
    for (int e = 0; e < E; ++e) {
        if (e >= KEEP && e < E - KEEP) continue;
        const int first = e * T + (e < KEEP ? N / 2 : N / 2 - G);  // row of thread 0
        if constexpr (T >= 8) {
            const unsigned base = (unsigned)(first / 8) * (unsigned)a.GT * 8u;
            store_streaming(D + base + BST_IDX(lane, elems - base, 2), v[e]);
        } else {
            const unsigned p = (unsigned)(first + j);
            store_streaming(D + BST_IDX(((p >> 3) * (unsigned)a.GT + (unsigned)col) * 8u + (p & 7u), elems, 2), v[e]);
        }
    }
}

// Keys cubic convolution (a = -1/2) over samples m0-1 .. m0+2 at fraction g:
// the Catmull-Rom weights.
__device__ __forceinline__ float2 keys4(float2 sm, float2 s0, float2 s1, float2 s2, float g) {
    const float g2 = g * g, g3 = g2 * g;
    const float wm = 0.5f * (-g3 + 2.f * g2 - g);
    const float w0 = 0.5f * (3.f * g3 - 5.f * g2 + 2.f);
    const float w1 = 0.5f * (-3.f * g3 + 4.f * g2 + g);
    const float w2 = 0.5f * (g3 - g2);
    return make_float2(fmaf(w2, s2.x, fmaf(w1, s1.x, fmaf(w0, s0.x, wm * sm.x))),
                       fmaf(w2, s2.y, fmaf(w1, s1.y, fmaf(w0, s0.y, wm * sm.y))));
}
// Angular (linear) combination of the two rows' radial values: weight
// 1 - |w1| for the j0 row, conjugated in the lower half-plane, and w1 (sign =
// conjugation) for the j1 row.
__device__ __forceinline__ float2 angular(float2 u0, float2 u1, float w1, bool lower) {
    const float a0 = 1.f - fabsf(w1);
    const float w0 = lower ? -a0 : a0;
    return make_float2(fmaf(fabsf(w1), u1.x, a0 * u0.x), fmaf(w1, u1.y, w0 * u0.y));
}

// One polar row's taps for the Q slices: linear taps read the samples m0,
// m0+1 (16 Q bytes), cubic taps m0-1 .. m0+2 (32 Q bytes); then their radial
// values.
template <int TAPS, int Q>
__device__ __forceinline__ void load_row(__amdgpu_buffer_rsrc_t P, unsigned off, float4 (&q)[TAPS * Q / 2]) {
#pragma unroll
    for (int i = 0; i < TAPS * Q / 2; ++i) q[i] = load16(P, off + 16u * i);
}
// value of slice k at tap t: complex number t Q + k of the row's run
template <int Q>
__device__ __forceinline__ float2 tap(const float4* q, int t, int k) {
    const int i = t * Q + k;
    const float4& h = q[i >> 1];
    return (i & 1) ? make_float2(h.z, h.w) : make_float2(h.x, h.y);
}
template <int TAPS, int Q>
__device__ __forceinline__ void radial_row(const float4 (&q)[TAPS * Q / 2], float g, float2 (&u)[Q]) {
#pragma unroll
    for (int k = 0; k < Q; ++k) {
        if constexpr (TAPS == 2) {
            const float2 x0 = tap<Q>(q, 0, k), x1 = tap<Q>(q, 1, k);
            u[k] = make_float2(fmaf(g, x1.x - x0.x, x0.x), fmaf(g, x1.y - x0.y, x0.y));
        } else {
            u[k] = keys4(tap<Q>(q, 0, k), tap<Q>(q, 1, k), tap<Q>(q, 2, k), tap<Q>(q, 3, k), g);
        }
    }
}

// One block's work: columns lblock * F .. + F - 1 for the slices
// [s_begin, s_end) (whole groups of Q). The slices share one angle set: the
// plan's, or (per-slice counts) that of slice s_begin.
template <int LOGG, int TAPS, bool NU, bool TENT, int Q, int CAP, bool PIPE>
__device__ __forceinline__ void gather_body(const GatherArgs& a, int lblock, int s_begin, int s_end) {
    using C = GatherCfg<LOGG, Q, CAP, PIPE>;
    constexpr int G = C::G, T = C::T, F = C::F, E = C::E;
    constexpr unsigned kSampleBytes = Q * sizeof(float2);
    constexpr bool TILED = Q == 2 && TAPS == 2;  // the 2 x 4 x 2 tiles of PolarTiles
    __shared__ float2 lds[C::NREG * C::REGION];
    __shared__ float red[Q * ((C::WG + 63) / 64)];
    const int fid = threadIdx.x % F;
    const int j = threadIdx.x / F;
    const int col = lblock * F + fid;
    const int V = a.Vs ? a.Vs[s_begin] : a.V;  // this chunk's projections
    AngleView av{V, a.vpi_f, a.vpi_lo, a.dir};
    if (a.Vs) {
        const double vpi = (double)V / M_PI;
        av.vpi_f = (float)vpi;
        av.vpi_lo = (float)(vpi - (double)av.vpi_f);
        av.dir = a.dir + a.ang_off[s_begin];
    }
    const float dc_scale = a.Vs ? a.dc_rule / (float)V : a.dc_scale;
    const bool live = col < G / 2;
    const FftTwiddles<LOGG, +1, E, 2> tw(j, a.tw);

    // Stencils, held in registers for the whole chunk of slices. Uniform
    // angles: the table reads of all the thread's points first, so that they
    // are in flight together. The variants with a library arctangent keep one
    // copy of it in a rolled loop, staged through the still unused transform
    // LDS in chunks of CH points.
    Stencil pt[E];
    const int c = live ? col : 0;
    auto row = [&](int e) {  // signed row of point e
        const int b = j + e * T;
        return live ? (b < G / 2 ? b : b - G) : 0;
    };
    if (!NU && V >= kSeriesAngles) {
        // the upper half-plane's rows, and from each its mirror image, which
        // thread T - j (of the same column) takes over through LDS: row b of
        // thread j and point e is row -b of thread T - j and point E - 1 - e
        // (of thread 0 and point E - e for j = 0). Half the coordinates: one 256^2
        // slice 18.4 -> 17.9 us, 96 uneven sinograms 3.48 -> 3.43 ms
        constexpr int H = E / 2;
        static_assert(C::NREG * C::REGION * 2 >= C::WG * H * 3, "the exchange needs LDS");
        unsigned* xch = reinterpret_cast<unsigned*>(lds);
        int guess[H];
        float4 cs[H];
#pragma unroll
        for (int e = 0; e < H; ++e) {
            guess[e] = angle_guess(c, row(e), av);
            cs[e] = av.dir[guess[e]];
        }
#pragma unroll
        for (int e = 0; e < H; ++e) {
            Stencil m;
            pt[e] = point_stencil<NU, TENT, TILED, true>(c, row(e), a, av, guess[e], cs[e], &m);
            unsigned* d = xch + (e * 3) * C::WG + threadIdx.x;
            d[0] = m.o0;
            d[C::WG] = __float_as_uint(m.g);
            d[2 * C::WG] = __float_as_uint(m.w1);
        }
        __syncthreads();
        const int from = (j == 0 ? 0 : (T - j) * F) + fid;
#pragma unroll
        for (int e = H; e < E; ++e) {
            const int se = j == 0 ? min(E - e, H - 1) : E - 1 - e;
            const unsigned* d = xch + (se * 3) * C::WG + from;
            pt[e].o0 = d[0];
            pt[e].g = __uint_as_float(d[C::WG]);
            pt[e].w1 = __uint_as_float(d[2 * C::WG]);
            if constexpr (TENT) {
                const int2 tc = a.tent_cols[c];
                if (live && row(e) >= -tc.y) {
                    pt[e].o0 = (unsigned)(tc.x + row(e) + tc.y) | 0x80000000u;
                    pt[e].g = pt[e].w1 = 0.f;
                }
            }
        }
        if (j == 0) {  // row -G/2 has no mirror image in the grid
            const int g0 = angle_guess(c, row(H), av);
            pt[H] = point_stencil<NU, TENT, TILED, true>(c, row(H), a, av, g0, av.dir[g0]);
        }
        __syncthreads();  // the transforms reuse this LDS
    } else {
        constexpr int CH = 2;
        constexpr int NW = 3;  // words per stencil
        static_assert(C::NREG * C::REGION * 2 >= C::WG * CH * NW, "stencil staging needs LDS");
        unsigned* stage = reinterpret_cast<unsigned*>(lds);
#pragma unroll
        for (int c0 = 0; c0 < E; c0 += CH) {
#pragma unroll 1
            for (int h = 0; h < CH; ++h) {
                const int guess = NU ? 0 : angle_guess(c, row(c0 + h), av);
                const float4 cs = NU ? make_float4(0.f, 0.f, 0.f, 0.f) : av.dir[guess];
                const Stencil st = point_stencil<NU, TENT, TILED, false>(c, row(c0 + h), a, av, guess, cs);
                unsigned* d = stage + (h * NW) * C::WG + threadIdx.x;
                d[0] = st.o0;
                d[C::WG] = __float_as_uint(st.g);
                d[2 * C::WG] = __float_as_uint(st.w1);
            }
#pragma unroll
            for (int h = 0; h < CH; ++h) {
                const unsigned* d = stage + (h * NW) * C::WG + threadIdx.x;
                pt[c0 + h].o0 = d[0];
                pt[c0 + h].g = __uint_as_float(d[C::WG]);
                pt[c0 + h].w1 = __uint_as_float(d[2 * C::WG]);
            }
        }
        __syncthreads();  // the transforms reuse this LDS
    }
    // non-uniform angles: the j0 conjugation flips move to one bit mask; the
    // tent rule: wide points likewise (their o0 keeps the patch slot)
    unsigned flips = 0u, wide = 0u;
    if constexpr (NU || TENT) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            (NU ? flips : wide) |= (pt[e].o0 >> 31) << e;
            pt[e].o0 &= kOffsetMask;
        }
    }
    const unsigned zcode = sample_code<TILED>(a, 0, a.zero_slot);  // a zero sample
    const unsigned zoff = (zcode & kSampleMask) * kSampleBytes;

    const PolarTiles lay{Q, a.V, a.S};
    const unsigned group_bytes = (unsigned)(lay.group_elems() * sizeof(float2));
    const unsigned row_bytes = (unsigned)a.S * kSampleBytes;
    const unsigned wrap_bytes = 0u - (unsigned)(V - 1) * row_bytes;  // back to row 0
    // tiled: from angle j to j + 1 (j even: the tile's second half; j odd:
    // the next tile row's first), and from angle V - 1 back to angle 0
    const unsigned tile_row_bytes = (unsigned)lay.tiles_per_row() * 128u;
    const unsigned tile_next = tile_row_bytes - 64u;
    const unsigned tile_wrap = 0u - (unsigned)((V - 1) >> 1) * tile_row_bytes - (unsigned)((V - 1) & 1) * 64u;
    const unsigned off = (unsigned)(fid * C::STRIDE) * 8u;  // column fid's transform region
    const int xm = region_xor<LOGG, F>(fid);
    float2* const park = lds + (C::NREG - 1) * C::REGION + threadIdx.x;  // the thread's own slots, WG apart
    const int keep = (a.N * E) / (2 * G);  // E/2, E/4 or E/8 for P_c = 1, 2, 4 (store_rows)

    // The group being gathered: its polar block, its first slice, its origin values.
    __amdgpu_buffer_rsrc_t P = polar_rsrc(a.polar + (size_t)(s_begin / Q) * lay.group_elems(), group_bytes);
    int sg = s_begin;
    float dcv[Q];
    auto open_group = [&](int s0) {
        sg = s0;
        P = polar_rsrc(a.polar + (size_t)(s0 / Q) * lay.group_elems(), group_bytes);
        if (lblock == 0) {
            // sums of the slices' V origin terms by W threads, U terms of each
            // slice in flight: one after the other they are the longest chain of a
            // launch (one slice of 256^2 with V = 16384 61 us in all, now 37; 8 222,
            // now 140). One order of additions for every launch of a G.
            constexpr int W = gather_sum_threads(G), U = 8;
            static_assert(W <= C::WG, "a thread per lane of the sum");
            const float* row[Q];
            float acc[Q];
#pragma unroll
            for (int k = 0; k < Q; ++k) {
                row[k] = a.dc + (size_t)min(s0 + k, s_end - 1) * a.V;
                acc[k] = 0.f;
            }
            if (threadIdx.x < W) {
#pragma unroll 1
                for (int i = threadIdx.x; i < V; i += U * W) {
                    float t[Q][U];
#pragma unroll
                    for (int k = 0; k < Q; ++k) {
#pragma unroll
                        for (int u = 0; u < U; ++u) t[k][u] = row[k][min(i + u * W, V - 1)];
                    }
#pragma unroll
                    for (int k = 0; k < Q; ++k) {
#pragma unroll
                        for (int u = 0; u < U; ++u) acc[k] += i + u * W < V ? t[k][u] : 0.f;
                    }
                }
            }
            block_sums<C::WG, Q>(acc, red);
#pragma unroll
            for (int k = 0; k < Q; ++k) dcv[k] = acc[k] * dc_scale;
        }
    };
    // The polar reads of point e, then its values. PIPE: slice 0 of a pair into
    // the thread's parking slot, the other one into nxt[0]; else nxt[slice].
    // points in flight together: those of one pass
    constexpr int D = (E + Q * fft_passes<LOGG, +1, E>() - 1) / (Q * fft_passes<LOGG, +1, E>());
    float4 qa[D][TAPS * Q / 2], qb[D][TAPS * Q / 2];
    float2 nxt[PIPE ? 1 : Q][E];
    // (the stencils are made opaque at each use: otherwise every point's four
    // addresses and both signed weights are formed once and spill)
    auto issue = [&](auto pe) {
        constexpr int e = decltype(pe)::value;
        Stencil& st = pt[e];
        asm volatile("" : "+v"(st.o0), "+v"(st.g));
        const bool wrap = __float_as_uint(st.g) >> 31;
        const bool zero = TENT && ((wide >> e) & 1u);
        if constexpr (TILED) {
            // (j0, m0) and (j0, m0 + 1): 16 bytes apart, or 80 across a tile edge
            const unsigned code = zero ? zcode : st.o0;
            const unsigned oa = BST_IDX((code & kSampleMask) * 16u, group_bytes - 15u, 0);
            const unsigned ob = BST_IDX(oa + (((code >> 29) & 1u) ? 80u : 16u), group_bytes - 15u, 0);
            const unsigned d1 = wrap ? tile_wrap : (((code >> 30) & 1u) ? tile_next : 64u);
            qa[e % D][0] = load16(P, oa);
            qa[e % D][1] = load16(P, ob);
            qb[e % D][0] = load16(P, BST_IDX(oa + d1, group_bytes - 15u, 0));
            qb[e % D][1] = load16(P, BST_IDX(ob + d1, group_bytes - 15u, 0));
        } else {
            [[maybe_unused]] constexpr unsigned kLast = TAPS * kSampleBytes - 1u;  // bytes read past the offset
            const unsigned o0 = BST_IDX(zero ? zoff : st.o0 * kSampleBytes, group_bytes - kLast, 0);
            const unsigned o1 = BST_IDX(o0 + (wrap ? wrap_bytes : row_bytes), group_bytes - kLast, 0);
            load_row<TAPS, Q>(P, o0, qa[e % D]);
            load_row<TAPS, Q>(P, o1, qb[e % D]);
        }
    };
    auto take = [&](auto pe) {
        constexpr int e = decltype(pe)::value;
        Stencil& st = pt[e];
        asm volatile("" : "+v"(st.g), "+v"(st.w1));
        const float g = fabsf(st.g);
        float2 u0[Q], u1[Q], val[Q];
        radial_row<TAPS, Q>(qa[e % D], g, u0);
        radial_row<TAPS, Q>(qb[e % D], g, u1);
#pragma unroll
        for (int k = 0; k < Q; ++k) val[k] = angular(u0[k], u1[k], st.w1, lower_j0<NU>(flips, e, 2 * e >= E));
        if constexpr (TENT) {
            // wide points: the value pre-gathered over their tent of angles
            if ((wide >> e) & 1u) {
#pragma unroll
                for (int k = 0; k < Q; ++k) {
                    const int sk = min(sg + k, a.batch - 1);
                    val[k] = a.patch[(size_t)sk * a.tent_w + BST_IDX(st.o0, (unsigned)a.tent_w, 1)];
                }
            }
        }
        // origin: column 0, row 0 is thread j = 0's first point
        if constexpr (e == 0) {
            if (col == 0 && j == 0) {
#pragma unroll
                for (int k = 0; k < Q; ++k) val[k] = make_float2(dcv[k], 0.f);
            }
        }
        // formed here: left to itself the compiler keeps the reads' registers
        // until the value is used, a whole transform later
        if constexpr (PIPE) {
            if constexpr (Q == 2) park[e * C::WG] = val[0];
            nxt[0][e] = val[Q - 1];
            asm volatile("" : "+v"(nxt[0][e].x), "+v"(nxt[0][e].y));
        } else {
#pragma unroll
            for (int k = 0; k < Q; ++k) {
                nxt[k][e] = val[k];
                asm volatile("" : "+v"(nxt[k][e].x), "+v"(nxt[k][e].y));
            }
        }
    };
    // The next group's points are spread over the passes of this group's
    // transforms: pass r takes the points issued in pass r - 1 and issues its
    // own, their reads spaced out between the pass's butterflies (a burst of
    // reads from all waves at once would stall them in issue).
    constexpr int PASSES = Q * fft_passes<LOGG, +1, E>();
    constexpr int kReads = TAPS * Q;  // read instructions of a point
    auto first_of = [](int r) constexpr { return r * E / PASSES; };
    auto take_pass = [&](auto pr) {
        constexpr int lo = first_of(decltype(pr)::value), hi = first_of(decltype(pr)::value + 1);
        static_for<hi - lo>([&](auto pi) { take(std::integral_constant<int, lo + decltype(pi)::value>{}); });
    };
    auto issue_pass = [&](auto pr) {
        constexpr int lo = first_of(decltype(pr)::value), hi = first_of(decltype(pr)::value + 1);
        static_for<hi - lo>([&](auto pi) { issue(std::integral_constant<int, lo + decltype(pi)::value>{}); });
        static_for<(hi - lo) * kReads>([&](auto) {
            __builtin_amdgcn_sched_group_barrier(0x0020, 1, 0);   // one vector memory read
            __builtin_amdgcn_sched_group_barrier(0x0002, kReadSpacing, 0);  // arithmetic
        });
    };
    auto step = [&](auto pr) {
        constexpr int r = decltype(pr)::value;
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (r > 0) take_pass(std::integral_constant<int, r - 1>{});
        __builtin_amdgcn_sched_barrier(0);
        issue_pass(pr);
    };

    // a group gathered on its own, D points' reads in flight
    auto gather_group = [&]() {
        static_for<D>([&](auto pe) { issue(pe); });
        static_for<E>([&](auto pe) {
            constexpr int e = decltype(pe)::value;
            take(pe);
            if constexpr (e + D < E) issue(std::integral_constant<int, e + D>{});
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    // One group's transforms, with (MORE) the next group's gather between their
    // exchanges. nq: the slices of the group in the batch.
    auto transforms = [&](auto pmore, int s0, int nq) {
        constexpr bool MORE = decltype(pmore)::value;
        float2 cur[Q][E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            if constexpr (C::PARK) cur[0][e] = park[e * C::WG];
            if constexpr (PIPE) {
                cur[Q - 1][e] = nxt[0][e];
            } else {
#pragma unroll
                for (int k = 0; k < Q; ++k) cur[k][e] = nxt[k][e];
            }
        }
        if constexpr (MORE) open_group(s0 + Q);
        static_for<Q>([&](auto pk) {
            constexpr int k = decltype(pk)::value;
            if (!MORE && k >= nq) return;
            // Re-derive the lane's row index for each transform: otherwise every
            // address that depends on it (LDS passes, grid stores) is computed
            // once and held in registers, which spills.
            int jk = j;
            asm volatile("" : "+v"(jk));
            FftTwiddles<LOGG, +1, E, 2> twl = tw;
            twl.pin();
            auto hook = [&](auto ph) {
                if constexpr (MORE) step(std::integral_constant<int, k * (PASSES / Q) + decltype(ph)::value>{});
            };
            fft(cur[k], lds, off, jk, twl, xm, hook);
            if (live) {
                float2* D = a.grid + (size_t)(s0 + k) * a.N * a.GT;
                if (keep == E / 2) store_rows<LOGG, E, E / 2>(cur[k], D, a, jk, col);
                else if (keep == E / 4) store_rows<LOGG, E, E / 4>(cur[k], D, a, jk, col);
                else store_rows<LOGG, E, E / 8>(cur[k], D, a, jk, col);
            }
        });
        if constexpr (MORE) take_pass(std::integral_constant<int, PASSES - 1>{});
    };
    if constexpr (PIPE) {
        // the first group has nothing to hide its reads behind
        open_group(s_begin);
        gather_group();
        int s0 = s_begin;
#pragma unroll 1
        for (; s0 + Q < s_end; s0 += Q) transforms(std::true_type{}, s0, Q);
        transforms(std::false_type{}, s0, s_end - s0);
    } else {
#pragma unroll 1
        for (int s0 = s_begin; s0 < s_end; s0 += Q) {
            open_group(s0);
            gather_group();
            transforms(std::false_type{}, s0, s_end - s0);
        }
    }
}

template <int LOGG, int TAPS, bool PIPE>
using GatherKernelCfg = GatherCfg<LOGG, polar_group(TAPS), gather_threads(1 << LOGG, PIPE), PIPE>;

template <int LOGG, int TAPS, bool NU, bool TENT, bool PIPE>
__global__ void __launch_bounds__((GatherKernelCfg<LOGG, TAPS, PIPE>::WG))
__attribute__((amdgpu_waves_per_eu(GatherKernelCfg<LOGG, TAPS, PIPE>::WAVES, 8))) k_gather_colifft(GatherArgs a) {
    const int s_begin = blockIdx.y * a.slices_per_block;  // a multiple of Q
    gather_body<LOGG, TAPS, NU, TENT, polar_group(TAPS), gather_threads(1 << LOGG, PIPE), PIPE>(
        a, xcd_contiguous(blockIdx.x, gridDim.x), s_begin, min(a.batch, s_begin + a.slices_per_block));
}

// Persistent launch of uneven batches (one slice per group, uniform angles):
// every block walks the work list (slice, column block) in steps of the grid,
// the blocks of one XCD taking contiguous items (the neighbouring columns of
// one slice, which read the same polar lines). Blocks of 512 threads at every
// length (96 uneven sinograms: 3.5 ms, with 256 threads 4.7, with 1024 5.2).
constexpr int kItemsThreads = 512;
template <int LOGG>
using ItemsCfg = GatherCfg<LOGG, 1, kItemsThreads, false>;
template <int LOGG, int TAPS>
__global__ void __launch_bounds__((ItemsCfg<LOGG>::WG))
__attribute__((amdgpu_waves_per_eu(ItemsCfg<LOGG>::WAVES, 8))) k_gather_items(GatherArgs a) {
    const int local = xcd_contiguous(blockIdx.x, gridDim.x);
    for (int base = 0; base < a.n_items; base += gridDim.x) {
        const int it = base + local;
        if (it >= a.n_items) break;
        const int2 w = a.items[it];
        __syncthreads();  // the previous item's LDS reads are done
        gather_body<LOGG, TAPS, false, false, 1, kItemsThreads, false>(a, w.y, w.x, w.x + 1);
    }
}

// Slices per block where the plan leaves it open: as many groups as still fill
// the GPU's 256 compute units at the kernel's waves per SIMD (fewer leave units
// idle: 8 slices of 256^2 in blocks of one group 13.2 us, of four 27.4), so
// that a point's coordinates are formed once for all of them (4 slices of
// 2048^2: blocks of one group 123 us, of two 117; 64 slices: 2923 and, of
// eight, 2053), but no more than 16 slices of pairs and 6 single ones, beyond
// which fewer, longer blocks balance worse (64 cubic slices of 2048^2 at P_c =
// 1: 1100 us with 6, 1227 with 64; 64 of 1024^2: 471 with 16, 528 with 64).
template <class C>
static int auto_slices(int batch) {
    constexpr int kThreads = 256 * 4 * 64 * C::WAVES;
    constexpr int kMost = C::Q == 2 ? 8 : 6;  // groups
    const int groups = (batch + C::Q - 1) / C::Q;
    long long n = (long long)groups * (C::G / 2) * C::T / kThreads;
    n = n < 1 ? 1 : (n > kMost ? kMost : n);
    const int chunks = (int)((groups + n - 1) / n);
    return (groups + chunks - 1) / chunks * C::Q;  // chunks of equal length
}

template <int LOGG, int TAPS, bool NU, bool TENT>
static hipError_t launch_gather_k(const GatherArgs& a0, hipStream_t st) {
    constexpr bool CAN_PIPE = gather_points(1 << LOGG) == 16;
    constexpr int Q = polar_group(TAPS);
    using L = GatherKernelCfg<LOGG, TAPS, false>;
    GatherArgs a = a0;
    if (a.slices_per_block == 0) a.slices_per_block = auto_slices<L>(a.batch);
    const int chunks = (a.batch + a.slices_per_block - 1) / a.slices_per_block;
    if constexpr (CAN_PIPE) {
        // overlapped where a block has a second group to overlap; and at G = 4096, where
        // only its 512 threads hold two columns, for polar spectra that do not stay
        // in the caches, whose lines the two columns share (2 slices of 2048^2 with
        // 16384 projections 247 -> 207 us, 8192 168 -> 136, 4096 78 -> 82; cubic
        // taps, one slice: 181 -> 144, 98 -> 87, 73 -> 67, with 2048 56 -> 58)
        const size_t group = PolarTiles{Q, a.V, a.S}.group_elems() * sizeof(float2);
        const bool spread = LOGG == 12 && group > (Q == 2 ? (size_t)150000000 : (size_t)60000000);
        if ((a.slices_per_block > Q && a.batch > Q) || spread) {
            using C = GatherKernelCfg<LOGG, TAPS, true>;
            hipLaunchKernelGGL((k_gather_colifft<LOGG, TAPS, NU, TENT, true>), dim3((C::G / 2 + C::F - 1) / C::F, chunks),
                               dim3(C::WG), 0, st, a);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((k_gather_colifft<LOGG, TAPS, NU, TENT, false>), dim3((L::G / 2 + L::F - 1) / L::F, chunks),
                       dim3(L::WG), 0, st, a);
    return hipGetLastError();
}

template <int LOGG, int TAPS>
static hipError_t launch_gather_t(const GatherArgs& a, hipStream_t st) {
    if (a.slices_per_block < 0 || a.slices_per_block % polar_group(TAPS) != 0) return hipErrorInvalidValue;
    if (a.tent_cols) {
        // tent rule: uniform angles and linear radial taps only (checked by the plan)
        if constexpr (TAPS == 2) return launch_gather_k<LOGG, TAPS, false, true>(a, st);
        else return hipErrorInvalidValue;
    }
    if (a.uniform) return launch_gather_k<LOGG, TAPS, false, false>(a, st);
    return launch_gather_k<LOGG, TAPS, true, false>(a, st);
}

static_assert(kTentSlices % kPolarSlices == 0, "a tent group spans whole polar groups");

// Tent rule, step 1: the first `rows` radial samples of every angle,
// radius-major with kTentSlices slices interleaved ([group][m][j][slice]), so
// one angular tap of step 2 reads its slices' values as one contiguous 64-byte
// run. A block moves a tile of 32 radii x 8 angles of every slice of its
// group through LDS: reads are 32-sample runs of a polar row, writes are the
// tile's 8 angles x 8 slices of each radius, one contiguous 512-byte run.
// Slices past the batch are written as zeros.
__global__ void __launch_bounds__(256) k_tent_transpose(TentArgs a, int batch) {
    __shared__ float2 tile[kTentSlices][8][33];
    const int grp = blockIdx.z;
    const int m0 = blockIdx.x * 32, j0 = blockIdx.y * 8;
    // reads follow the interleaved polar layout: the Q slices of one sample,
    // then consecutive samples (runs of 4 samples with Q = 2, 32 otherwise)
    constexpr int Q = kPolarSlices, NG = kTentSlices / kPolarSlices;
#pragma unroll
    for (int it = 0; it < 8; ++it) {
        const int idx = it * 256 + threadIdx.x;
        const int k4 = idx % Q, m = (idx / Q) & 31, kh = (idx / (32 * Q)) % NG, j = idx / 256;
        const int k = kh * Q + k4;
        const int s = grp * kTentSlices + k;
        float2 v = make_float2(0.f, 0.f);
        if (s < batch && j0 + j < a.V && m0 + m < a.rows) {
            const PolarTiles lay{Q, a.V, a.S};
            v = a.polar[(size_t)(s / Q) * lay.group_elems() +
                        lay.sample(j0 + j, BST_IDX(a.lead + m0 + m, a.S, 3)) * Q + k4];
        }
        tile[k][j][m] = v;
    }
    __syncthreads();
    float2* Tg = a.trans + (size_t)grp * a.rows * a.V * kTentSlices;
#pragma unroll
    for (int it = 0; it < 8; ++it) {
        const int idx = it * 256 + threadIdx.x;
        const int k = idx & 7, j = (idx >> 3) & 7, m = idx >> 6;
        if (m0 + m < a.rows && j0 + j < a.V)
            Tg[BST_IDX(((size_t)(m0 + m) * a.V + j0 + j) * kTentSlices + k, (size_t)a.rows * a.V * kTentSlices, 4)] =
                tile[k][j][m];
    }
}

// Tent rule, step 2: one thread per chunk of at most kTentChunk angle taps
// of one wide point, for kTentSlices slices. The point (a, b) of the chunk's
// slot comes from the column table; its taps are the angle indices j of the
// period-pi continuation with |q - j| < h, weights (1 - |q - j| / h), on the
// two radial samples m0, m0 + 1 (linear weights); j outside [0, V) reads the
// conjugated image of j mod V, and the lower half-plane conjugates the
// result. Coordinates are formed in FP64 as on the host. Splitting the long
// tap ranges near the origin (over a thousand taps) into chunks keeps every
// thread's loop short.
__device__ __forceinline__ int tent_column(const TentArgs& a, int slot) {
    // the last column whose first slot is <= slot
    int lo = 0, hi = a.ncols - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (a.cols[mid].x <= slot) lo = mid; else hi = mid - 1;
    }
    return lo;
}

__global__ void __launch_bounds__(256) k_tent_chunks(TentArgs a, int batch) {
    // neighbouring chunks read the same angle taps: keep them on one XCD
    const int c = xcd_contiguous(blockIdx.x, gridDim.x) * 256 + threadIdx.x;
    const int s0 = blockIdx.y * kTentSlices;
    if (c >= a.C) return;
    const int ns = min(kTentSlices, batch - s0);
    const int4 ch = a.chunk[c];
    const int col = BST_IDX(tent_column(a, ch.x), a.ncols, 5);
    const int2 tc = a.cols[col];
    const int b = ch.x - tc.x - tc.y;
    const double rho = sqrt((double)col * col + (double)b * b);
    const double phi = atan2((double)b, (double)col);
    const bool lower = phi < 0.0;
    const double q = (lower ? phi + M_PI : phi) * ((double)a.V / M_PI);
    const double h = (double)a.V / (M_PI * rho);
    const double r = rho * a.rscale;
    const int m0 = BST_IDX((int)floor(r), a.rows, 6);
    const float g = (float)(r - (double)m0);
    const float w1r = m0 + 1 < a.rows ? g : 0.f;  // samples past M/2 are zero
    const float inv_h = (float)(1.0 / h);
    // the slice group's radius-major rows m0 and m0 + 1, 8 slices per angle
    const float4* T0 = reinterpret_cast<const float4*>(
        a.trans + ((size_t)blockIdx.y * a.rows + m0) * a.V * kTentSlices);
    const float4* T1 = T0 + (m0 + 1 < a.rows ? (size_t)a.V * (kTentSlices / 2) : 0);
    float ax[kTentSlices], ay[kTentSlices];
#pragma unroll
    for (int k = 0; k < kTentSlices; ++k) ax[k] = ay[k] = 0.f;
    float total = 0.f;
    for (int jc = ch.y; jc <= ch.z; ++jc) {
        const float w = 1.f - fabsf((float)(q - (double)jc)) * inv_h;
        if (w <= 0.f) continue;
        total += w;
        const bool flip = jc < 0 || jc >= a.V;
        const int jj = BST_IDX(jc < 0 ? jc + a.V : (jc >= a.V ? jc - a.V : jc), a.V, 7);
        const float wy = flip ? -w : w;
        float2 v0[kTentSlices], v1[kTentSlices];
#pragma unroll
        for (int k = 0; k < kTentSlices; k += 2) {
            const float4 p0 = T0[(size_t)jj * (kTentSlices / 2) + k / 2];
            const float4 p1 = T1[(size_t)jj * (kTentSlices / 2) + k / 2];
            v0[k] = make_float2(p0.x, p0.y);
            v0[k + 1] = make_float2(p0.z, p0.w);
            v1[k] = make_float2(p1.x, p1.y);
            v1[k + 1] = make_float2(p1.z, p1.w);
        }
#pragma unroll
        for (int k = 0; k < kTentSlices; ++k) {
            const float vx = fmaf(w1r, v1[k].x - v0[k].x, v0[k].x);
            const float vy = fmaf(w1r, v1[k].y - v0[k].y, v0[k].y);
            ax[k] = fmaf(w, vx, ax[k]);
            ay[k] = fmaf(wy, vy, ay[k]);
        }
    }
#pragma unroll
    for (int k = 0; k < kTentSlices; ++k)
        if (k < ns) a.part[(size_t)(s0 + k) * a.C + c] = make_float2(ax[k], lower ? -ay[k] : ay[k]);
    if (blockIdx.y == 0) a.wsum[c] = total;
}

// Tent rule, step 3: each wide point's value is the sum of its chunks'
// partial sums over the sum of their weights (chunks in order).
__global__ void __launch_bounds__(256) k_tent_reduce(TentArgs a) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    const int s = blockIdx.y;
    if (i >= a.W) return;
    const int c1 = a.coff[i + 1];
    float ax = 0.f, ay = 0.f, tot = 0.f;
    for (int c = a.coff[i]; c < c1; ++c) {
        const float2 p = a.part[(size_t)s * a.C + c];
        ax += p.x;
        ay += p.y;
        tot += a.wsum[c];
    }
    const float inv = tot > 0.f ? 1.f / tot : 0.f;
    a.patch[(size_t)s * a.W + i] = make_float2(ax * inv, ay * inv);
}

hipError_t launch_tent(const bst_plan_s& p, const TentArgs& a, int batch, hipStream_t st) {
    (void)p;
    if (a.W <= 0) return hipSuccess;
    const int groups = (batch + kTentSlices - 1) / kTentSlices;
    hipLaunchKernelGGL(k_tent_transpose, dim3((a.rows + 31) / 32, (a.V + 7) / 8, groups), dim3(256), 0, st, a,
                       batch);
    if (a.C > 0)
        hipLaunchKernelGGL(k_tent_chunks, dim3((a.C + 255) / 256, (batch + kTentSlices - 1) / kTentSlices), dim3(256),
                           0, st, a, batch);
    hipLaunchKernelGGL(k_tent_reduce, dim3((a.W + 255) / 256, batch), dim3(256), 0, st, a);
    return hipGetLastError();
}

template <int LOGG>
static hipError_t launch_gather_items_t(const GatherArgs& a, int taps, int blocks, hipStream_t st) {
    using C = ItemsCfg<LOGG>;
    if (taps == 4) hipLaunchKernelGGL((k_gather_items<LOGG, 4>), dim3(blocks), dim3(C::WG), 0, st, a);
    else hipLaunchKernelGGL((k_gather_items<LOGG, 2>), dim3(blocks), dim3(C::WG), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_gather_items(const bst_plan_s& p, const GatherArgs& a, int blocks, hipStream_t st) {
    if (a.tent_cols || !a.Vs) return hipErrorInvalidValue;
    switch (p.logG) {
        case 4: return launch_gather_items_t<4>(a, p.taps, blocks, st);
        case 5: return launch_gather_items_t<5>(a, p.taps, blocks, st);
        case 6: return launch_gather_items_t<6>(a, p.taps, blocks, st);
        case 7: return launch_gather_items_t<7>(a, p.taps, blocks, st);
        case 8: return launch_gather_items_t<8>(a, p.taps, blocks, st);
        case 9: return launch_gather_items_t<9>(a, p.taps, blocks, st);
        case 10: return launch_gather_items_t<10>(a, p.taps, blocks, st);
        case 11: return launch_gather_items_t<11>(a, p.taps, blocks, st);
        case 12: return launch_gather_items_t<12>(a, p.taps, blocks, st);
        case 13: return launch_gather_items_t<13>(a, p.taps, blocks, st);
        default: return hipErrorInvalidValue;
    }
}

template <int LOGG>
static int gather_cols_t() {
    using C = ItemsCfg<LOGG>;
    return (C::G / 2 + C::F - 1) / C::F;
}

int gather_blocks_per_slice(const bst_plan_s& p) {
    switch (p.logG) {
        case 4: return gather_cols_t<4>();
        case 5: return gather_cols_t<5>();
        case 6: return gather_cols_t<6>();
        case 7: return gather_cols_t<7>();
        case 8: return gather_cols_t<8>();
        case 9: return gather_cols_t<9>();
        case 10: return gather_cols_t<10>();
        case 11: return gather_cols_t<11>();
        case 12: return gather_cols_t<12>();
        case 13: return gather_cols_t<13>();
        default: return 0;
    }
}

hipError_t launch_gather_colifft(const bst_plan_s& p, const GatherArgs& a, hipStream_t st) {
    const bool cubic = p.taps == 4;
    switch (p.logG) {
        case 4: return cubic ? launch_gather_t<4, 4>(a, st) : launch_gather_t<4, 2>(a, st);
        case 5: return cubic ? launch_gather_t<5, 4>(a, st) : launch_gather_t<5, 2>(a, st);
        case 6: return cubic ? launch_gather_t<6, 4>(a, st) : launch_gather_t<6, 2>(a, st);
        case 7: return cubic ? launch_gather_t<7, 4>(a, st) : launch_gather_t<7, 2>(a, st);
        case 8: return cubic ? launch_gather_t<8, 4>(a, st) : launch_gather_t<8, 2>(a, st);
        case 9: return cubic ? launch_gather_t<9, 4>(a, st) : launch_gather_t<9, 2>(a, st);
        case 10: return cubic ? launch_gather_t<10, 4>(a, st) : launch_gather_t<10, 2>(a, st);
        case 11: return cubic ? launch_gather_t<11, 4>(a, st) : launch_gather_t<11, 2>(a, st);
        case 12: return cubic ? launch_gather_t<12, 4>(a, st) : launch_gather_t<12, 2>(a, st);
        case 13: return cubic ? launch_gather_t<13, 4>(a, st) : launch_gather_t<13, 2>(a, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace bst

BST_CHECK_MODULE(gather)
