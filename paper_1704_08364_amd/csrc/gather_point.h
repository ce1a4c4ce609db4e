// gather_point.h -- where a Cartesian grid point falls between the polar samples:
// radius index and fraction, and the fraction of the angle step. Plain FP32
// arithmetic whose errors are those of one or two roundings of the result, also
// at indices of a few thousand; host code can run it too.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>

namespace bst {

// An FP64 value as an FP32 one and the rest.
inline float2 split_float(double x) {
    const float hi = (float)x;
    return make_float2(hi, (float)(x - (double)hi));
}
// (cos, sin) of an angle for angle_offset: (cos, its rest, sin, its rest).
inline float4 split_direction(double c, double s) {
    const float2 a = split_float(c), b = split_float(s);
    return make_float4(a.x, a.y, b.x, b.y);
}

// The radius scale P_r / P_c = 2^shift, between 1/4 and 4.
struct RadiusScale {
    int shift;
    float below;    // 2^shift, less more than an approximate root's error
    float inverse;  // 2^-shift
    float down;     // 4^min(shift, 0)
};
inline RadiusScale radius_scale(double rscale) {
    const int shift = std::ilogb(rscale);
    return RadiusScale{shift, (float)(rscale * (1.0 - 0x1p-21)), (float)(1.0 / rscale),
                       shift < 0 ? (float)(rscale * rscale) : 1.f};
}

struct RadialIndex {
    int m;        // floor(r)
    float g;      // r - m
    float ri;     // 2^shift / r to one ulp
    float dinv;   // 1 - r ri 2^-shift
};

// r = sqrt(n) 2^shift, n = a^2 + b^2 (exact, at most 2^25), from ri = 1 / sqrt(n)
// to one ulp. A root q at most 8e-7 r below r gives m = floor(r) or one less, told
// apart by the exact d = r^2 - m^2 (integers after scaling by 4^-shift for
// shift < 0). The fraction g = q - m (exact, as a difference) is off by what q
// is, up to 3e-3; two Newton steps on d = 2 m g + g^2, whose residual is exact
// but for the last place of g^2, leave only the rounding of g: rms 1.3e-8, largest
// 3.0e-8, as from an FP64 root (the quotient (r^2 - m^2) / (r + m) in FP32:
// 2.3e-8 and 1.3e-7).
__host__ __device__ inline __attribute__((always_inline)) RadialIndex radial_index(int n, float ri,
                                                                                   const RadiusScale& s) {
    const int up = s.shift > 0 ? 2 * s.shift : 0, down = s.shift < 0 ? -2 * s.shift : 0;
    RadialIndex p;
    p.ri = ri;
    const float q = (float)n * ri * s.below;
    p.m = (int)q;
#ifdef __HIP_DEVICE_COMPILE__
    const int m2 = (int)__umul24((unsigned)p.m, (unsigned)p.m);
#else
    const int m2 = p.m * p.m;
#endif
    int d = (n << up) - (m2 << down);
    const int next = (2 * p.m + 1) << down;
    if (d >= next) {
        d -= next;
        p.m += 1;
    }
    const float m = (float)p.m, sq = (float)d * s.down, rinv = ri * s.inverse, half = 0.5f * rinv;
    float g = q - m;
    g = fmaf(fmaf(-g, g, fmaf(-2.f * m, g, sq)), half, g);
    g = fmaf(fmaf(-g, g, fmaf(-2.f * m, g, sq)), half, g);
    p.g = fabsf(g);  // 0 may come out as -1e-20
    p.dinv = fmaf(-p.g, rinv, fmaf(-m, rinv, 1.f));
    return p;
}

// Angle from the direction dir (split_direction) to the point (x, y) at p, in
// angle steps: the arcsine of cross / r times V / pi (vpi and the rest of it).
// The cross product keeps the rounding error of the product it subtracts, so its
// error is one rounding of itself however small it is; that of the quotient and
// the series beyond its first term are added last. rms 1.9e-8, largest 9e-8 for
// every V (FP64 products, then FP32: 3.0-4.7e-8 and 2.1e-7). Directions at most
// 1.1 pi / 16 apart: the series to s^9 is exact to FP32 rounding.
__host__ __device__ inline __attribute__((always_inline)) float angle_offset(float x, float y, float4 dir,
                                                                             const RadialIndex& p, float vpi,
                                                                             float vpi_lo) {
    const float w = x * dir.z;
    const float cross = fmaf(y, dir.x, -w);
    const float rest = fmaf(-x, dir.z, w) + fmaf(y, dir.y, -(x * dir.w));
    const float s = cross * p.ri, s2 = s * s;
    const float ds = fmaf(rest, p.ri, fmaf(cross, p.ri, -s));
    float q = fmaf(s2, 0.0303819444f, 0.0446428571f);
    q = fmaf(s2, q, 0.075f);
    q = fmaf(s2, q, 0.1666666667f);
    const float tail = fmaf(s2 * s, q, fmaf(s, p.dinv, ds));
    return fmaf(s, vpi, fmaf(s, vpi_lo, tail * vpi));
}

}  // namespace bst
