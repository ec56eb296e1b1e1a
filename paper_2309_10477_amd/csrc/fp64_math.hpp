// Double-precision elementary functions of the path kernels.
//
// A Milstein step in FP64 is bound by VALU issue (every FP64 instruction takes
// a SIMD's quad-cycle), and most of its instructions were the math library's
// log, sincospi, sqrt and exp2, which carry range reductions, scalings and
// special cases that the arguments here never need: uniforms are odd multiples
// of 2^-24, variances are >= 0 and far from the ends of the exponent range.
// With these forms a step of the fused arithmetic-Asian kernel issues 237
// instead of 430 VALU instructions and one of the scenario-split European
// kernel 40 instead of 65: a daily Asian put with fused bumps, 200 003 paths x
// 251 steps, 882 -> 495 us per call; a 64-option FP64 batch 1.95x.
// Each function's error in ulps is checked on the CPU (tests/host/fp64_math_test.cpp):
// the Box-Muller radius 0.37 rms (the library's 0.33), cosine and sine 0.34 of
// 2^-53, exponentials 0.30 (at most 0.89), square root and reciprocal correctly
// rounded.  The averages of 252-step paths, measured against an 80-bit simulation,
// were off by 4.4e-16 rms before and after (base parameters); by 6.4e-15 before and
// 7.6e-15 after, with the same median, on a long Feller-violating set.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fp64_tables.hpp"

namespace heston {

// The tables in LDS (8 KiB): a wave's 64 lanes read 64 unrelated rows, which
// LDS serves in a few cycles more than one row and the vector cache would
// serve a few lanes per cycle.
struct Fp64Tables {
    double log[256][2];
    double trig[256][2];
};
__device__ __forceinline__ Fp64Tables &fp64_tables()
{
    __shared__ Fp64Tables t;
    return t;
}
// Every thread of the block calls it before the first use (BLOCK a power of two).
template <int BLOCK_SIZE> __device__ __forceinline__ void load_fp64_tables()
{
    Fp64Tables &t = fp64_tables();
    for (int i = threadIdx.x; i < 256; i += BLOCK_SIZE) {
        t.log[i][0] = LOG_TABLE[i][0];
        t.log[i][1] = LOG_TABLE[i][1];
        t.trig[i][0] = TRIG_TABLE[i][0];
        t.trig[i][1] = TRIG_TABLE[i][1];
    }
    __syncthreads();
}

// -2 ln(d 2^-shift) of a normal d > 0: d = z 2^k with z in [0.70801, 1.41602),
// and the value is (shift - k) 2 ln 2 - 2 ln c - 2 ln(1 + r), r = z / c - 1,
// |r| < 2^-9, the last by its series through r^6 (truncation below 2^-64.8, or
// 2^-55.8 relative to r).
__device__ __forceinline__ double neg2_log(double d, int shift)
{
    const int t = __double2hiint(d) - (int)LOG_OFFSET;
    const double *row = fp64_tables().log[(t >> 12) & 255];
    const double z = __hiloint2double((t & 0xFFFFF) + (int)LOG_OFFSET, __double2loint(d));
    const double r = fma(z, row[0], -1.0);
    const double hi = fma((double)(shift - (t >> 20)), 1.38629436111989061883, row[1]);
    double p = fma(r, 1.0 / 3.0, -0.4);
    p = fma(r, p, 0.5);
    p = fma(r, p, -2.0 / 3.0);
    p = fma(r, p, 1.0);
    p = fma(r, p, -2.0);
    return fma(r, p, hi);
}
// -2 ln u of the uniform u = ((w >> 9) + 1/2) 2^-23 of a random word: u 2^24 is
// the odd integer (w >> 8) | 1, exact in double.
__device__ __forceinline__ double neg2_log_uniform(uint32_t w)
{
    return neg2_log((double)((w >> 8) | 1u), 24);
}

// (C + i S) e^{i d} for a table angle (C, S) and |d| <= pi / 256: the addition
// theorems with the series of sin d and cos d - 1 (truncations below 2^-75 and 2^-66).
__device__ __forceinline__ void turn(double C, double S, double d, double &c, double &s)
{
    const double q = d * d;
    double sp = fma(q, -1.0 / 5040.0, 1.0 / 120.0);
    sp = fma(q, sp, -1.0 / 6.0);
    const double sd = fma(d * q, sp, d);
    double cp = fma(q, -1.0 / 720.0, 1.0 / 24.0);
    cp = fma(q, cp, -0.5);
    const double cd = q * cp; // cos d - 1
    c = C + fma(C, cd, -(S * sd));
    s = S + fma(S, cd, C * sd);
}

// cos and sin of 2 pi u, u the uniform of a random word, from the nearest of
// the 256 table angles.
__device__ __forceinline__ void cos_sin_uniform(uint32_t w, double &c, double &s)
{
    const double *row = fp64_tables().trig[(w + 0x800000u) >> 24];
    const double d = fma((double)((int32_t)(w << 8) >> 17), 0x1.921fb54442d18p-21, 0x1.921fb54442d18p-22);
    turn(row[0], row[1], d, c, s);
}

// cos and sin of x, |x| below about 1e6 (pi / 128 in two parts).
__device__ __forceinline__ void cos_sin(double x, double &c, double &s)
{
    const double n = rint(x * 0x1.45f306dc9c883p+5);
    const double d = fma(-n, 0x1.1a62633145c07p-60, fma(-n, 0x1.921fb54442d18p-6, x));
    const double *row = fp64_tables().trig[(uint32_t)(int)n & 255u];
    turn(row[0], row[1], d, c, s);
}

// sqrt(x) for x >= 0 (exactly 0 at 0): from the hardware's reciprocal square
// root (2^-25), one Newton step and one correction by the remainder x - g^2.
// Correctly rounded on 2^21 arguments, as the library's form, which adds
// scalings for the ends of the exponent range and selects for special cases;
// the floor under the reciprocal keeps it finite at 0.
__device__ __forceinline__ double sqrt_nonneg(double x)
{
    const double y = __builtin_amdgcn_rsq(fmax(x, 0x1p-1000));
    double g = x * y;
    const double h = 0.5 * y;
    g = fma(g, fma(-h, g, 0.5), g);
    return fma(fma(-g, g, x), h, g);
}

// 1 / x and 1 / sqrt(x) for normal x > 0 in the middle of the exponent range:
// the hardware's estimates (2^-25) refined by two Newton steps (0.500 ulp) and
// one third-order step (0.99 ulp).
__device__ __forceinline__ double rcp_pos(double x)
{
    double y = __builtin_amdgcn_rcp(x);
    y = fma(y, fma(-x, y, 1.0), y);
    return fma(y, fma(-x, y, 1.0), y);
}
__device__ __forceinline__ double rsqrt_pos(double x)
{
    const double y = __builtin_amdgcn_rsq(x), e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}

// 2^y: y = n + f, |f| <= 1/2, and 2^f = 1 + f q(f), q of degree 10 (near-minimax
// over [-1/2, 1/2], 2.0e-17); v_ldexp saturates to 0 and infinity by itself.
__device__ __forceinline__ double exp2_plain(double y)
{
    const double n = rint(y), f = y - n;
    double q = 0x1.e9d3fe3952179p-32;
    q = fma(f, q, 0x1.e6063f7217bc6p-28);
    q = fma(f, q, 0x1.b524fae627834p-24);
    q = fma(f, q, 0x1.62bfd47773353p-20);
    q = fma(f, q, 0x1.ffcbfc670dcd4p-17);
    q = fma(f, q, 0x1.430913096fd9fp-13);
    q = fma(f, q, 0x1.5d87fe78a5276p-10);
    q = fma(f, q, 0x1.3b2ab6fba1ddap-7);
    q = fma(f, q, 0x1.c6b08d704a0c2p-5);
    q = fma(f, q, 0x1.ebfbdff82c598p-3);
    q = fma(f, q, 0x1.62e42fefa39efp-1);
    return __builtin_amdgcn_ldexp(fma(f, q, 1.0), (int)n);
}

// e^x: x = n ln 2 + f with ln 2 in two parts, e^f = 1 + f q(f), q of degree 10
// (near-minimax over |f| <= ln 2 / 2, 9.8e-18).  For |x| up to 1e40: f is of the
// order of x's last place there, and its eleventh power overflows beyond.
__device__ __forceinline__ double exp_plain(double x)
{
    const double n = rint(x * 0x1.71547652b82fep+0);
    const double f = fma(-n, 0x1.a39ef35793c76p-33, fma(-n, 0x1.62e42fee00000p-1, x));
    double q = 0x1.af4ddda1c08cdp-26;
    q = fma(f, q, 0x1.28a2c0bee04a5p-22);
    q = fma(f, q, 0x1.71de0237484cdp-19);
    q = fma(f, q, 0x1.a019a66a5f0b6p-16);
    q = fma(f, q, 0x1.a01a01abe6323p-13);
    q = fma(f, q, 0x1.6c16c17f43acbp-10);
    q = fma(f, q, 0x1.11111111100dfp-7);
    q = fma(f, q, 0x1.55555555520afp-5);
    q = fma(f, q, 0x1.5555555555557p-3);
    q = fma(f, q, 0x1.0000000000005p-1);
    q = fma(f, q, 1.0);
    return __builtin_amdgcn_ldexp(fma(f, q, 1.0), (int)n);
}

// e^x for any x below 1e40, 0 far below: x is cut off where e^x is 0 (a path's
// log-price falls below -1e40 with an initial variance of that order).  NaN stays.
// The cut takes 2% of the FP64 Asian adjoint's forward pass.
__device__ __forceinline__ double exp_low(double x) { return exp_plain(x < -1100.0 ? -1100.0 : x); }

// ln(x) of a normal x > 0.
__device__ __forceinline__ double log_pos(double x) { return -0.5 * neg2_log(x, 0); }

// The argument of x + i y, (x, y) away from 0 and the ends of single precision's
// range: a single-precision estimate (7e-4) picks the nearest table angle n pi / 128;
// the rest is atan of the turned vector's slope, |slope| < 0.0133, by its
// series (truncation below 2^-59).
__device__ __forceinline__ double angle(double x, double y)
{
    const float xf = (float)x, yf = (float)y, ax = fabsf(xf), ay = fabsf(yf);
    const float t = fminf(ax, ay) * __builtin_amdgcn_rcpf(fmaxf(ax, ay)), t2 = t * t;
    float a = t * (0.99535f + t2 * (-0.28869f + t2 * 0.07934f));
    a = ay > ax ? 1.57079633f - a : a;
    a = xf < 0.0f ? 3.14159265f - a : a;
    const float nf = rintf(copysignf(a, yf) * 40.7436654f);
    const double *row = fp64_tables().trig[(uint32_t)(int)nf & 255u];
    const double C = row[0], S = row[1];
    const double d = fma(y, C, -(x * S)) * rcp_pos(fma(x, C, y * S)), q = d * d;
    double p = fma(q, -1.0 / 7.0, 0.2);
    p = fma(q, p, -1.0 / 3.0);
    return fma((double)nf, 0x1.921fb54442d18p-6, fma(d * q, p, d));
}
// The same for any normal (x, y) away from 0, first scaled to |x| + |y| = 1.
__device__ __forceinline__ double angle_scaled(double x, double y)
{
    const double f = rcp_pos(fabs(x) + fabs(y));
    return angle(x * f, y * f);
}

} // namespace heston
