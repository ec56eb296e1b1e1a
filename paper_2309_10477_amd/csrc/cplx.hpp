// Double-precision complex arithmetic for device code (the semi-analytic
// geometric price and the exact sampler's characteristic function): plain
// struct.
#pragma once

#include <hip/hip_runtime.h>

namespace heston {

struct Cx {
    double re, im;
};
__device__ __forceinline__ Cx operator+(Cx a, Cx b) { return {a.re + b.re, a.im + b.im}; }
__device__ __forceinline__ Cx operator-(Cx a, Cx b) { return {a.re - b.re, a.im - b.im}; }
__device__ __forceinline__ Cx operator*(Cx a, Cx b)
{
    return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
__device__ __forceinline__ Cx operator*(Cx a, double s) { return {a.re * s, a.im * s}; }
// Smith's division (no overflow of |b|^2 for large operands), two real
// divisions.
__device__ __forceinline__ Cx operator/(Cx a, Cx b)
{
    if (fabs(b.re) >= fabs(b.im)) {
        const double t = b.im / b.re, inv = 1.0 / (b.re + b.im * t);
        return {(a.re + a.im * t) * inv, (a.im - a.re * t) * inv};
    }
    const double t = b.re / b.im, inv = 1.0 / (b.re * t + b.im);
    return {(a.re * t + a.im) * inv, (a.im * t - a.re) * inv};
}
__device__ __forceinline__ Cx cexp(Cx z)
{
    double s, c;
    sincos(z.im, &s, &c);
    const double e = exp(z.re);
    return {e * c, e * s};
}
__device__ __forceinline__ Cx operator*(double s, Cx a) { return {a.re * s, a.im * s}; }
__device__ __forceinline__ Cx operator-(Cx a) { return {-a.re, -a.im}; }
__device__ __forceinline__ double cabs(Cx z) { return hypot(z.re, z.im); }

} // namespace heston
