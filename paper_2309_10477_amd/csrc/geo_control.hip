// Semi-analytic price of the geometric-average Asian option under Heston, on
// the device: the expectation of the control in the arithmetic-Asian
// control-variate estimator.
//
// ln G = (1/n) sum_i ln S(t_i) is a linear functional of the affine state
// (ln S, V), so E[exp(u ln G)] = exp(u ln S0 + A + B v0).  Going backwards
// from the last fixing date, the coefficient a of ln S is u/n times the number
// of dates still ahead, and over each gap between dates (A, B) follow the
// Riccati equations of the Heston model with that a, whose solution is closed
// form: with c2 = sigma^2/2, c1 = rho sigma a - kappa, c0 = (a^2 - a)/2 and the
// roots r_- (attracting) and r_+ of c2 x^2 + c1 x + c0,
//   B(tau) = (r_- - r_+ g e^{-d tau}) / (1 - g e^{-d tau}),  g = (B0 - r_-)/(B0 - r_+),
//   A(tau) = A0 + r a tau + kappa theta (r_- tau - ln((1 - g e^{-d tau})/(1 - g)) / c2).
// The call price is e^{-rT} ((E[G] - K)/2 + (1/pi) int_0^inf Re[e^{-iv ln K}
// (M(1+iv) - K M(iv)) / (iv)] dv) (Gil-Pelaez), integrated by 16-point
// Gauss-Legendre on panels of width GEO_PANEL_WIDTH up to a power of two v_max
// where the integrand's modulus bound is below 1e-15 (E[G] + K).
//
// A gap's step is linear-fractional in B, so with B = x / y it is a 2x2 matrix
// on (x, y), N = M / (r_- - r_+), whose entries depend on a and tau alone; N is
// scaled so that the logarithm's argument is y' / y.  A block takes eight
// transforms (32 in long ranges), its threads shared evenly, and goes through the
// gaps 64 (16) at a time: all threads form the matrices (square roots,
// exponentials, divisions), one thread per transform multiplies the vectors
// through them, and all threads take the arguments of y' / y (the moduli
// telescope).  One thread per transform doing all of it in order was a chain of
// 252 steps of some 6000 cycles each, 585 us for a daily Asian on 9 blocks,
// longer than the 2^18 paths beside it; the chain is now sixteen FMAs per step,
// the kernel takes about 50 us beside them and the call 226 instead of 627 us.
// Against an 80-bit evaluation the price's error is 1e-15 to 1e-12 relative,
// smaller than the serial form's on 25 of 35 parameter and date sets.
// The first pass integrates over [0, g.v_max] (a range the host sizes from
// the variance of ln G) in one node launch that also evaluates the bound at
// its end; only if that bound is not small does the caller run the search: a
// bound kernel at v = 2^k, then nodes up to the first 2^k whose bound is small
// (a fixed grid whose blocks beyond it only write a zero partial).  A finish
// kernel sums the block partials in a fixed order.
#include <hip/hip_runtime.h>

#include <cmath>

#include "cplx.hpp"
#include "device_math.hpp"
#include "internal.hpp"

namespace heston {
namespace {

constexpr int GEO_MAX_LOG2_RANGE = 14; // v_max <= 2^14
// Panel width: the integrand varies on the scale of 1 / sd(ln G) and is
// analytic in a strip about the real axis, so 16 nodes per 4 units resolve
// it to rounding (checked against adaptive quadrature: 1e-13 relative up to
// width 8 on the tested parameter sets).
constexpr uint32_t GEO_PANEL_WIDTH = 4;
static_assert(GEO_MAX_LOG2_RANGE < GEO_BOUND_POINTS, "bound table too short");
// Transforms per block, whose threads they share evenly.
constexpr uint32_t GEO_SLOTS = 8, GEO_SLOTS_MANY = 32;
constexpr uint32_t GEO_SHORT_RANGE = 1024; // up to it GEO_SLOTS: see many_slots
constexpr uint32_t GEO_MAX_NODES = 2u * (16u << GEO_MAX_LOG2_RANGE) / GEO_PANEL_WIDTH; // x 2 transforms
constexpr uint32_t GEO_CELLS = 512;            // gaps per round of a block, over its transforms
constexpr uint32_t GEO_RESCALE = 8;            // steps between rescalings of (x, y), unrolled
constexpr double GEO_TOL = 1e-15;

__device__ __forceinline__ double fix_time(const GeoControl &g, uint32_t i)
{
    return (g.steps ? (double)g.steps[i] : (double)(i + 1)) * g.dt;
}

template <uint32_t SLOTS> struct GeoShared {
    static constexpr uint32_t LANES = BLOCK / SLOTS, CHUNK = GEO_CELLS / SLOTS;
    static_assert(CHUNK % GEO_RESCALE == 0 && LANES >= GEO_RESCALE, "whole groups of steps");
    static_assert(LANES <= 32 && (LANES & (LANES - 1)) == 0, "a transform's threads within half a wave");
    Cx n[SLOTS][CHUNK][4];              // N of each gap: (11, 12, 21, 22)
    Cx y[SLOTS][CHUNK + 1];             // y before the chunk and after each of its gaps
    Cx end[SLOTS];                      // x / y and, in `log_y`, ln |y| of the last gap
    double log_y[SLOTS];
    double red[SLOTS];
};

// Principal square root (non-negative real part) of z away from the ends of
// the exponent range.
__device__ __forceinline__ Cx lean_csqrt(Cx z)
{
    const double m = sqrt_nonneg(z.re * z.re + z.im * z.im);
    const double t = sqrt_nonneg(0.5 * (m + fabs(z.re)));
    const double o = t > 0.0 ? 0.5 * z.im * rcp_pos(t) : 0.0;
    return z.re >= 0.0 ? Cx{t, o} : Cx{fabs(o), copysign(t, z.im)};
}

// Sum over a transform's threads.
template <uint32_t LANES> __device__ __forceinline__ double slot_sum(double v)
{
#pragma unroll
    for (uint32_t off = LANES / 2; off > 0; off >>= 1)
        v += __shfl_xor(v, off, LANES);
    return v;
}

// Exponent of E[exp(u ln G)]: u ln S0 + A + B v0, for the transform of the
// thread's slot; every thread of the block calls it.
template <uint32_t SLOTS> __device__ Cx log_transform(const GeoControl &g, Cx u, GeoShared<SLOTS> &sh)
{
    constexpr uint32_t LANES = GeoShared<SLOTS>::LANES, CHUNK = GeoShared<SLOTS>::CHUNK;
    const uint32_t slot = threadIdx.x / LANES, lane = threadIdx.x % LANES;
    const Cx w = u * (1.0 / (double)g.n_fix);
    const double c2 = 0.5 * g.sigma * g.sigma, h = 0.5 / c2;
    const Cx one{1.0, 0.0};
    double ar = 0.0, ai = 0.0, turn = 0.0; // this thread's share of A without the logarithms, of arg y
    Cx x{0.0, 0.0}, y = one;               // threads 0 .. SLOTS - 1: slot threadIdx.x
    double scale = 0.0;                    // powers of two taken out of (x, y)
    for (uint32_t base = 0; base < g.n_fix; base += CHUNK) {
        const uint32_t len = min(CHUNK, g.n_fix - base);
        for (uint32_t i = lane; i < len; i += LANES) {
            const uint32_t k = g.n_fix - 1 - (base + i); // from the last date to the first
            const double tau = fix_time(g, k) - (k ? fix_time(g, k - 1) : 0.0);
            const Cx a = w * (double)(g.n_fix - k);
            const Cx c1 = a * (g.rho * g.sigma) - Cx{g.kappa, 0.0};
            const Cx c0 = (a * a - a) * 0.5;
            const Cx d = lean_csqrt(c1 * c1 - c0 * (4.0 * c2));
            const Cx rm = (-c1 - d) * h, rp = (d - c1) * h;
            double ec, es;
            cos_sin(-tau * d.im, ec, es);
            const double em = exp_low(-tau * d.re);
            const Cx e{em * ec, em * es};
            const Cx diff = rm - rp;
            const double n2 = rcp_pos(diff.re * diff.re + diff.im * diff.im);
            const Cx inv{diff.re * n2, -diff.im * n2};
            sh.n[slot][i][0] = (rm - rp * e) * inv;
            sh.n[slot][i][1] = rm * rp * (e - one) * inv;
            sh.n[slot][i][2] = (one - e) * inv;
            sh.n[slot][i][3] = (rm * e - rp) * inv;
            ar += tau * (g.r * a.re + g.kappa * g.theta * rm.re);
            ai += tau * (g.r * a.im + g.kappa * g.theta * rm.im);
        }
        // the last group of steps is filled up with identities
        if (len + lane < (len + GEO_RESCALE - 1) / GEO_RESCALE * GEO_RESCALE) {
            sh.n[slot][len + lane][0] = sh.n[slot][len + lane][3] = one;
            sh.n[slot][len + lane][1] = sh.n[slot][len + lane][2] = Cx{0.0, 0.0};
        }
        __syncthreads();
        if (threadIdx.x < SLOTS) {
            const Cx(*n)[4] = sh.n[threadIdx.x];
            sh.y[threadIdx.x][0] = y;
            for (uint32_t i = 0; i < len; i += GEO_RESCALE) {
#pragma unroll
                for (uint32_t e = 0; e < GEO_RESCALE; ++e) {
                    const Cx xn = n[i + e][0] * x + n[i + e][1] * y;
                    y = n[i + e][2] * x + n[i + e][3] * y;
                    x = xn;
                    sh.y[threadIdx.x][i + e + 1] = y;
                }
                const int ex = ilogb(fabs(y.re) + fabs(y.im));
                x = Cx{ldexp(x.re, -ex), ldexp(x.im, -ex)};
                y = Cx{ldexp(y.re, -ex), ldexp(y.im, -ex)};
                scale += ex;
            }
            if (base + len == g.n_fix) {
                sh.end[threadIdx.x] = x / y;
                sh.log_y[threadIdx.x] = log(cabs(y)) + scale * 0.69314718055994530942;
            }
        }
        __syncthreads();
        for (uint32_t i = lane; i < len; i += LANES) {
            const Cx p = sh.y[slot][i], q = sh.y[slot][i + 1];
            turn += angle_scaled(q.re * p.re + q.im * p.im, q.im * p.re - q.re * p.im);
        }
        __syncthreads(); // the chunk is read before the next one overwrites it
    }
    const double f = g.kappa * g.theta / c2;
    const Cx A{slot_sum<LANES>(ar) - f * sh.log_y[slot], slot_sum<LANES>(ai) - f * slot_sum<LANES>(turn)};
    return u * g.lnS0 + A + sh.end[slot] * g.v0;
}

// Part `which` of the Gil-Pelaez integrand at v: which 0 gives
// Im(e^{-iv ln K} M(1+iv)) / v, which 1 gives -K Im(e^{-iv ln K} M(iv)) / v.
// (lt: the transform's exponent.)
__device__ double integrand_part(const GeoControl &g, Cx lt, double v, int which)
{
    const Cx m = cexp(lt - Cx{0.0, v * g.lnK});
    return (which ? -g.K : 1.0) * m.im / v;
}

// Modulus bound of one part: |M(u)| (times K for part 1) / v.
__device__ double bound_part(const GeoControl &g, Cx lt, double v, int which)
{
    return (which ? g.K : 1.0) * exp(lt.re) / v;
}

// Slot numbers 2 k + which: the bounds at v = 2^k; then E[G].
template <uint32_t SLOTS>
__global__ __launch_bounds__(BLOCK) void geo_bound_kernel(const GeoControl g, double *bound,
                                                          double *out)
{
    __shared__ GeoShared<SLOTS> sh;
    constexpr uint32_t LANES = GeoShared<SLOTS>::LANES;
    load_fp64_tables<BLOCK>();
    const uint32_t t = blockIdx.x * SLOTS + threadIdx.x / LANES;
    const bool is_bound = t < 2 * GEO_BOUND_POINTS;
    const double v = is_bound ? ldexp(1.0, (int)(t >> 1)) : 0.0;
    const int which = is_bound ? (int)(t & 1) : 0;
    const Cx lt = log_transform<SLOTS>(g, Cx{which ? 0.0 : 1.0, v}, sh);
    if (threadIdx.x % LANES != 0)
        return;
    if (is_bound)
        bound[t] = bound_part(g, lt, v, which);
    else if (t == 2 * GEO_BOUND_POINTS)
        out[0] = exp(lt.re); // E[G]
}

// Range of the integral: the first 2^k (k <= GEO_MAX_LOG2_RANGE) whose bound
// is below tolerance, or 0 if none is.
__device__ uint32_t range_from(const double *bound, double EG, double K)
{
    const double tol = GEO_TOL * (EG + K);
    for (int k = 0; k <= GEO_MAX_LOG2_RANGE; ++k)
        if (bound[2 * k] + bound[2 * k + 1] <= tol)
            return 1u << k;
    return 0u;
}

// Gauss-Legendre nodes of the integral over [0, range], two transforms per
// node, from block `block0` of the whole range on; a later launch (block0 > 0)
// adds to the partials of the one before.  With a `fixed` range the three slots
// after the nodes evaluate the modulus bound at v = fixed (out[1], out[2]) and
// E[G] (out[0]); otherwise the range comes from the bound table of
// geo_bound_kernel.
template <uint32_t SLOTS>
__global__ __launch_bounds__(BLOCK) void geo_node_kernel(const GeoControl g, uint32_t fixed,
                                                         uint32_t block0, const double *bound,
                                                         double *out, double *partials)
{
    __shared__ GeoShared<SLOTS> sh;
    constexpr uint32_t LANES = GeoShared<SLOTS>::LANES;
    const uint32_t range = fixed ? fixed : range_from(bound, out[0], g.K);
    const uint32_t width = range < GEO_PANEL_WIDTH ? range : GEO_PANEL_WIDTH;
    const uint32_t panels = width ? range / width : 0u;
    const uint32_t first = (block0 + blockIdx.x) * SLOTS, t = first + threadIdx.x / LANES;
    const uint32_t n_nodes = 32u * panels;
    if (first >= n_nodes + (fixed ? 3u : 0u)) { // nothing for the whole block
        if (threadIdx.x == 0 && block0 == 0)
            partials[blockIdx.x] = 0.0;
        return;
    }
    load_fp64_tables<BLOCK>();
    const bool is_node = t < n_nodes, is_bound = !is_node && t < n_nodes + 2;
    const int which = is_node || is_bound ? (int)(t & 1) : 0;
    double v = 0.0, weight = 0.0;
    if (is_node) {
        const uint32_t node = t >> 1, panel = node >> 4, j = node & 15;
        const double x = j < 8 ? -g.gl_x[7 - j] : g.gl_x[j - 8];
        const double w = j < 8 ? g.gl_w[7 - j] : g.gl_w[j - 8];
        v = ((double)panel + 0.5 + 0.5 * x) * (double)width;
        weight = 0.5 * (double)width * w;
    } else if (is_bound) {
        v = (double)fixed;
    }
    const Cx lt = log_transform<SLOTS>(g, Cx{which ? 0.0 : 1.0, v}, sh);
    if (threadIdx.x % LANES == 0) {
        sh.red[threadIdx.x / LANES] = is_node ? weight * integrand_part(g, lt, v, which) : 0.0;
        if (fixed && is_bound)
            out[1 + which] = bound_part(g, lt, v, which);
        else if (fixed && t == n_nodes + 2)
            out[0] = exp(lt.re); // E[G]
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double b = 0.0;
#pragma unroll
        for (uint32_t k = 0; k < SLOTS; ++k)
            b += sh.red[k];
        partials[blockIdx.x] = block0 ? partials[blockIdx.x] + b : b;
    }
}

__global__ __launch_bounds__(BLOCK) void geo_finish_kernel(const GeoControl g, uint32_t fixed,
                                                           uint32_t n_blocks, const double *bound,
                                                           const double *partials,
                                                           const double *out, double *prices)
{
    __shared__ double red[BLOCK];
    double s = 0.0;
    for (uint32_t b = threadIdx.x; b < n_blocks; b += BLOCK)
        s += partials[b];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int h = BLOCK / 2; h > 0; h >>= 1) {
        if (threadIdx.x < (unsigned)h)
            red[threadIdx.x] += red[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double EG = out[0], I = red[0];
        const double D = exp(-g.r * g.T);
        const bool ok = fixed ? out[1] + out[2] <= GEO_TOL * (EG + g.K)
                              : range_from(bound, EG, g.K) != 0u;
        const double call = D * (0.5 * (EG - g.K) + I / M_PI);
        const double nan = __builtin_nan("");
        prices[0] = ok ? call : nan;
        prices[1] = ok ? call - D * (EG - g.K) : nan;
    }
}

} // namespace

// A range up to 1024 takes eight transforms per block: its blocks do not fill the
// device, and more threads per transform shorten each (252 dates, range 1024: 121
// us a call of 2000 paths, with 32 per block 138).  Beyond it the blocks queue, and
// 32 per block run the serial chains of four times as many transforms in the same
// instructions (range 2048: 191 -> 179 us, 246 -> 186 beside 2^18 paths; 4096: 337 ->
// 287; twelve dates, searched range: 173 -> 109).
static bool many_slots(const GeoControl &g) { return g.v_max > GEO_SHORT_RANGE; }
static uint32_t fixed_blocks(const GeoControl &g)
{
    const uint32_t slots = many_slots(g) ? GEO_SLOTS_MANY : GEO_SLOTS;
    return (32u * (g.v_max / GEO_PANEL_WIDTH) + 3u + slots - 1) / slots;
}
static_assert(32u * GEO_SHORT_RANGE / GEO_PANEL_WIDTH / GEO_SLOTS < GEO_NODE_BLOCKS &&
                  32u * GEO_MAX_FIXED_RANGE / GEO_PANEL_WIDTH / GEO_SLOTS_MANY < GEO_NODE_BLOCKS,
              "fixed ranges within the partials buffer");

hipError_t launch_geo_nodes_fixed(const GeoControl &g, double *partials, double *buf,
                                  hipStream_t stream)
{
    if (g.v_max < GEO_PANEL_WIDTH || g.v_max > GEO_MAX_FIXED_RANGE || g.v_max % GEO_PANEL_WIDTH)
        return hipErrorInvalidValue;
    const dim3 grid(fixed_blocks(g));
    if (many_slots(g))
        hipLaunchKernelGGL(geo_node_kernel<GEO_SLOTS_MANY>, grid, dim3(BLOCK), 0, stream, g, g.v_max,
                           0u, (const double *)buf, buf + GEO_OUT, partials);
    else
        hipLaunchKernelGGL(geo_node_kernel<GEO_SLOTS>, grid, dim3(BLOCK), 0, stream, g, g.v_max, 0u,
                           (const double *)buf, buf + GEO_OUT, partials);
    return hipGetLastError();
}

hipError_t launch_geo_finish_fixed(const GeoControl &g, double *partials, double *buf,
                                   double *prices, hipStream_t stream)
{
    hipLaunchKernelGGL(geo_finish_kernel, dim3(1), dim3(BLOCK), 0, stream, g, g.v_max,
                       fixed_blocks(g), (const double *)buf, (const double *)partials,
                       buf + GEO_OUT, prices);
    return hipGetLastError();
}

hipError_t launch_geo_price_search(const GeoControl &g, double *partials, double *buf,
                                   double *prices, hipStream_t stream)
{
    constexpr uint32_t SLOTS = GEO_SLOTS_MANY;
    hipLaunchKernelGGL(geo_bound_kernel<SLOTS>, dim3(2 * GEO_BOUND_POINTS / SLOTS + 1), dim3(BLOCK),
                       0, stream, g, buf, buf + GEO_OUT);
    // (all but the first launch exit at once up to a range of 8192)
    for (uint32_t b = 0; b < GEO_MAX_NODES / SLOTS; b += GEO_NODE_BLOCKS)
        hipLaunchKernelGGL(geo_node_kernel<SLOTS>, dim3(GEO_NODE_BLOCKS), dim3(BLOCK), 0, stream, g,
                           0u, b, (const double *)buf, buf + GEO_OUT, partials);
    hipLaunchKernelGGL(geo_finish_kernel, dim3(1), dim3(BLOCK), 0, stream, g, 0u, GEO_NODE_BLOCKS,
                       (const double *)buf, (const double *)partials, buf + GEO_OUT, prices);
    return hipGetLastError();
}

} // namespace heston
