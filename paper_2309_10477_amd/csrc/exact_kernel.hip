// Exact simulation of the Heston model (paper: algorithm "Broadie and Kaya
// exact simulation algorithm", section "Heston Model Exact simulation", and
// the sections on its two bottlenecks), FP64, one path per 16 lanes at a time.
//
// Step of length D from (x = ln S/S0, V_u):
//  1. V_t = c X, X non-central chi-square with d = 4 kappa theta / sigma^2
//     degrees of freedom and non-centrality lambda = V_u e^{-kappa D} / c,
//     c = sigma^2 (1 - e^{-kappa D}) / (4 kappa): for d > 1,
//     X = 2 Gamma((d-1)/2) + (Zv + sqrt(lambda))^2; for d <= 1,
//     X = 2 Gamma(d/2 + N), N ~ Poisson(lambda / 2) by inversion.  Gamma draws
//     by Marsaglia and Tsang (ACM TOMS 26(3), 2000; full acceptance test,
//     shapes below one raised by one and multiplied by U^(1/shape)).
//  2. I = int_u^t V given (V_u, V_t): inversion of its CDF, F(x) = h x / pi +
//     (2/pi) sum_j sin(h j x)/j Re Phi(h j), at a uniform U, where Phi is the
//     conditional characteristic function of the paper (exponents negative,
//     the Bessel-function ratio I_nu(z(a)) / I_nu(z(0)), nu = d/2 - 1, taken
//     on the branch continuous along the grid, ln z summed from its factors).  The grid spacing h = pi / u_eps
//     with u_eps = mean + 12 sd (from the slope and curvature of log Phi at
//     0), the grid length the first power of two >= 64 at which |Phi|/J falls
//     below pi 1e-10 / 2, truncated after the last point above it.  Inversion:
//     bisection on [0, u_eps] with Newton steps, to |F - U| < 1e-13.
//  3. x += r D - I/2 + rho (V_t - V_u - kappa theta D + kappa I) / sigma
//          + sqrt(1 - rho^2) sqrt(I) Zs.
// I_nu(z) = (z/2)^nu S(z) / Gamma(nu + 1) with S(z) = sum_k (z^2/4)^k
// Gamma(nu+1) / (k! Gamma(k+nu+1)), summed directly: the Gamma(nu + 1) cancels
// in the ratio, and (z/2)^nu takes the continuous argument of z.  The sum loses
// about e^{|z| - Re z} times the rounding unit; a path whose grid needs
// |z| - Re z > 20 or |z| > 600, more than EXACT_MAX_GRID points, a Poisson
// mean above EXACT_MAX_POISSON_MEAN or EXACT_MAX_GAMMA_ATTEMPTS rejections is
// counted as failed (payoff 0) and the call reports it.
//
// Random inputs: block k of step j of path p is Philox4x32-10 at counter
// (j, lo32 p, hi32 p, 5 + 256 k).  Block 0: Box-Muller of words 0, 1 gives
// (Zv, Zs), word 2 the uniform U of the inversion, word 3 the Poisson
// uniform; blocks k >= 1 are the gamma sampler's attempts (the first normal
// of words 0, 1 and the acceptance uniform of word 2; word 3 of block 1 is
// the uniform that lowers a shape below one).
//
// Layout: a draw's characteristic function at 120 to 700 grid points is nearly
// all of the work, and points are independent, so a group of 16 lanes (a DPP
// row) takes one path and its lanes the points 16 m + 1 .. 16 m + 16: a wave
// holds four paths instead of 64, whose grid lengths, series and iteration
// counts otherwise leave two fifths of its lanes idle, and a launch of 2^16
// paths has 16 waves per SIMD of work instead of one.  Group sums are DPP
// butterflies (the same value in every lane, so a group's control flow is
// uniform).  The gamma sampler's attempts run one per lane as well.
// A point costs about 350 VALU instructions (900 before): one square root, a
// sine and exponential and one complex logarithm give g, e^{-gD/2} and ln z,
// z^2/4 is formed without a logarithm, and the Bessel series takes its
// 1 / (k (k + nu)) from an LDS table.
// The Re Phi / j of the current draw stay in LDS up to EXACT_LDS_POINTS points
// of a group, beyond that in the group's row of `scratch`: 39 KiB per block and
// 128 VGPRs, four blocks per CU (three with 320 points in LDS and 168 VGPRs ran
// 18% longer: the sampler waits on its own dependent chains; VALU-busy 0.72 at
// four, 0.58-0.63 at three).
// European call, 2^18 paths, one step: 3.33 -> 1.11 ms; the quarterly Asian
// (paper's parameters, four steps), 2^16 paths: 19.9 -> 2.66 ms.
//
// Each group walks paths group, group + n_groups, ... and its first lane keeps
// FP64 sums of the estimators, reduced per block at the end.
#include <hip/hip_runtime.h>

#include "cplx.hpp"
#include "device_math.hpp"
#include "internal.hpp"
#include "path_step.hpp"

namespace heston {
namespace {

constexpr double PI = 3.14159265358979323846;
constexpr double GRID_EPS = 1e-10;
constexpr int GROUP = EXACT_GROUP;
constexpr int GROUPS = BLOCK / GROUP; // groups per block
constexpr uint32_t LDS_ROW = EXACT_LDS_POINTS + 16; // rows of neighbouring groups on other banks
constexpr int RC_TABLE = 256;

struct ExactShared {
    double w[GROUPS][LDS_ROW]; // Re Phi(h j) / j, j = 1 ..
    double rc[RC_TABLE];       // 1 / (k (k + nu)), k = 1 .. RC_TABLE
    double red[BLOCK / 64][EXACT_REC];
};

template <int CTRL> __device__ __forceinline__ double row_move(double v)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}
// Sum over the group's 16 lanes, bitwise the same in each: quads by
// quad_perm, their halves and the row by mirrors.
__device__ __forceinline__ double group_sum(double v)
{
    v += row_move<0xB1>(v);  // lane ^ 1
    v += row_move<0x4E>(v);  // lane ^ 2
    v += row_move<0x141>(v); // half mirror
    v += row_move<0x140>(v); // mirror
    return v;
}
__device__ __forceinline__ int group_lane() { return threadIdx.x & (GROUP - 1); }
// Bit l: the condition in lane l of the group.
__device__ __forceinline__ uint32_t group_vote(bool c)
{
    const uint64_t b = __builtin_amdgcn_ballot_w64(c);
    return (uint32_t)(b >> (threadIdx.x & 48u)) & 0xFFFFu;
}

// Philox blocks of one (path, step).
struct Draw {
    uint32_t plo, phi, step, k0, k1;
    __device__ U4 block(uint32_t k) const
    {
        return philox4x32_10(U4{step, plo, phi, EXACT_COUNTER_TAG + (k << 8)}, k0, k1);
    }
};

// Gamma(alpha, 1), NaN after too many rejections: lane l of the group takes
// attempts l + 1, l + 17, ...; the first accepted one counts, as in a
// sequential walk.
__device__ double gamma_draw(double alpha, const Draw &dr)
{
    const double a = alpha < 1.0 ? alpha + 1.0 : alpha;
    const double d = a - 1.0 / 3.0, c = 1.0 / sqrt(9.0 * d);
    double g = __builtin_nan("");
    uint32_t w1 = 0; // word 3 of block 1 (lane 0's first attempt)
    for (int k0 = 1; k0 <= EXACT_MAX_GAMMA_ATTEMPTS; k0 += GROUP) {
        const U4 w = dr.block((uint32_t)(k0 + group_lane()));
        if (k0 == 1)
            w1 = w.w;
        double x, unused;
        box_muller_words(w.x, w.y, x, unused);
        const double v1 = 1.0 + c * x, v = v1 * v1 * v1;
        const bool ok = v1 > 0.0 &&
                        -0.5 * neg2_log_uniform(w.z) < 0.5 * x * x + d - d * v + d * log(v);
        const uint32_t accepted = group_vote(ok);
        if (accepted) {
            g = __shfl(d * v, __builtin_ctz(accepted), GROUP);
            break;
        }
    }
    if (alpha < 1.0)
        g *= pow(uniform_f64((uint32_t)__shfl((int)w1, 0, GROUP)), 1.0 / alpha);
    return g;
}
static_assert(EXACT_MAX_GAMMA_ATTEMPTS % GROUP == 0, "whole rounds of attempts");

// Smallest k with u <= P(N <= k), N ~ Poisson(mu); NaN above the mean limit.
__device__ double poisson_inverse(double mu, double u)
{
    if (mu > EXACT_MAX_POISSON_MEAN)
        return __builtin_nan("");
    double pk = exp(-mu), F = pk;
    const int cap = (int)(mu + 40.0 * sqrt(mu) + 100.0);
    int k = 0;
    while (u > F && k < cap) {
        ++k;
        pk *= mu / k;
        F += pk;
    }
    return (double)k;
}

// 1 / (k (k + nu)): hardware reciprocal and one Newton step.
__device__ __forceinline__ double series_rc(int k, double nu)
{
    const double den = (double)k * ((double)k + nu);
    const double rc = __builtin_amdgcn_rcp(den);
    return rc * fma(-den, rc, 2.0);
}

// S = sum_k q^k / (k! (nu+1)_k), q = z^2 / 4, four terms between checks (their
// table entries read ahead); `bad` set if the sum does not settle.
__device__ __forceinline__ Cx bessel_sum(Cx q, const double *rc, double nu, bool &bad)
{
    Cx t{1.0, 0.0}, s{1.0, 0.0};
    const double q2 = q.re * q.re + q.im * q.im;
    auto four = [&](double f0, double f1, double f2, double f3) {
        t = t * (q * f0);
        s = s + t;
        t = t * (q * f1);
        s = s + t;
        t = t * (q * f2);
        s = s + t;
        t = t * (q * f3);
        s = s + t;
    };
    // k > |z| / 2 (as k^4 > |q|^2) and |t| < 1e-17 |s|, the moduli by their parts:
    // S reaches e^600, whose square is beyond double's range
    auto settled = [&](int k) {
        const double k2 = (double)(k * k);
        return k2 * k2 > q2 && fabs(t.re) + fabs(t.im) < 1e-17 * (fabs(s.re) + fabs(s.im));
    };
    for (int k = 0; k < RC_TABLE; k += 4) {
        four(rc[k], rc[k + 1], rc[k + 2], rc[k + 3]);
        if (settled(k + 4))
            return s;
    }
    for (int k = RC_TABLE + 1; k < 2000; k += 4) {
        four(series_rc(k, nu), series_rc(k + 1, nu), series_rc(k + 2, nu), series_rc(k + 3, nu));
        if (settled(k + 3))
            return s;
    }
    bad = true;
    return s;
}
// The same at a real z >= 0.
__device__ __forceinline__ double bessel_sum_real(double q, double az, const double *rc, double nu,
                                                  bool &bad)
{
    double t = 1.0, s = 1.0;
    for (int k = 1; k < 2000; ++k) {
        t *= q * (k <= RC_TABLE ? rc[k - 1] : series_rc(k, nu));
        s += t;
        if ((double)k > 0.5 * az && t < 1e-17 * s)
            return s;
    }
    bad = true;
    return s;
}

// Per-draw constants of Phi.
struct PhiCtx {
    double sum_v; // (vu + vt) / sigma^2
    double vv;    // vu vt
    double c0;    // the constant part of ln|Phi / S|
};

// Phi(a) = e^{lp} S: lp returned, S = S(z(a)) and |z^2/4|^2 in *s and *q2.  With
// g = sqrt(kappa^2 - 2 i sigma^2 a) and z = (4/sigma^2) sqrt(vu vt) g
// e^{-gD/2} / (1 - e^{-gD}), ln(g / (1 - e^{-gD})) - gD/2 is the logarithm of
// both the first factor of Phi and of z up to constants; its imaginary part,
// arg(g conj(1 - e^{-gD})) - Im g D/2, is continuous along a >= 0 (each
// argument stays within (-3 pi/4, pi/2)), the branch of (z/2)^nu; the modulus
// |g|^2 = |kappa^2 - 2 i sigma^2 a|.  Summed from its factors it cannot
// underflow; q = z^2/4 may, where S is 1.
__device__ __forceinline__ Cx log_phi_part(const ExactLaunch &L, const PhiCtx &pc, const double *rc,
                                           double a, Cx *s, double *q2, bool &bad)
{
    const double b = L.two_sigma2 * a;
    const double m = sqrt_nonneg(fma(b, b, L.kappa2 * L.kappa2));
    // gr = sqrt(x) and gi = -b / (2 gr) from one reciprocal square root
    const double x = 0.5 * (m + L.kappa2), ir = rsqrt_pos(x);
    const double g0 = x * ir, gr = fma(fma(-g0, g0, x), 0.5 * ir, g0), gi = -0.5 * b * ir;
    const double u = 0.5 * L.D * gr, ph = -0.5 * L.D * gi;
    double c, sn;
    cos_sin(ph, c, sn);
    const double e = exp_plain(-u);
    const Cx e1{e * c, e * sn}, eg = e1 * e1;
    const Cx ome{1.0 - eg.re, -eg.im};
    const double w2 = ome.re * ome.re + ome.im * ome.im, iw = rcp_pos(w2);
    const double x1 = -0.25 * neg2_log(m * iw, 0) - u;
    const double A = angle(gr * ome.re + gi * ome.im, gi * ome.re - gr * ome.im) + ph;
    // (1 + e^{-gD}) / (1 - e^{-gD})
    const Cx ct{(1.0 - (eg.re * eg.re + eg.im * eg.im)) * iw, 2.0 * eg.im * iw};
    Cx lp;
    lp.re = x1 * (L.nu + 1.0) + pc.c0 + (L.coth_k - (gr * ct.re - gi * ct.im)) * pc.sum_v;
    lp.im = A * (L.nu + 1.0) - (gr * ct.im + gi * ct.re) * pc.sum_v;
    const double f = 2.0 * L.inv_sigma2 * iw;
    const Cx q = Cx{L.kappa2, -b} * eg * (Cx{ome.re * ome.re - ome.im * ome.im, -2.0 * ome.re * ome.im} *
                                          (f * f * pc.vv));
    *q2 = q.re * q.re + q.im * q.im;
    // |z| > 10: the series loses about e^{|z| - Re z} roundings (a wave-uniform
    // branch, else the compiler evaluates it for every point)
    if (__builtin_amdgcn_ballot_w64(*q2 > 625.0)) {
        const double az = 2.0 * sqrt_nonneg(sqrt_nonneg(*q2));
        double cA, sA;
        cos_sin(A, cA, sA);
        if (az > 10.0 && (az > 600.0 || az - az * cA > 20.0))
            bad = true;
    }
    *s = bessel_sum(q, rc, L.nu, bad);
    return lp;
}

// ln |s|; scaled where the square of a part could leave double's range.
__device__ __forceinline__ double log_modulus(Cx s)
{
    const bool big = fabs(s.re) + fabs(s.im) > 0x1p500;
    const double f = big ? 0x1p-500 : 1.0, re = s.re * f, im = s.im * f;
    return 0.5 * log_pos(re * re + im * im) + (big ? 500.0 * 0.69314718055994530942 : 0.0);
}

// Conditional mean and standard deviation of I from log Phi at a = h, 2h (even
// and odd lanes).
__device__ __forceinline__ void moments(const ExactLaunch &L, const PhiCtx &pc, const double *rc,
                                        double vu, double vt, double &mu, double &sd, bool &bad)
{
    const double guess = fmax(0.5 * (vu + vt) * L.D, 1e-10);
    const double h = 1e-3 / guess;
    Cx s;
    double q2;
    const Cx lp = log_phi_part(L, pc, rc, (threadIdx.x & 1) ? 2.0 * h : h, &s, &q2, bad);
    const Cx l{lp.re + log_modulus(s), lp.im + angle_scaled(s.re, s.im)};
    const double ore = row_move<0xB1>(l.re), oim = row_move<0xB1>(l.im);
    const bool odd = threadIdx.x & 1;
    const double re0 = odd ? ore : l.re, re1 = odd ? l.re : ore;
    const double im0 = odd ? oim : l.im, im1 = odd ? l.im : oim;
    mu = (8.0 * im0 - im1) / (6.0 * h);
    const double var = -(16.0 * re0 - re1) / (6.0 * h * h);
    sd = sqrt(fmax(var, (1e-3 * mu) * (1e-3 * mu)));
}

// F(x) = h x / pi + (2/pi) sum_j sin(h j x) w_j, its density and the density's
// derivative: lane l sums j = l + 1, l + 17, ... by a rotation of 16 h x,
// re-anchored at EXACT_LDS_POINTS and every 64 terms from there.  (Lanes whose
// last row lies beyond K keep their j a row behind; they have no later terms.)
__device__ __forceinline__ void cdf_pdf(const double *row, const double *far, uint32_t K, double h,
                                        double x, double &F, double &f, double &fp)
{
    const double th = h * x;
    double s, c, s16, c16;
    double j = (double)(group_lane() + 1);
    cos_sin(th * j, c, s);
    s16 = __shfl(s, GROUP - 1, GROUP);
    c16 = __shfl(c, GROUP - 1, GROUP);
    double sf = 0.0, sp = 0.0, sd = 0.0;
    auto terms = [&](const double *w_at, uint32_t from, uint32_t to) {
        for (uint32_t i = from; i < to; i += GROUP) {
            const double w = w_at[i], jw = j * w;
            sf += s * w;
            sp += c * jw;
            sd += s * (j * jw);
            j += (double)GROUP;
            const double sn = s * c16 + c * s16;
            c = c * c16 - s * s16;
            s = sn;
        }
    };
    const uint32_t l = (uint32_t)group_lane();
    terms(row, l, min(K, EXACT_LDS_POINTS));
    for (uint32_t b = EXACT_LDS_POINTS; b < K; b += 64 * GROUP) {
        cos_sin(th * j, c, s);
        terms(far, b + l, min(K, b + 64 * GROUP));
    }
    F = h * x * (1.0 / PI) + (2.0 / PI) * group_sum(sf);
    f = h / PI + (2.0 * h / PI) * group_sum(sp);
    fp = -(2.0 * h * h / PI) * group_sum(sd);
}

// Standard normal quantile to 4.5e-4 (Abramowitz and Stegun 26.2.23), for the
// inversion's first guess only.
__device__ __forceinline__ float rough_normal(float u)
{
    const float p = u < 0.5f ? u : 1.0f - u;
    const float t = __builtin_amdgcn_sqrtf(-1.38629436f * __builtin_amdgcn_logf(p));
    const float z = t - (2.515517f + t * (0.802853f + t * 0.010328f)) /
                            (1.0f + t * (1.432788f + t * (0.189269f + t * 0.001308f)));
    return u < 0.5f ? -z : z;
}

// One draw of I given (vu, vt) at the uniform u; `row` is the group's LDS row,
// `far` its scratch row.
__device__ double sample_integral(const ExactLaunch &L, double vu, double vt, double u, double *row,
                                  double *far, const double *rc, bool &bad)
{
    PhiCtx pc;
    pc.sum_v = (vu + vt) * L.inv_sigma2;
    pc.vv = vu * vt;
    pc.c0 = L.t1_const + L.nu * (L.log4_over_sigma2 - L.log_zk_scale);
    if (pc.vv != 0.0) {
        const double azk = sqrt_nonneg(pc.vv) * exp_plain(L.log_zk_scale);
        if (azk > 600.0)
            bad = true;
        pc.c0 -= log_pos(bessel_sum_real(0.25 * azk * azk, azk, rc, L.nu, bad));
    }
    double mu, sd;
    moments(L, pc, rc, vu, vt, mu, sd, bad);
    const double ueps = mu + 12.0 * sd;
    const double h = PI / ueps;
    const double thr = PI * GRID_EPS / 2.0;
    // The grid is the first power of two J >= 64 points at whose end |Phi| / J
    // is below the threshold, kept up to the last point K whose |Phi| / j
    // reaches it.  Rows of 16 points end before J where no later point can
    // reach the threshold or fail: |Phi| = G |S| with G / j decreasing in a
    // (|g / sinh(gD/2)| falls and Re(g coth(gD/2)) rises with a), and with
    // |q| <= (nu + 1) / 4 every zero of S (4 |q| >= 4 (nu + 1) by Rayleigh's
    // sum of the zeros of J_nu) is far enough that |S| can grow by less than 2.
    const double q_small = fmin(0.25 * (L.nu + 1.0), 25.0), q2_small = q_small * q_small;
    uint32_t J = 64, K = 0;
    for (uint32_t m = 0;; m += GROUP) {
        const uint32_t i = m + (uint32_t)group_lane();
        const double j = (double)(i + 1);
        Cx s;
        double q2;
        const Cx lp = log_phi_part(L, pc, rc, h * j, &s, &q2, bad);
        double c, sn;
        cos_sin(lp.im, c, sn);
        const double e = exp_plain(lp.re);
        const double re = e * (c * s.re - sn * s.im), im = e * (c * s.im + sn * s.re);
        const double w = re * rcp_pos(j);
        if (i < EXACT_LDS_POINTS)
            row[i] = w;
        else
            far[i] = w;
        const double a2 = re * re + im * im, t2 = (thr * j) * (thr * j);
        if (a2 >= t2)
            K = i + 1;
        // the row's last point decides
        const int flags = (a2 < t2 ? 1 : 0) | (4.0 * a2 < t2 && q2 <= q2_small ? 2 : 0);
        const int last = __builtin_amdgcn_mov_dpp(flags, 0x15F, 0xF, 0xF, true); // lane 15's
        if (last & 2)
            break;
        if (m + GROUP == J) {
            if (last & 1)
                break;
            if (J >= EXACT_MAX_GRID || group_vote(bad)) { // the next points would not fit
                bad = true;
                break;
            }
            J *= 2;
        }
    }
    bad = group_vote(bad) != 0;
    // the last point at or above the threshold over the group's lanes
    K = max(K, (uint32_t)__builtin_amdgcn_mov_dpp((int)K, 0xB1, 0xF, 0xF, true));
    K = max(K, (uint32_t)__builtin_amdgcn_mov_dpp((int)K, 0x4E, 0xF, 0xF, true));
    K = max(K, (uint32_t)__builtin_amdgcn_mov_dpp((int)K, 0x141, 0xF, 0xF, true));
    K = max(K, (uint32_t)__builtin_amdgcn_mov_dpp((int)K, 0x140, 0xF, 0xF, true));
    if (K == 0)
        K = 1;
    if (bad || !(ueps > 0.0))
        return __builtin_nan("");
    // First guess: the quantile of the lognormal with I's mean and deviation;
    // then Halley steps within a shrinking bracket (about three evaluations;
    // Newton from the mean took six).
    double lo = 0.0, hi = ueps;
    const float v = (float)(sd / mu), ls = 0.69314718f * __builtin_amdgcn_logf(1.0f + v * v);
    const float zq = rough_normal((float)u);
    double x = mu * (double)fast_exp(__builtin_amdgcn_sqrtf(ls) * zq - 0.5f * ls);
    x = fmin(fmax(x, 1e-12), 0.999999 * ueps);
    for (int it = 0; it < 200; ++it) {
        double F, f, fp;
        cdf_pdf(row, far, K, h, x, F, f, fp);
        const double e = F - u;
        if (fabs(e) < 1e-13)
            return x;
        if (e > 0.0)
            hi = x;
        else
            lo = x;
        if (hi - lo < 1e-14 * fmax(1.0, hi))
            return x;
        const double newton = e / f, damp = 1.0 - 0.5 * newton * fp / f;
        const double step = damp > 0.5 && damp < 2.0 ? newton / damp : newton;
        const double xn = f > 0.0 ? x - step : 0.5 * (lo + hi);
        x = (lo < xn && xn < hi) ? xn : 0.5 * (lo + hi);
    }
    return x;
}

__global__ __launch_bounds__(BLOCK, 4) void exact_kernel(const ExactLaunch L)
{
    __shared__ ExactShared sh;
    load_fp64_tables<BLOCK>();
    for (int k = threadIdx.x; k < RC_TABLE; k += BLOCK)
        sh.rc[k] = series_rc(k + 1, L.nu);
    __syncthreads();
    const uint32_t group = blockIdx.x * GROUPS + threadIdx.x / GROUP;
    const bool first_lane = group_lane() == 0;
    // sums of price, pathwise Delta and Rho (value, square) and the failures
    double acc[7] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    const bool asian = L.opt_type >= 2, geo = L.opt_type >= 4;
    const bool call = L.opt_type == 0 || L.opt_type == 2 || L.opt_type == 4;
    const double sgn = call ? 1.0 : -1.0;
    const double disc = exp(-L.r * L.T), lnS0 = log(L.S0), nfix = (double)L.n_fix;
    const double D = L.D;
    if (group < L.n_groups) {
        double *row = sh.w[threadIdx.x / GROUP];
        double *far = L.scratch + (uint64_t)group * EXACT_FAR_POINTS;
        for (uint64_t i = group; i < L.n_paths; i += L.n_groups) {
            const uint64_t p = L.first_path + i;
            Draw dr{(uint32_t)p, (uint32_t)(p >> 32), 0u, (uint32_t)L.seed,
                    (uint32_t)(L.seed >> 32)};
            double x = 0.0, V = L.v0, A = 0.0, B = 0.0, Itot = 0.0;
            bool bad = false;
            for (uint32_t j = 0; j < L.n_steps && !bad; ++j) {
                dr.step = j;
                const U4 w = dr.block(0);
                double zv, zs;
                box_muller_words(w.x, w.y, zv, zs);
                const double lam = V * L.ekD / L.c;
                double shape = 0.5 * (L.d - 1.0), square = 0.0;
                if (L.d > 1.0) {
                    const double sq = zv + sqrt_nonneg(lam);
                    square = sq * sq;
                } else { // NaN above the mean limit
                    shape = 0.5 * L.d + poisson_inverse(0.5 * lam, uniform_f64(w.w));
                }
                const double X = 2.0 * gamma_draw(shape, dr) + square;
                const double vt = L.c * X;
                if (!(vt >= 0.0)) {
                    bad = true;
                    break;
                }
                const double I = sample_integral(L, V, vt, uniform_f64(w.z), row, far, sh.rc, bad);
                if (bad)
                    break;
                Itot += I;
                const double isq = (vt - V - L.kappa * L.theta * D + L.kappa * I) / L.sigma;
                x += L.r * D - 0.5 * I + L.rho * isq + L.rho_bar * sqrt(fmax(I, 0.0)) * zs;
                V = vt;
                if (asian && is_fixing(L.fix_bits, j + 1)) {
                    const double t = (double)(j + 1) * D;
                    if (geo) {
                        A += lnS0 + x;
                        B += t;
                    } else {
                        const double S = L.S0 * exp(x);
                        A += S;
                        B += t * S;
                    }
                }
            }
            const double ST = L.S0 * exp(x);
            const double Xv = geo ? exp(A / nfix) : asian ? A / nfix : ST;
            if (geo)
                B = Xv * B;
            const bool itm = sgn * (Xv - L.K) > 0.0;
            double est[3];
            est[0] = itm ? disc * sgn * (Xv - L.K) : 0.0;
            est[1] = itm ? sgn * disc * Xv / L.S0 : 0.0;
            est[2] = !itm ? 0.0
                     : asian ? disc * (sgn * B / nfix - L.T * sgn * (Xv - L.K))
                             : sgn * disc * L.K * L.T;
            if (!first_lane)
                continue;
            if (bad) {
                acc[6] += 1.0;
            } else {
#pragma unroll
                for (int e = 0; e < 3; ++e) {
                    acc[2 * e] += est[e];
                    acc[2 * e + 1] += est[e] * est[e];
                }
            }
            if (L.dump != nullptr) {
                double *rec = L.dump + i * DUMP_WIDTH;
                const double nan = __builtin_nan("");
                rec[0] = bad ? nan : ST;
                rec[1] = bad ? nan : V;
                rec[2] = bad ? nan : Xv;
                rec[3] = bad ? nan : est[0];
                rec[4] = bad ? nan : est[1];
                rec[5] = bad ? nan : est[2];
#pragma unroll
                for (int k = 6; k < 14; ++k)
                    rec[k] = nan;
                rec[14] = bad ? nan : x;
                rec[15] = bad ? nan : Itot;
            }
        }
    }
    const int wl = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < EXACT_REC; ++k) {
        const double v = k < 6 ? acc[k] : k == N_ACC ? acc[6] : 0.0;
        const double s = wave_sum(v);
        if (wl == 0)
            sh.red[wave][k] = s;
    }
    __syncthreads();
    if (threadIdx.x < EXACT_REC) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < BLOCK / 64; ++w)
            s += sh.red[w][threadIdx.x];
        L.partials[(uint64_t)blockIdx.x * EXACT_REC + threadIdx.x] = s;
    }
}

} // namespace

hipError_t launch_exact(const ExactLaunch &L, hipStream_t stream)
{
    if (L.n_groups == 0 || L.n_groups % GROUPS != 0 || L.n_groups > EXACT_MAX_GROUPS)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(exact_kernel, dim3(L.n_groups / GROUPS), dim3(BLOCK), 0, stream, L);
    return hipGetLastError();
}

} // namespace heston
