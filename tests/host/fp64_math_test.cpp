// CPU test of the double-precision elementary functions (fp64_math.hpp compiled
// by the host compiler): each against long double over the arguments its callers
// pass, with the hardware's reciprocal estimates off by up to 2^-25 either way.
// Errors in units of the last place (ulp) of the reference; each bound is the sum
// of the roundings on the way (named beside it).
#include <cstdio>
#include <random>

#include "fp64_math.hpp"

using namespace heston;
typedef long double L;

static int failed = 0;
static double ulps(double got, L want)
{
    const double w = (double)want;
    const double u = fmax(nextafter(fabs(w), INFINITY) - fabs(w), 0x1p-1074);
    return fabs((double)(((L)got - want) / u));
}
struct Worst {
    const char *name;
    double bound, worst = 0, at = 0, sum2 = 0;
    long n = 0;
    Worst(const char *name, double bound) : name(name), bound(bound) {}
    void see(double e, double x)
    {
        sum2 += e * e;
        ++n;
        if (!(e <= worst)) {
            worst = e;
            at = x;
        }
    }
    ~Worst()
    {
        if (getenv("SHOW"))
            printf("%-24s worst %.4f (%a) rms %.4f of %ld\n", name, worst, at, std::sqrt(sum2 / n), n);
        if (!(worst <= bound)) {
            printf("%s: %.4f above %.4f at %a\n", name, worst, bound, at);
            failed = 1;
        }
    }
};
static void check(bool ok, const char *what)
{
    if (!ok) {
        printf("%s\n", what);
        failed = 1;
    }
}
static std::mt19937_64 gen(1);
static double uniform(double lo, double hi) { return std::uniform_real_distribution<double>(lo, hi)(gen); }
static double log_uniform(double lo, double hi) { return exp(uniform(log(lo), log(hi))); }

// Every seventh uniform and the first and last of each binade's cells.
static void box_muller()
{
    // the radius: half the relative error of the logarithm's two roundings, its
    // constants and the series (below 2 ulp) and the square root's rounding
    Worst log2u("neg2_log_uniform", 2), radius("radius", 1.5);
    // cos and sin next to 1: the table's and the final rounding; in ulp of 1/2 .. 1
    Worst circle("cos_sin_uniform / 2^-53", 2);
    const L pi = acosl(-1.0L);
    for (uint32_t m = 0; m < 1u << 23; m += (m < 64 || (m & 0x7FFF) < 4 || m > (1u << 23) - 64) ? 1 : 7) {
        const uint32_t w = m << 9 | (m * 2654435761u >> 23);
        const L u = ((L)m + 0.5L) * 0x1p-23L, want = -2.0L * logl(u);
        const double got = neg2_log_uniform(w);
        log2u.see(ulps(got, want), (double)u);
        radius.see(ulps(sqrt_nonneg(got), sqrtl(want)), (double)u);
        double c, s;
        cos_sin_uniform(w, c, s);
        // the angle less its quarter turns, exactly
        const L quarter = floorl(4 * u + 0.5L), y = 2 * pi * (u - quarter / 4);
        const int k = (int)quarter & 3;
        const L cy = cosl(y), sy = sinl(y);
        const L wc = k == 0 ? cy : k == 1 ? -sy : k == 2 ? -cy : sy;
        const L ws = k == 0 ? sy : k == 1 ? cy : k == 2 ? -sy : -cy;
        circle.see(fabs((double)((L)c - wc)) * 0x1p53, (double)u);
        circle.see(fabs((double)((L)s - ws)) * 0x1p53, (double)u);
    }
}

static void roots_and_reciprocals()
{
    Worst root("sqrt_nonneg", 0.501); // one rounding behind a remainder correction
    Worst rcp("rcp_pos", 0.501);      // one rounding behind two Newton steps
    Worst rsqrt("rsqrt_pos", 1.01);   // the last rounding, and x y's in the residual
    for (int i = 0; i < 1 << 20; ++i) {
        const double x = log_uniform(1e-200, 1e200), near1 = 1.0 + i * 0x1p-20;
        for (double v : {x, near1, 4 * near1 - 2}) {
            root.see(ulps(sqrt_nonneg(v), sqrtl(v)), v);
            rcp.see(ulps(rcp_pos(v), 1.0L / v), v);
            rsqrt.see(ulps(rsqrt_pos(v), 1.0L / sqrtl(v)), v);
        }
    }
    check(sqrt_nonneg(0.0) == 0.0, "sqrt_nonneg(0)");
    check(std::isnan(sqrt_nonneg(NAN)), "sqrt_nonneg(NaN)");
}

static void exponentials_and_logarithm()
{
    // the product's rounding in the last term's sum and the sum's (f q up to 0.42)
    Worst e2("exp2_plain", 1), e1("exp_plain", 1), ln("log_pos", 2);
    for (int i = 0; i < 1 << 20; ++i) {
        const double y = i & 1 ? uniform(-1000, 1000) : uniform(-1, 1);
        e2.see(ulps(exp2_plain(y), exp2l(y)), y);
        const double x = i & 1 ? uniform(-700, 700) : uniform(-1, 1);
        e1.see(ulps(exp_plain(x), expl(x)), x);
        const double v = i & 1 ? log_uniform(1e-300, 1e300) : uniform(0.9, 1.1);
        if (v != 1.0)
            ln.see(ulps(log_pos(v), logl(v)), v);
    }
    check(log_pos(1.0) == 0.0, "log_pos(1)");
    for (double x : {-745.2, -1100.0, -1e5, -1e17, -1e43, -1e200, -1.7e308, (double)-INFINITY})
        check(exp_low(x) == 0.0, "exp_low far below");
    for (double x : {-1e5, -1e17, -1e30, -1e40})
        check(exp_plain(x) == 0.0 && exp2_plain(x) == 0.0, "exponentials down to -1e40");
    check(std::isinf(exp_plain(710.0)) && std::isinf(exp2_plain(1024.0)), "exponentials above");
    check(std::isnan(exp_low(NAN)) && std::isnan(exp2_plain(NAN)), "exponentials of NaN");
    check(exp_low(-1099.5) == exp_plain(-1099.5) && exp_low(3.0) == exp_plain(3.0), "exp_low");
}

static void angles()
{
    Worst circle("cos_sin / 2^-53", 2.5); // as above, and the argument's reduction in two parts
    Worst arg("angle / 2^-51", 1.5);      // ulp of the largest angles; its sum, the table, the slope
    for (int i = 0; i < 1 << 19; ++i) {
        const double x = i & 1 ? uniform(-4, 4) : uniform(-1e6, 1e6);
        double c, s;
        cos_sin(x, c, s);
        circle.see(fabs((double)((L)c - cosl(x))) * 0x1p53, x);
        circle.see(fabs((double)((L)s - sinl(x))) * 0x1p53, x);
        const double t = uniform(-3.14159, 3.14159), r = log_uniform(1e-15, 1e15);
        const double px = r * cos(t), py = r * sin(t), f = log_uniform(1e-130, 1e130);
        arg.see(fabs((double)((L)angle(px, py) - atan2l(py, px))) * 0x1p51, t);
        arg.see(fabs((double)((L)angle_scaled(px * f, py * f) - atan2l(py * f, px * f))) * 0x1p51, t);
    }
    check(angle(1.0, 0.0) == 0.0 && fabs(angle(-1.0, 0.0) - M_PI) < 1e-15 &&
              fabs(angle(0.0, -2.0) + M_PI_2) < 1e-15,
          "angle on the axes");
}

int main()
{
    load_fp64_tables<1>();
    for (double err : {0.0, 0x1p-25, -0x1p-25}) {
        fake::estimate_error = err;
        box_muller();
        roots_and_reciprocals();
        exponentials_and_logarithm();
        angles();
    }
    if (!failed)
        printf("ok\n");
    return failed;
}
