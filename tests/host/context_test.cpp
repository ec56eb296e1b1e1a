// CPU test of the context's host code (api.hip compiled by the host compiler
// against the stand-in runtime of fake_hip, the kernels' launchers left empty):
// the device memory a call asks for, and what error returns leave behind.
#include <cstdio>

#include "api.hip"

namespace heston {
hipError_t launch_step_weights(const PriceLaunch &, void *, hipStream_t s) { return fake::work(s); }
hipError_t launch_sobol_hi(const uint32_t *, const int32_t *, uint32_t, uint32_t, uint32_t *,
                           hipStream_t s)
{
    return fake::work(s);
}
hipError_t launch_sobol_low(const uint32_t *, uint32_t, uint32_t *, hipStream_t s)
{
    return fake::work(s);
}
hipError_t launch_sobol_shifts(uint64_t, const int32_t *, uint32_t, uint32_t, uint32_t *,
                               hipStream_t s)
{
    return fake::work(s);
}
hipError_t launch_paths(const PriceLaunch &, hipStream_t s) { return fake::work(s); }
hipError_t launch_bump_combine(const double *, uint64_t, uint32_t, const BumpScales &, double *,
                               uint32_t, hipStream_t s)
{
    return fake::work(s);
}
hipError_t launch_reduce_rows(const double *, uint32_t, uint32_t, double *, hipStream_t s)
{
    return fake::work(s);
}
hipError_t launch_reduce(const PriceLaunch &, double *, hipStream_t s) { return fake::work(s); }
hipError_t launch_adjoint_forward(const PriceLaunch &, hipStream_t s) { return fake::work(s); }
hipError_t launch_adjoint(const PriceLaunch &, double, double *, hipStream_t s)
{
    return fake::work(s);
}
hipError_t launch_exact(const ExactLaunch &, hipStream_t s) { return fake::work(s); }
hipError_t launch_geo_nodes_fixed(const GeoControl &, double *, double *, hipStream_t s)
{
    return fake::work(s);
}
hipError_t launch_geo_finish_fixed(const GeoControl &, double *, double *, double *prices,
                                   hipStream_t s)
{
    prices[0] = prices[1] = 1.0;
    return fake::work(s);
}
hipError_t launch_geo_price_search(const GeoControl &, double *, double *, double *, hipStream_t s)
{
    return fake::work(s);
}
} // namespace heston

static int failed = 0;
#define CHECK(c)                                                                                   \
    do {                                                                                           \
        if (!(c)) {                                                                                \
            printf("line %d: %s\n", __LINE__, #c);                                                 \
            failed = 1;                                                                            \
        }                                                                                          \
    } while (0)

static const heston_params P = {100, 100, 0.05, 1, 0.04, 2, 0.04, 0.3, -0.7};

static uint64_t pages(uint64_t bytes) { return (bytes + 4095) & ~uint64_t(4095); }

// An exact call fits the budget that one lane per path took: a column of the
// grid per lane, one partial per 256 lanes and the sums.
static void exact_budget()
{
    heston_opts o;
    heston_default_opts(&o);
    o.precision = HESTON_FP64;
    o.scheme = HESTON_EXACT;
    o.greeks = HESTON_GREEKS_PATHWISE;
    for (uint64_t n : {2ull, 255ull, 256ull, 257ull, 4096ull, 16383ull, 16384ull, 16385ull, 100000ull,
                       131072ull, 1000000ull}) {
        const uint64_t lanes = std::min<uint64_t>((n + 255) / 256 * 256, 131072);
        const uint64_t budget = pages(lanes * EXACT_MAX_GRID * 8) +
                                pages(lanes / 256 * EXACT_REC * 8) + pages(EXACT_REC * 8);
        heston_ctx *c = nullptr;
        CHECK(heston_ctx_create(0, nullptr, budget, &c) == HESTON_OK);
        heston_result r;
        CHECK(heston_price_greeks_ex(c, &P, HESTON_EURO_CALL, n, 1, 1, &o, &r) == HESTON_OK);
        CHECK(heston_ctx_destroy(c) == HESTON_OK);
    }
}

// The control's buffers take no more of the budget than with one partial per 256
// transforms: four pages for the partials and one for the rest, at every range.
static void control_budget()
{
    heston_opts o;
    heston_default_opts(&o);
    o.control_variate = HESTON_CONTROL_GEOMETRIC;
    for (double T : {1.0, 0.01, 1e-4}) {
        heston_params p = P;
        p.T = T;
        o.bump_T_abs = T / 100;
        heston_ctx *c = nullptr;
        CHECK(heston_ctx_create(0, nullptr, 0, &c) == HESTON_OK);
        heston_result r;
        CHECK(heston_price_greeks_ex(c, &p, HESTON_ASIAN_CALL, 10000, 12, 1, &o, &r) == HESTON_OK);
        CHECK(c->geo_partials.bytes <= 4 * 4096 && c->geo_buf.bytes <= 4096);
        CHECK(heston_ctx_destroy(c) == HESTON_OK);
    }
}

// Whichever call fails, a control request returns with its side stream idle --
// its uploads read the caller's fixing dates, its last kernel writes pinned host
// memory -- and the context frees nothing while a stream has work.
static void control_error_returns()
{
    const uint32_t steps[] = {3, 6, 12};
    heston_opts o;
    heston_default_opts(&o);
    o.control_variate = HESTON_CONTROL_GEOMETRIC;
    o.fixing_steps = steps;
    o.n_fixings = 3;
    long points = 0;
    for (bool done = false; !done; ++points) {
        heston_ctx *c = nullptr;
        fake::pending.clear();
        CHECK(heston_ctx_create(0, nullptr, 0, &c) == HESTON_OK);
        fake::fail_at = fake::calls + points;
        heston_result r;
        done = heston_price_greeks_ex(c, &P, HESTON_ASIAN_CALL, 10000, 12, 1, &o, &r) == HESTON_OK;
        fake::fail_at = -1;
        CHECK(!c->side || fake::pending[c->side] == 0);
        CHECK(heston_ctx_destroy(c) == HESTON_OK);
    }
    CHECK(points > 20);
}

int main()
{
    control_error_returns();
    exact_budget();
    control_budget();
    for (auto &f : fake::faults) {
        printf("%s\n", f.c_str());
        failed = 1;
    }
    if (!failed)
        printf("ok\n");
    return failed;
}
