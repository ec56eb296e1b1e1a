"""GPU parity of the arithmetic-Asian price with the geometric-average control
variate.

Per path: the pricing kernel's dumped records (arithmetic payoff in column 3,
the control's geometric payoff in column 15) against the oracle's arithmetic
and geometric paths on the same inputs, at the per-path bar of the other
parity tests (1e-12 FP64, 1e-5 FP32 relative, floor S0).  Estimates: the
library's control mean (computed on the device by Gauss-Legendre panels)
against the oracle's transform price (adaptive quadrature) to 1e-9 relative,
and beta, the estimate and its error against oracle.control_variate on the
oracle's own paths (FP64); in FP32, against oracle.control_variate on the
kernel's dumped payoffs, and the gap to the oracle's estimate within the bound
that the per-path payoff bar implies.
"""
import math

import numpy as np
import pytest

import oracle
from workloads import BASE, PAPER, paper_fixing_steps

pytestmark = pytest.mark.gpu

PB = oracle.Params(**BASE)
PP = oracle.Params(**PAPER)
TOL = {0: 1e-12, 1: 1e-5}
GEO = {oracle.ASIAN_CALL: oracle.GEO_ASIAN_CALL, oracle.ASIAN_PUT: oracle.GEO_ASIAN_PUT}


@pytest.fixture(scope="module")
def hm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2309_10477_amd as hm
    hm.lib()
    return hm


@pytest.fixture(scope="module")
def ctx(hm):
    c = hm.Context(0)
    yield c
    c.close()


def close(name, g, o, tol, floor):
    err = np.abs(g - o) / np.maximum(np.abs(o), floor)
    if (err > tol).any():
        i = int(np.argmax(err))
        raise AssertionError(f"{name}: {int((err > tol).sum())} paths off, worst {i}: "
                             f"gpu {g[i]!r} oracle {o[i]!r} rel {err[i]:.3e}")


def fp32_estimate(r, d, a, g, mu, est_o, beta_o, R=None):
    """FP32 estimate checks.  The library's combination of its own FP64 sums
    equals the oracle's formula applied to the payoffs the kernel dumps; the
    gap from there to the oracle's estimate follows exactly from the per-path
    payoff errors: est_d - est_o = mean(a_d - a) - beta_d mean(g_d - g)
    - (beta_d - beta_o)(mean(g) - mu), each payoff error at most 1e-5 of
    max(S0, payoff) by the per-path check."""
    ad, gd = d[:, 3], d[:, 15]
    if R is None:
        est_d, se_d, beta_d = oracle.control_variate(ad, gd, mu)
    else:
        est_d, se_d, beta_d = oracle.control_variate_reps(ad, gd, mu, R)
    assert r["cv_beta"] == pytest.approx(beta_d, rel=1e-9)
    assert r["cv_price"][0] == pytest.approx(est_d, rel=1e-9)
    assert r["cv_price"][1] == pytest.approx(se_d, rel=1e-6)
    assert beta_d == pytest.approx(beta_o, rel=1e-3)
    scale = TOL[1] * max(PB.S0, np.abs(a).max(), np.abs(g).max())
    bar = scale * (1 + abs(beta_d)) + abs(beta_d - beta_o) * abs(g.mean() - mu)
    assert abs(est_d - est_o) <= bar, (est_d, est_o, bar)


def oracle_pays(p, opt, N, seed, n, mode, fix, za=None, zb=None):
    if mode == oracle.QE:
        a = oracle.simulate_qe(p, opt, N, seed, 0, n, fix, threads=8)[0][:, 3]
        g = oracle.simulate_qe(p, GEO[opt], N, seed, 0, n, fix, threads=8)[0][:, 3]
        return a, g
    a = oracle.simulate(p, opt, N, seed, 0, n, mode, fix, za, zb, threads=8)[:, 3]
    g = oracle.simulate(p, GEO[opt], N, seed, 0, n, mode, fix, za, zb, threads=8)[:, 3]
    return a, g


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("opt", [oracle.ASIAN_CALL, oracle.ASIAN_PUT])
@pytest.mark.parametrize("fix", [None, (3, 5, 9, 12)], ids=["every-step", "dates"])
def test_dumped_payoffs_and_estimate(hm, ctx, prec, opt, fix):
    n, N, seed = 5000 + 77, 12, 31
    opts = hm.Options(precision=prec, fixings=fix, control_variate=hm.CONTROL_GEOMETRIC,
                      greeks=hm.GREEKS_PATHWISE | hm.GREEKS_BUMP_FUSED)
    d = ctx.dump_paths(PB.__dict__, opt, n, N, seed, 0, n, opts).cpu().numpy()
    a, g = oracle_pays(PB, opt, N, seed, n, oracle.FULL_TRUNC, fix)
    close("pay", d[:, 3], a, TOL[prec], PB.S0)
    close("geo pay", d[:, 15], g, TOL[prec], PB.S0)
    r = ctx.price_greeks(PB.__dict__, opt, n, N, seed, opts)
    mu = oracle.geometric_control_mean(PB, opt, N, fix)
    assert r["cv_mean"] == pytest.approx(mu, rel=1e-9)
    est, se, beta = oracle.control_variate(a, g, mu)
    if prec == 0:
        assert r["cv_beta"] == pytest.approx(beta, rel=1e-9)
        assert r["cv_price"][0] == pytest.approx(est, rel=1e-9)
        assert r["cv_price"][1] == pytest.approx(se, rel=1e-6)
    else:
        fp32_estimate(r, d, a, g, mu, est, beta)
    plain = oracle.mean_se(a)
    assert r["price"][0] == pytest.approx(plain[0], rel=1e-9 if prec == 0 else 1e-5)


@pytest.mark.parametrize("scheme", [oracle.ABSORB, oracle.QE])
def test_other_schemes(hm, ctx, scheme):
    n, N, seed = 3001, 16, 5
    p = PP if scheme == oracle.ABSORB else PB
    opt = oracle.ASIAN_CALL
    opts = hm.Options(scheme=scheme, control_variate=hm.CONTROL_GEOMETRIC,
                      greeks=hm.GREEKS_PATHWISE)
    d = ctx.dump_paths(p.__dict__, opt, n, N, seed, 0, n, opts).cpu().numpy()
    a, g = oracle_pays(p, opt, N, seed, n, scheme, None)
    skip = np.zeros(n, bool)
    if scheme == oracle.QE:  # branch decisions taken within 1e-9 of the switch
        _, margin, _ = oracle.simulate_qe(p, opt, N, seed, 0, n, threads=8)
        skip = margin < 1e-9
        assert skip.mean() < 0.01
    close("pay", d[~skip, 3], a[~skip], 1e-12, p.S0)
    close("geo pay", d[~skip, 15], g[~skip], 1e-12, p.S0)
    r = ctx.price_greeks(p.__dict__, opt, n, N, seed, opts)
    mu = oracle.geometric_control_mean(p, opt, N)
    assert r["cv_mean"] == pytest.approx(mu, rel=1e-9)
    if not skip.any():
        est, se, beta = oracle.control_variate(a, g, mu)
        assert r["cv_price"][0] == pytest.approx(est, rel=1e-9)
        assert r["cv_price"][1] == pytest.approx(se, rel=1e-6)


@pytest.mark.parametrize("prec", [0, 1])
def test_sobol_replicates(hm, ctx, prec):
    from oracle import sobol
    R, M, N, seed = 8, 512, 12, 3
    n = R * M
    opt = oracle.ASIAN_PUT
    opts = hm.Options(precision=prec, rng=hm.SOBOL_BRIDGE, qmc_replicates=R,
                      control_variate=hm.CONTROL_GEOMETRIC, greeks=hm.GREEKS_PATHWISE)
    za, zb = sobol.normals(N, 0, n, R, M, seed)
    a, g = oracle_pays(PB, opt, N, seed, n, oracle.FULL_TRUNC, None, za, zb)
    d = ctx.dump_paths(PB.__dict__, opt, n, N, seed, 0, n, opts).cpu().numpy()
    close("pay", d[:, 3], a, TOL[prec], PB.S0)
    close("geo pay", d[:, 15], g, TOL[prec], PB.S0)
    r = ctx.price_greeks(PB.__dict__, opt, n, N, seed, opts)
    mu = oracle.geometric_control_mean(PB, opt, N)
    est, se, beta = oracle.control_variate_reps(a, g, mu, R)
    if prec == 0:
        assert r["cv_beta"] == pytest.approx(beta, rel=1e-9)
        assert r["cv_price"][0] == pytest.approx(est, rel=1e-9)
        assert r["cv_price"][1] == pytest.approx(se, rel=1e-6)
    else:
        fp32_estimate(r, d, a, g, mu, est, beta, R)


@pytest.mark.parametrize("p", [PB.replace(T=0.1, sigma=1.0, kappa=0.5),
                               PB.replace(T=5.0, rho=0.3, v0=0.09),
                               PP.replace(rho=-0.9),
                               PB.replace(T=0.01, v0=0.01, theta=0.01, sigma=0.1),
                               PB.replace(v0=0.01, theta=0.01, sigma=2.0, kappa=1.0)],
                         ids=["short-high-volvol", "long-positive-rho", "paper-rho-0.9",
                              "very-short-low-vol", "range-search"])
def test_control_mean_across_parameters(hm, ctx, p):
    """The last case's transform (vol of vol 2 over a variance level of 0.01)
    decays far more slowly than the library's first range assumes, so the
    library searches a longer one."""
    N = 48
    fix = tuple(range(4, 49, 4))
    for opt in (oracle.ASIAN_CALL, oracle.ASIAN_PUT):
        r = ctx.price_greeks(p.__dict__, opt, 1000, N, 1,
                             hm.Options(fixings=fix, control_variate=hm.CONTROL_GEOMETRIC,
                                        greeks=hm.GREEKS_PATHWISE))
        assert r["cv_mean"] == pytest.approx(oracle.geometric_control_mean(p, opt, N, fix),
                                             rel=1e-9)


@pytest.mark.parametrize("N", [1, 7, 9, 63, 64, 65, 129])
def test_control_mean_at_the_edges_of_its_chunks(hm, ctx, N):
    """The transform goes through the dates 64 at a time and 8 to an unrolled
    group: one date, either side of a group, of a chunk and of two chunks."""
    opts = hm.Options(precision=1, control_variate=hm.CONTROL_GEOMETRIC,
                      greeks=hm.GREEKS_PATHWISE)
    r = ctx.price_greeks(PB.__dict__, oracle.ASIAN_PUT, 256, N, 3, opts)
    assert r["cv_mean"] == pytest.approx(oracle.geometric_control_mean(PB, oracle.ASIAN_PUT, N, None),
                                         rel=1e-9)


@pytest.mark.parametrize("N", [8, 16, 17, 48])
@pytest.mark.parametrize("p", [PB, PB.replace(T=0.01, v0=0.01, theta=0.01, sigma=0.1),
                               PB.replace(v0=0.01, theta=0.01, sigma=2.0, kappa=1.0)],
                         ids=["short-range", "long-range", "search"])
def test_control_mean_at_the_edges_of_its_layouts(hm, ctx, p, N):
    """Eight transforms per block in a short range, 32 in a long (4096) and in a
    searched one, whose dates go sixteen to a chunk: up to one chunk, more."""
    opts = hm.Options(precision=1, control_variate=hm.CONTROL_GEOMETRIC,
                      greeks=hm.GREEKS_PATHWISE)
    for opt in (oracle.ASIAN_CALL, oracle.ASIAN_PUT):
        r = ctx.price_greeks(p.__dict__, opt, 256, N, 3, opts)
        assert r["cv_mean"] == pytest.approx(oracle.geometric_control_mean(p, opt, N, None), rel=1e-9)


def test_full_size_variance_reduction_and_agreement(hm, ctx):
    """2^20 paths x 252 daily fixings, FP32: the control cuts the standard
    error at least fivefold and the two estimates agree within their errors."""
    opts = hm.Options(precision=hm.FP32, control_variate=hm.CONTROL_GEOMETRIC,
                      greeks=hm.GREEKS_PATHWISE)
    r = ctx.price_greeks(PB.__dict__, hm.ASIAN_CALL, 1 << 20, 252, 42, opts)
    assert r["cv_price"][1] < 0.2 * r["price"][1]
    assert abs(r["cv_price"][0] - r["price"][0]) < 3.5 * r["price"][1]
    assert 0.5 < r["cv_beta"] < 1.5


def test_paper_exact_simulation_quarterly_asian(hm, ctx):
    """Paper parameters, quarterly fixings, absorption, 128 steps, 2^20 paths:
    the paper's exact-simulation value 4.3840 (0.0064)."""
    N = 128
    opts = hm.Options(precision=hm.FP32, scheme=hm.ABSORPTION, fixings=paper_fixing_steps(N),
                      control_variate=hm.CONTROL_GEOMETRIC, greeks=hm.GREEKS_PATHWISE)
    r = ctx.price_greeks(PP.__dict__, hm.ASIAN_CALL, 1 << 20, N, 29, opts)
    assert abs(r["cv_price"][0] - 4.3840) < 3 * math.hypot(r["cv_price"][1], 0.0064)


def test_rejections(hm, ctx):
    import torch
    cv = hm.Options(control_variate=hm.CONTROL_GEOMETRIC, greeks=hm.GREEKS_PATHWISE)
    cases = [
        (PB, hm.EURO_CALL, 100, 4, cv, -1),
        (PB, hm.GEO_ASIAN_CALL, 100, 4, cv, -1),
        (PB.replace(sigma=0.0), hm.ASIAN_CALL, 100, 4, cv, -1),
        (PB, hm.ASIAN_CALL, 100, hm.CONTROL_MAX_FIXINGS + 1, cv, -5),
        (PB, hm.ASIAN_CALL, 100, 4,
         hm.Options(control_variate=hm.CONTROL_GEOMETRIC, greeks=hm.GREEKS_BUMP_PLAIN), -5),
        (PB, hm.ASIAN_CALL, 100, 4, hm.Options(control_variate=7), -1),
    ]
    for p, t, n, N, o, status in cases:
        with pytest.raises(hm.HestonError) as e:
            ctx.price_greeks(p.__dict__, t, n, N, 1, o)
        assert e.value.status == status, (t, N)
    ck = torch.empty(hm.ckpt_bytes(256, 8, 8, hm.FP64), dtype=torch.uint8, device="cuda:0")
    with pytest.raises(hm.HestonError) as e:
        ctx.adjoint_forward(PB.__dict__, hm.ASIAN_CALL, 256, 8, 1, ck, 8, cv)
    assert e.value.status == -5
    with pytest.raises(hm.HestonError) as e:
        ctx.price_batch([dict(params=PB.__dict__, type=hm.ASIAN_CALL, n_steps=4, n_paths=100,
                              seed=1, want=1)], cv)
    assert e.value.status == -5


def test_full_size_sampled_paths_and_estimate(hm, ctx):
    """The benchmark's control-variate step (2^20 x 252, FP32, fused bumps), in
    the launch it times: sampled paths' arithmetic and control payoffs against
    the oracle, and beta and the estimate against oracle.control_variate on
    every dumped path (the kernel's FP32 payoffs, so the host arithmetic alone
    is compared) with the device control mean."""
    n, N, seed = 1 << 20, 252, 42
    opts = hm.Options(precision=hm.FP32, control_variate=hm.CONTROL_GEOMETRIC)
    r = ctx.price_greeks(PB.__dict__, hm.ASIAN_CALL, n, N, seed, opts)
    full = ctx.dump_paths(PB.__dict__, hm.ASIAN_CALL, n, N, seed, 0, n, opts).cpu().numpy()
    for first in (0, n // 2 + 4321, n - 300):
        a = oracle.simulate(PB, oracle.ASIAN_CALL, N, seed, first, 300, threads=8)[:, 3]
        g = oracle.simulate(PB, oracle.GEO_ASIAN_CALL, N, seed, first, 300, threads=8)[:, 3]
        close("pay", full[first:first + 300, 3], a, TOL[1], PB.S0)
        close("geo pay", full[first:first + 300, 15], g, TOL[1], PB.S0)
    est, se, beta = oracle.control_variate(full[:, 3], full[:, 15], r["cv_mean"])
    assert r["cv_beta"] == pytest.approx(beta, rel=1e-9)
    assert r["cv_price"][0] == pytest.approx(est, rel=1e-10)
    assert r["cv_price"][1] == pytest.approx(se, rel=1e-6)
