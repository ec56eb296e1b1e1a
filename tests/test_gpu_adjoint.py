"""GPU parity of the adjoint (reverse-mode) kernel and of plain bump-and-revalue.

Per-path payoffs and derivatives from heston_adjoint_backward against the
oracle's forward-mode derivatives (which are pinned to finite differences in
test_oracle.py): |gpu - oracle| <= max(tol max(|oracle|, floor), 4 x spread),
tol 1e-12 in FP64 and 1e-5 in FP32; floors S0 for the payoff, d/dv0,
d/dsigma and d/drho, 1 for d/dS0, K T for d/dr, S0 T for d/dkappa and
d/dtheta.  The spread is how far Monte-Carlo-arithmetic evaluations of the
same derivatives in the kernel's precision land from the oracle on that path
(tests/tangent_binary32.py); it exceeds the plain bar only where the variance
comes close to zero and the scheme amplifies rounding, and CPU tests
(test_adjoint_conditioning.py) show both that no evaluation in that precision
meets the plain bar there and that the bar covers independent evaluations.
Paths whose averaged price lies within 1e3 tol K of the strike may switch the
payoff indicator and are exempt.
"""
import math

import numpy as np
import pytest

import oracle
import tangent_binary32 as tb
from workloads import BASE, PAPER

pytestmark = pytest.mark.gpu

PB = oracle.Params(**BASE)
PP = oracle.Params(**PAPER)
TOL = {0: 1e-12, 1: 1e-5}


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


def adjoint_per_path(hm, ctx, p, opt_type, n, N, seed, prec, every, scheme=0, fixings=None,
                     dprice=1.0):
    import torch
    opts = hm.Options(precision=prec, scheme=scheme, greeks=hm.GREEKS_PATHWISE, fixings=fixings)
    ck = torch.empty(hm.ckpt_bytes(n, N, every, prec), dtype=torch.uint8, device="cuda:0")
    price, _ = ctx.adjoint_forward(p.__dict__, opt_type, n, N, seed, ck, every, opts)
    pp = torch.empty((n, 8), dtype=torch.float64, device="cuda:0")
    grads, _ = ctx.adjoint_backward(p.__dict__, opt_type, n, N, seed, ck, every, dprice, opts,
                                    per_path=pp)
    return price, grads, pp.cpu().numpy()


def check_against_tangent(d, p, opt_type, N, seed, first, n, prec, scheme, fixings):
    """Per-path bars of the module docstring; under QE (scheme 2) paths whose
    branch margin lies below 1e-9 (FP64) or 1e-4 (FP32) may take the other
    branch in the other precision and are exempt (at most 3% of them)."""
    tol = TOL[prec]
    mode = {0: oracle.FULL_TRUNC, 1: oracle.ABSORB, 2: oracle.QE}[scheme]
    tan = oracle.tangent(p, opt_type, N, seed, first, n, mode, fixings, threads=8)
    rec = oracle.simulate(p, opt_type, N, seed, first, n, mode, fixings, threads=8)
    near = np.abs(rec[:, 2] - p.K) < 1e3 * tol * p.K
    if scheme == 2:
        close = tan[:, 8] < (1e-9 if prec == 0 else 1e-4)
        assert close.mean() < 0.03, close.mean()
        near |= close
    bar = tb.bars(p, opt_type, N, seed, first, n, tan, mode, fixings,
                  np.float64 if prec == 0 else np.float32)
    names = ["pay", "S0", "v0", "r", "kappa", "theta", "sigma", "rho"]
    err = np.abs(d[:, :8] - tan[:, :8]) / bar
    for k in range(8):
        bad = (err[:, k] > 1.0) & ~near
        assert not bad.any(), (names[k], int(bad.sum()), float(err[bad, k].max()),
                               int(np.argmax(np.where(bad, err[:, k], 0))))
    return tan


@pytest.mark.parametrize("opt_type", [0, 1, 2, 3])
@pytest.mark.parametrize("scheme", [0, 1])
def test_adjoint_fp64_matches_tangent(hm, ctx, opt_type, scheme):
    n, N, seed = 2000 + 13, 37, 11
    p = PP if scheme == 1 else PB.replace(sigma=0.6)
    fix = (3, 10, 20, 37) if opt_type >= 2 else None
    price, grads, d = adjoint_per_path(hm, ctx, p, opt_type, n, N, seed, 0, 8, scheme, fix)
    check_against_tangent(d, p, opt_type, N, seed, 0, n, 0, scheme, fix)
    for k in range(7):
        m, se = oracle.mean_se(d[:, 1 + k])
        assert grads[k][0] == pytest.approx(m, rel=1e-10, abs=1e-12)
        assert grads[k][1] == pytest.approx(se, rel=1e-6, abs=1e-12)


@pytest.mark.parametrize("scheme", [0, 1])
@pytest.mark.parametrize("N,every,fix", [
    (1, 8, (1,)), (31, 8, (31,)), (32, 16, (1, 32)), (33, 8, (31, 32, 33)),
    (65, 16, (15, 16, 17, 31, 32, 48, 63, 64, 65)), (65, 16, None)])
def test_adjoint_fixing_flags_of_a_segment(hm, ctx, N, every, fix, scheme):
    """Fixing dates at the edges of the flag words and of the checkpoint
    segments, sparse and at every step, with an odd last step."""
    _, _, d = adjoint_per_path(hm, ctx, PB, 2, 300, N, 3, 0, every, scheme, fix)
    check_against_tangent(d, PB, 2, N, 3, 0, 300, 0, scheme, fix)


@pytest.mark.parametrize("scheme", [0, 1])
@pytest.mark.parametrize("opt_type", [1, 3])
def test_fp64_vanishing_price_under_an_enormous_variance(hm, ctx, opt_type, scheme):
    """v0 = 1e50: e^x is 0 at every date, a put pays K, and only r moves its
    price, in the adjoint's two passes and in a batch."""
    p = PB.replace(v0=1e50)
    price, grads, d = adjoint_per_path(hm, ctx, p, opt_type, 300, 8, 3, 0, 8, scheme)
    pay = p.K * math.exp(-p.r * p.T)
    want = [0.0, 0.0, -p.T * pay, 0.0, 0.0, 0.0, 0.0]
    assert price[0] == pytest.approx(pay, rel=1e-14)
    assert [g[0] for g in grads] == pytest.approx(want, rel=1e-14)
    assert d[:, 0] == pytest.approx(pay, rel=1e-14)
    rq = [dict(params=p.__dict__, type=opt_type, n_steps=8, n_paths=300, seed=3, want=w)
          for w in (hm.WANT_PATHWISE, hm.WANT_ADJOINT)]
    res, _ = ctx.price_batch(rq, hm.Options(scheme=scheme, greeks=hm.GREEKS_PATHWISE))
    for r in res:
        assert r["price"][0] == pytest.approx(pay, rel=1e-14)
        assert r["pw_rho"][0] == pytest.approx(want[2], rel=1e-14)
    assert [a[0] for a in res[1]["adj"]] == pytest.approx(want, rel=1e-14)


@pytest.mark.parametrize("every", [8, 16])
@pytest.mark.parametrize("opt_type", [0, 2])
def test_adjoint_fp32_matches_tangent(hm, ctx, every, opt_type):
    n, N, seed = 4096 + 100, 100, 5
    price, grads, d = adjoint_per_path(hm, ctx, PB, opt_type, n, N, seed, 1, every)
    check_against_tangent(d, PB, opt_type, N, seed, 0, n, 1, 0, None)


def test_adjoint_fp32_feller_violated_matches_tangent(hm, ctx):
    """FP32 at vol of vol 0.6 (Feller violated): the variance comes close to
    zero on many paths, where the bar is set by the binary32 spread."""
    p, n, N, seed = PB.replace(sigma=0.6), 4096 + 100, 100, 5
    for opt_type in (0, 2):
        _, _, d = adjoint_per_path(hm, ctx, p, opt_type, n, N, seed, 1, 16)
        check_against_tangent(d, p, opt_type, N, seed, 0, n, 1, 0, None)


QE_PARAMS = {"base": PB, "feller-violated": PB.replace(sigma=0.9, kappa=1.0, theta=0.05)}


@pytest.mark.parametrize("opt_type", [0, 1, 2, 3])
@pytest.mark.parametrize("case", list(QE_PARAMS))
def test_adjoint_qe_fp64_matches_tangent(hm, ctx, opt_type, case):
    """Andersen's QE scheme (the paper's Future Work) in the adjoint: per-path
    payoffs and derivatives against the oracle's QE tangent, FP64, with a
    ragged path count, an odd step count and explicit Asian fixings."""
    p, n, N, seed = QE_PARAMS[case], 2013, 37, 11
    fix = (3, 10, 20, 37) if opt_type >= 2 else None
    price, grads, d = adjoint_per_path(hm, ctx, p, opt_type, n, N, seed, 0, 8, hm.QE, fix)
    tan = check_against_tangent(d, p, opt_type, N, seed, 0, n, 0, 2, fix)
    for k in range(7):
        m, se = oracle.mean_se(d[:, 1 + k])
        assert grads[k][0] == pytest.approx(m, rel=1e-10, abs=1e-12)
    assert price[0] == pytest.approx(tan[:, 0].mean(), rel=1e-10, abs=1e-12)


@pytest.mark.parametrize("every", [8, 16])
@pytest.mark.parametrize("case", list(QE_PARAMS))
def test_adjoint_qe_fp32_matches_tangent(hm, ctx, every, case):
    p, n, N, seed = QE_PARAMS[case], 4096 + 100, 100, 5
    for opt_type in (0, 2):
        _, _, d = adjoint_per_path(hm, ctx, p, opt_type, n, N, seed, 1, every, hm.QE)
        check_against_tangent(d, p, opt_type, N, seed, 0, n, 1, 2, None)


def test_adjoint_qe_against_analytic(hm, ctx):
    """FP32 QE, 2^21 paths: the seven European-call sensitivities at 200 steps
    within 3 SE of the characteristic-function values plus the run's own
    discretisation allowance |g(200 steps) - g(100 steps)|."""
    from oracle import analytic
    g = analytic.heston_call_greeks(PB)
    _, g1, _ = adjoint_per_path(hm, ctx, PB, 0, 1 << 21, 100, 42, 1, 16, hm.QE)
    _, g2, _ = adjoint_per_path(hm, ctx, PB, 0, 1 << 21, 200, 43, 1, 16, hm.QE)
    ref = [g["delta"], g["vega"], g["rho"], g["d_kappa"], g["d_theta"], g["d_sigma"], g["d_rho"]]
    for k in range(7):
        allow = 3 * g2[k][1] + abs(g2[k][0] - g1[k][0])
        assert abs(g2[k][0] - ref[k]) < allow, (k, g2[k], g1[k], ref[k])


@pytest.mark.parametrize("opt_type,scheme", [(0, 0), (2, 1), (2, 2)])
def test_fp32_adjoint_is_the_same_in_small_and_large_launches(hm, ctx, opt_type, scheme):
    """At most one wave per SIMD (65536 paths) and one block more: other builds
    of the kernels, the same derivatives of each path, bit for bit; and the same
    option alone in a batch and beside a large one."""
    d = [adjoint_per_path(hm, ctx, PB, opt_type, n, 9, 5, 1, 8, scheme)[2] for n in (65536, 65792)]
    assert np.array_equal(d[0], d[1][:65536])
    opts = hm.Options(precision=hm.FP32, scheme=scheme, greeks=hm.GREEKS_PATHWISE)
    rq = [dict(params=PB.__dict__, type=opt_type, n_steps=9, n_paths=n, seed=5, want=hm.WANT_ADJOINT)
          for n in (8192, 1 << 18)]
    alone, beside = (ctx.price_batch(r, opts)[0][0] for r in (rq[:1], rq))
    assert alone["price"] == beside["price"] and alone["adj"] == beside["adj"]


def test_adjoint_seed_gradient_scales(hm, ctx):
    n, N = 1000, 20
    _, g1, d1 = adjoint_per_path(hm, ctx, PB, 0, n, N, 3, 0, 8)
    _, g2, d2 = adjoint_per_path(hm, ctx, PB, 0, n, N, 3, 0, 8, dprice=-2.5)
    assert np.allclose(d2[:, 1:], -2.5 * d1[:, 1:], rtol=1e-15, atol=0)
    assert np.allclose(d2[:, 0], d1[:, 0])


def test_adjoint_S0_and_r_equal_pathwise_estimators(hm, ctx):
    """d/dS0 and d/dr of the adjoint are the paper's pathwise Delta and Rho."""
    n, N, seed = 5000, 64, 21
    for opt_type in (0, 1, 2, 3):
        _, _, d = adjoint_per_path(hm, ctx, PB, opt_type, n, N, seed, 0, 16)
        dump = ctx.dump_paths(PB.__dict__, opt_type, n, N, seed, 0, n,
                              hm.Options(greeks=hm.GREEKS_PATHWISE)).cpu().numpy()
        assert np.allclose(d[:, 1], dump[:, 4], rtol=1e-12, atol=1e-14)
        assert np.allclose(d[:, 3], dump[:, 5], rtol=1e-11, atol=1e-11)


def test_adjoint_large_sampled(hm, ctx):
    """The 2^22-path x 365-step FP32 adjoint (checkpoints every 16 steps), in the
    configuration the benchmark times: sampled windows against the oracle's
    derivatives, and the reduced gradients against the per-path values."""
    import torch
    n, N, seed = 1 << 22, 365, 42
    for opt_type in (0, 2):
        price, grads, d = adjoint_per_path(hm, ctx, PB, opt_type, n, N, seed, 1, 16)
        for first in (0, n // 3, n - 600):
            check_against_tangent(d[first:first + 600], PB, opt_type, N, seed, first, 600, 1, 0,
                                  None)
        for k in range(7):
            m, se = oracle.mean_se(d[:, 1 + k])
            assert grads[k][0] == pytest.approx(m, rel=1e-9, abs=1e-12)
        del d
        torch.cuda.empty_cache()


def test_adjoint_qe_large_sampled(hm, ctx):
    """QE at the adjoint benchmark's size (2^22 paths x 365 steps, FP32,
    checkpoints every 16 steps): sampled windows against the oracle's QE
    tangent under the QE bars, and the reduced gradients against the per-path
    values."""
    import torch
    n, N, seed = 1 << 22, 365, 42
    for opt_type in (0, 2):
        price, grads, d = adjoint_per_path(hm, ctx, PB, opt_type, n, N, seed, 1, 16, hm.QE)
        for first in (0, n // 3, n - 600):
            check_against_tangent(d[first:first + 600], PB, opt_type, N, seed, first, 600, 1, 2,
                                  None)
        for k in range(7):
            m, se = oracle.mean_se(d[:, 1 + k])
            assert grads[k][0] == pytest.approx(m, rel=1e-9, abs=1e-12)
        del d
        torch.cuda.empty_cache()


def test_adjoint_against_analytic(hm, ctx):
    """FP32, 2^21 paths: the seven European-call sensitivities at 400 steps
    within 3 SE of the characteristic-function values, plus the discretisation
    allowance the run itself shows, |g(400 steps) - g(200 steps)| (the scheme's
    weak error is first order, so halving the step halves the bias)."""
    from oracle import analytic
    g = analytic.heston_call_greeks(PB)
    _, g2, _ = adjoint_per_path(hm, ctx, PB, 0, 1 << 21, 200, 42, 1, 16)
    _, g4, _ = adjoint_per_path(hm, ctx, PB, 0, 1 << 21, 400, 43, 1, 16)
    ref = [g["delta"], g["vega"], g["rho"], g["d_kappa"], g["d_theta"], g["d_sigma"], g["d_rho"]]
    for k in range(7):
        allow = 3 * g4[k][1] + abs(g4[k][0] - g2[k][0])
        assert abs(g4[k][0] - ref[k]) < allow, (k, g4[k], g2[k], ref[k])


def test_autograd_function(hm, ctx):
    import torch
    from paper_2309_10477_amd.autograd import AdjointSpec, HestonAdjoint
    theta = torch.tensor([PB.S0, PB.v0, PB.r, PB.kappa, PB.theta, PB.sigma, PB.rho],
                         dtype=torch.float64, requires_grad=True)
    spec = AdjointSpec(K=PB.K, T=PB.T, opt_type=2, n_paths=20000, n_steps=50, seed=4,
                       precision=hm.FP64, every=8, ctx=ctx)
    price = HestonAdjoint.apply(theta, spec)
    (3.0 * price).backward()
    n, N = 20000, 50
    _, grads, d = adjoint_per_path(hm, ctx, PB, 2, n, N, 4, 0, 8)
    assert float(price) == pytest.approx(d[:, 0].mean(), rel=1e-12)
    assert np.allclose(theta.grad.numpy(), 3.0 * np.array([v for v, _ in grads]), rtol=1e-12)


def test_invalid_adjoint_requests(hm, ctx):
    import torch
    ck = torch.empty(16, dtype=torch.uint8, device="cuda:0")
    with pytest.raises(hm.HestonError):
        ctx.adjoint_forward(BASE, 0, 1000, 10, 1, ck, 16)          # buffer too small
    ck = torch.empty(hm.ckpt_bytes(1000, 10, 16, hm.FP32), dtype=torch.uint8, device="cuda:0")
    with pytest.raises(hm.HestonError):
        ctx.adjoint_forward(BASE, 0, 1000, 10, 1, ck, 12)          # interval
    with pytest.raises(hm.HestonError):
        ctx.adjoint_forward(dict(BASE, rho=1.0), 0, 1000, 10, 1, ck, 16)


# ---------------------------------------------------------------------------
# Plain bump-and-revalue (nine independent revaluations)

def test_plain_bumps_match_oracle_fp64(hm, ctx):
    n, N, seed = 10_000, 100, 42
    r = ctx.price_greeks(PB.__dict__, hm.EURO_CALL, n, N, seed,
                         hm.Options(greeks=hm.GREEKS_PATHWISE | hm.GREEKS_BUMP_PLAIN))
    ref = oracle.price_greeks(PB, oracle.EURO_CALL, n, N, seed, threads=8)
    for k, (v, se) in ref.items():
        assert r[k][0] == pytest.approx(v, rel=1e-10, abs=1e-11), k
        assert r[k][1] == pytest.approx(se, rel=1e-6, abs=1e-12), k


def test_plain_and_fused_bumps_agree_fp32_asian(hm, ctx):
    n, N, seed = 1 << 16, 252, 42
    a = ctx.price_greeks(PB.__dict__, hm.ASIAN_CALL, n, N, seed,
                         hm.Options(precision=hm.FP32))
    b = ctx.price_greeks(PB.__dict__, hm.ASIAN_CALL, n, N, seed,
                         hm.Options(precision=hm.FP32, greeks=hm.GREEKS_PATHWISE |
                                    hm.GREEKS_BUMP_PLAIN))
    for k in ("price", "pw_delta", "pw_rho"):
        assert a[k] == b[k], k
    # the fused kernel evaluates the S0 and r scenarios algebraically from the
    # FP32 state; the plain launches re-simulate them in FP32
    for k in ("delta", "gamma", "vega", "rho", "theta"):
        assert abs(a[k][0] - b[k][0]) < 0.05 * a[k][1] + 1e-6 * abs(a[k][0]), (k, a[k], b[k])


def test_bump_revalue_seven_parameters(hm, ctx):
    """General plain bumps of the seven adjoint inputs against the oracle's
    central differences on the same paths (FP64)."""
    n, N, seed = 3000, 30, 8
    names = ["S0", "v0", "r", "kappa", "theta", "sigma", "rho"]
    idx = [hm.P_S0, hm.P_V0, hm.P_R, hm.P_KAPPA, hm.P_THETA, hm.P_SIGMA, hm.P_RHO]
    bumps = [(i, 0, 1e-3) for i in idx]
    r = ctx.bump_revalue(PB.__dict__, hm.ASIAN_PUT, n, N, seed, bumps)
    base = oracle.simulate(PB, oracle.ASIAN_PUT, N, seed, 0, n)[:, 3]
    assert r["price"][0] == pytest.approx(base.mean(), rel=1e-12)
    for k, name in enumerate(names):
        up = oracle.simulate(PB.replace(**{name: getattr(PB, name) + 1e-3}), oracle.ASIAN_PUT, N,
                             seed, 0, n)[:, 3]
        dn = oracle.simulate(PB.replace(**{name: getattr(PB, name) - 1e-3}), oracle.ASIAN_PUT, N,
                             seed, 0, n)[:, 3]
        m, se = oracle.mean_se((up - dn) / 2e-3)
        assert r["first"][k][0] == pytest.approx(m, rel=1e-8, abs=1e-9), name
        m2, _ = oracle.mean_se((up - 2 * base + dn) / 1e-6)
        assert r["second"][k][0] == pytest.approx(m2, rel=1e-5, abs=1e-4), name
