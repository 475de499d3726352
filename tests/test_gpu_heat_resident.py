"""The resident heat kernel (the stored operator kept on chip for a step) against
the per-product form, which shares none of its code but the epilogue: operators
of few and of many tiles (with streamed ones), tolerance mode at several check
cadences, every energy."""
import time

import numpy as np
import pytest
import torch

import paper_1502_06216_amd as jk
from workloads import heat_room

from _util import banner, dev, energies, host64, rel_l1

pytestmark = pytest.mark.gpu

# float32 sums of the operator's entries on one side, the series rounded once
# on the other, over 25 iterations: as the heat flows against the oracle.
TOL = 1e-5


def _ops(wl):
    m = torch.from_numpy(np.ascontiguousarray(wl.mask.astype(np.uint8))).cuda()
    return [jk.HeatOperator(wl.shape, wl.gamma, wl.heat_L, mask=m, per_product=pp) for pp in (False, True)]


@pytest.mark.parametrize("shape", [(18, 24), (23, 23), (40, 41), (64, 50), (90, 84), (104, 103), (112, 110)])
def test_step_matches_the_solves(shape):
    banner(f"heat resident {shape}")
    wl = heat_room(*shape, seed=4)
    en, _ = energies(wl)
    ps = [op.step(dev(wl.p0), en, wl.tau, max_iters=25)[0] for op in _ops(wl)]
    err = rel_l1(host64(ps[0]), host64(ps[1]))
    print(f"[gpu-test] heat resident {shape}: {err:.2e}", flush=True)
    assert err <= TOL


@pytest.mark.parametrize("shape", [(108, 107), (121, 118)])
def test_product_of_an_operator_beyond_the_cache(shape):
    """Operators of less and more than the last-level cache holds, whose tiles a product streams."""
    banner(f"heat product {shape}")
    wl = heat_room(*shape, seed=4)
    x = dev(np.where(wl.mask, np.random.default_rng(8).uniform(size=shape), 0.0))
    a, b = [host64(op.apply(x)) for op in _ops(wl)]
    assert rel_l1(a, b) <= 1e-6      # float32 entries and sums, as in the products against the oracle
    assert not a[~wl.mask].any()


@pytest.mark.parametrize("ce", [1, 2, 7, 200])
def test_tolerance_mode(ce):
    banner(f"heat resident tolerance ce={ce}")
    wl = heat_room(30, 40, seed=5)
    en, _ = energies(wl)
    out = [op.flow(dev(wl.p0), en, wl.tau, 2, max_iters=60, tol=1e-5, check_every=ce) for op in _ops(wl)]
    for a, b in zip(out[0][1], out[1][1]):
        assert (a["iters"], a["stop"]) == (b["iters"], b["stop"])
        assert a["mass"] == pytest.approx(b["mass"], rel=1e-6)
    assert rel_l1(host64(out[0][0]), host64(out[1][0])) <= TOL
    if ce < 60:
        assert out[0][1][0]["stop"] == "tol"


@pytest.mark.parametrize("kind", ["zero", "entropy", "porous", "gen_entropy", "binary_congestion"])
def test_energies(kind):
    banner(f"heat resident {kind}")
    wl = heat_room(40, 36, seed=6, tau=2.5 * 10 / 40 ** 2)
    n = float(wl.N)
    en = jk.EnergySpec(kind=kind, coef_scalar=0.2, density_scale=n, m=1.5,
                       kappa_scalar=float(np.float32(wl.kappa_scalar)), w=dev(0.02 * wl.w))
    ps = [op.step(dev(wl.p0), en, wl.tau, max_iters=10)[0] for op in _ops(wl)]
    a, b = host64(ps[0]), host64(ps[1])
    if kind == "binary_congestion":   # a threshold: cells on it may differ
        assert (a != b).mean() < 0.01
    else:
        assert rel_l1(a, b) <= TOL


@pytest.mark.parametrize("shape", [(30, 40), (104, 103)])
@pytest.mark.parametrize("ce", [1, 2, 5])
def test_a_stop_returns_the_checked_iterate(shape, ce):
    """A step that stops by tolerance returns, bit for bit, the iterate whose violation was small enough, and one
    that does not runs to its cap; the checks change nothing else."""
    banner(f"heat resident stop {shape} ce={ce}")
    wl = heat_room(*shape, seed=5)
    en, _ = energies(wl)
    op = _ops(wl)[0]
    p, st = op.step(dev(wl.p0), en, wl.tau, max_iters=40, tol=1e-4, check_every=ce)
    assert st["stop"] == "tol" and st["iters"] % ce == 0 and 0 < st["iters"] < 40
    assert st["marginal_l1"] <= 1e-4
    k = st["iters"]
    q, sq = op.step(dev(wl.p0), en, wl.tau, max_iters=k)
    assert torch.equal(p, q)
    assert sq["marginal_l1"] == pytest.approx(st["marginal_l1"], rel=1e-3)
    if k > ce:      # the check before did not pass
        assert op.step(dev(wl.p0), en, wl.tau, max_iters=k - ce)[1]["marginal_l1"] > 1e-4
    p, st = op.step(dev(wl.p0), en, wl.tau, max_iters=k, tol=1e-30, check_every=ce)
    assert (st["stop"], st["iters"]) == ("cap", k) and torch.equal(p, q)


@pytest.mark.parametrize("ce", [1, 3, 50])
def test_a_value_that_is_not_finite_ends_the_step(ce):
    banner(f"heat resident not finite ce={ce}")
    n = 512
    x = np.arange(n) - 0.15 * n
    p = np.exp(-x * x / 8.0)
    p[p < 1e-6 * p.max()] = 0.0
    gamma = 10.0 / n ** 2
    op = jk.HeatOperator((1, n), gamma, 10)
    with pytest.raises(jk.JKOError):
        op.step(dev(p[None] / p.sum()), jk.EnergySpec(kind="entropy"), 10.0 * gamma, max_iters=100, tol=1e-6,
                check_every=ce)


def test_checks_cost_little():
    """64 x 64: a check after each of 60 iterations against none at all."""
    banner("heat resident check cost")
    wl = heat_room(64, 64, seed=5)
    en, _ = energies(wl)
    op = _ops(wl)[0]
    best = [np.inf, np.inf]
    for _ in range(30):
        for i, kw in enumerate((dict(), dict(tol=1e-30, check_every=1))):
            torch.cuda.synchronize()
            t = time.perf_counter()
            op.step(dev(wl.p0), en, wl.tau, max_iters=60, **kw)
            torch.cuda.synchronize()
            best[i] = min(best[i], 1e6 * (time.perf_counter() - t))
    print(f"[gpu-test] heat resident 64 x 64: {best[0]:.0f} us, with checks {best[1]:.0f}", flush=True)
    assert best[1] <= 2.0 * best[0]
