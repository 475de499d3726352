"""The resident heat kernel (the stored operator kept on chip for a step) against
the per-product form, which shares none of its code but the epilogue: operators
of few and of many tiles (with streamed ones), tolerance mode at several check
cadences, every energy."""
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
