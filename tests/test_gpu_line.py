"""1D grids on the tile kernels, one column of cells: the attraction's two
couplings (whatever the kernel's width: the axis that stacks them never mixes
them), and steps, flows and gradients, against the axis passes.  Eight products on either side, each a sum of at most 1024
positive terms: 16 x 1024 x 2^-24 in FP32, and 16 x 3 x 2^-16 more split."""
import numpy as np
import pytest
import torch

import paper_1502_06216_amd as jk
import oracle as O
from workloads import gaussian_bumps, small_case

from _util import banner, dev, energies, f32, host64, rel_l1

pytestmark = pytest.mark.gpu

TOL = {"fp32": 16 * 1024 * 2.0 ** -24, "split_bf16": 16 * 1024 * 2.0 ** -24 + 48 * 2.0 ** -16}


@pytest.mark.parametrize("precision", ["fp32", "split_bf16"])
@pytest.mark.parametrize("n,gamma", [(40, 0.02), (96, 1e-3), (1000, 1.6e-5), (64, 0.3)])
def test_attraction_matches_axis_passes(n, gamma, precision):
    banner(f"line attraction {n} {gamma} {precision}")
    p = gaussian_bumps((n, 1), [(0.35, 0.5)], 0.1, [1.0]).reshape(n) + 1e-3
    r = gaussian_bumps((n, 1), [(0.6, 0.5)], 0.1, [1.0]).reshape(n) + 1e-3
    p, r = f32(p / p.sum()), f32(r / r.sum())
    en = jk.EnergySpec(kind="attraction", target=dev(r), kappa_scalar=float(4 * p.max()))
    a, b = (jk.step(dev(p), en, gamma, 0.5, max_iters=4, precision=precision, planes=planes)[0]
            for planes in (True, False))
    assert torch.isfinite(a).all()
    assert rel_l1(host64(a), host64(b)) <= TOL[precision]


@pytest.mark.parametrize("precision", ["fp32", "split_bf16"])
@pytest.mark.parametrize("n,cells", [(1, 1.0), (3, 1.0), (16, 3.0), (17, 3.0), (250, 5.0), (257, 4.0), (467, 3.0),
                                     (1000, 1.5), (1024, 5.0), (1024, 6.5), (1023, 9.0)])
def test_product_and_step(n, cells, precision):
    banner(f"line {n} {cells} {precision}")
    gamma = (cells / n) ** 2
    rng = np.random.default_rng(4)
    x = f32(rng.uniform(0.1, 1.0, size=n))
    y = jk.gibbs_apply(dev(x), gamma, precision)
    assert rel_l1(host64(y), O.gibbs_apply(x.astype(np.float64), gamma)) <= {"fp32": 1e-6, "split_bf16": 2e-5}[precision]
    wl = small_case((n,), "congestion", seed=2, gamma=gamma, tau=2.5 * gamma, n_boxes=0)
    en, _ = energies(wl)
    out = []
    for kw in (dict(), dict(resident=False), dict(planes=False)):
        kw["precision"] = precision
        p, st = jk.step(dev(wl.p0), en, gamma, wl.tau, max_iters=4, check_every=2, **kw)
        _, _, ck = jk.flow(dev(wl.p0), en, gamma, wl.tau, 1, max_iters=4, checkpoints=True, **kw)
        gw, gp = jk.backward(ck, [4], dev(np.ones(n)), en, gamma, wl.tau, **kw)
        out.append((p, st, gw, gp))
    a, b, c = out
    for i in (0, 2, 3):
        assert torch.equal(a[i], b[i])
    assert a[1] == b[1]
    assert a[1]["iters"] == c[1]["iters"]
    assert rel_l1(host64(a[0]), host64(c[0])) <= TOL[precision]
