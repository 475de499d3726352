"""1D grids on the tile kernels, one column of cells: the attraction's two
couplings (whatever the kernel's width: the axis that stacks them never mixes
them) against the axis passes.  Eight products on either side, each a sum of at most 1024
positive terms: 16 x 1024 x 2^-24 in FP32, and 16 x 3 x 2^-16 more split."""
import pytest
import torch

import paper_1502_06216_amd as jk
from workloads import gaussian_bumps

from _util import banner, dev, f32, host64, rel_l1

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
