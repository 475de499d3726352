"""The 3D plane and axis-0 passes on axes that are no multiple of 32: rows and
columns past an axis's end read as zeros, and partial groups of four at rows'
and the field's end.  Products against the FP64 oracle at the tolerances of the
whole-tile shapes; steps and gradients against the three axis passes, which sum
in another order: eight products on either side, each value a sum of positive
terms over three axes of at most 130, so 130 x 3 x 2^-24 of it in FP32 and
3 x 2^-16 more in split BF16, and four times that after the adjoint."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_1502_06216_amd as jk
from workloads import small_case

from _util import banner, dev, energies, f32, host64, rel_l1

pytestmark = pytest.mark.gpu

GIBBS_TOL = {"fp32": 1e-6, "split_bf16": 2e-5}
PRODUCT = {"fp32": 390 * 2.0 ** -24, "split_bf16": 390 * 2.0 ** -24 + 3 * 2.0 ** -16}
SHAPES = [(16, 16, 16), (17, 33, 31), (45, 38, 51), (31, 127, 18), (130, 16, 66), (40, 100, 36), (64, 32, 33)]


@pytest.mark.parametrize("precision", ["fp32", "split_bf16"])
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("cells", [1.5, 5.0])
def test_product_matches_oracle(shape, cells, precision):
    banner(f"ragged planes {shape} {cells} {precision}")
    gamma = (cells / max(shape)) ** 2
    rng = np.random.default_rng(7)
    x = rng.uniform(0.0, 1.0, size=shape) * np.exp(rng.normal(0, 2, size=shape))
    ref = O.gibbs_apply(f32(x).astype(np.float64), gamma)
    # an aligned input, and one that starts a float later
    buf = torch.empty(x.size + 1, dtype=torch.float32, device="cuda")
    buf[1:] = dev(x).reshape(-1)
    for t in (dev(x), buf[1:].view(*shape)):
        y = jk.gibbs_apply(t, gamma, precision)
        assert rel_l1(host64(y), ref) <= GIBBS_TOL[precision]


@pytest.mark.parametrize("precision", ["fp32", "split_bf16"])
@pytest.mark.parametrize("kind", ["congestion", "entropy", "porous", "zero"])
@pytest.mark.parametrize("shape", [(45, 38, 51), (17, 100, 36)])
def test_step_and_gradient_match_axis_passes(shape, kind, precision):
    banner(f"ragged plane step {shape} {kind} {precision}")
    gamma = (3.0 / max(shape)) ** 2
    wl = small_case(shape, kind, seed=3, gamma=gamma, tau=2.5 * gamma, n_boxes=0)
    if kind == "porous":
        wl.density_scale = float(np.prod(shape))
    en, _ = energies(wl)
    out = []
    for planes in (True, False):
        kw = dict(precision=precision, planes=planes)
        p, st = jk.step(dev(wl.p0), en, wl.gamma, wl.tau, max_iters=4, check_every=2, **kw)
        _, _, ck = jk.flow(dev(wl.p0), en, wl.gamma, wl.tau, 1, max_iters=4, checkpoints=True, **kw)
        gw, gp = jk.backward(ck, [4], dev(np.ones(shape)), en, wl.gamma, wl.tau,
                             want_w=kind == "congestion", **kw)
        out.append((p, gw, gp, st))
    tol = 2 * 8 * PRODUCT[precision]
    a, b = out
    assert rel_l1(host64(a[0]), host64(b[0])) <= tol
    assert a[3]["iters"] == b[3]["iters"] == 4
    assert a[3]["mass"] == pytest.approx(b[3]["mass"], rel=tol)
    if kind in ("entropy", "zero"):   # no kinks
        assert rel_l1(host64(a[2]), host64(b[2])) <= 4 * tol
