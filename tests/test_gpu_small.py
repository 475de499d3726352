"""The one-block form of the resident 2D kernel (grids of at most 16 tiles of
16 x 16) against the launch-per-application path: the same tile arithmetic and
order of sums, so the same bits, on grids at the edges of its tiles, chunks and
selection (the last two are beyond it in FP32)."""
import time

import numpy as np
import pytest
import torch

import paper_1502_06216_amd as jk
from workloads import small_case

from _util import banner, dev, energies, host64

pytestmark = pytest.mark.gpu

KEYS = ("iters", "absorptions", "stop", "status", "marginal_l1", "mass", "max_abs_log_a", "max_abs_log_b")


@pytest.mark.parametrize("precision", ["fp32", "split_bf16"])
@pytest.mark.parametrize("shape,width", [((16, 16), 2.0), ((15, 7), 2.0), ((17, 33), 3.0), ((1, 250), 3.0),
                                         ((250, 1), 3.0), ((64, 64), 1.4), ((48, 63), 4.0), ((64, 64), 5.0),
                                         ((16, 256), 6.0)])
def test_step_and_gradient_same_bits(shape, width, precision):
    banner(f"small grid {shape} width={width} {precision}")
    gamma = (width / max(shape)) ** 2
    wl = small_case(shape, "congestion", seed=6, gamma=gamma, tau=2.5 * gamma, n_boxes=0)
    en, _ = energies(wl)
    out = []
    for resident in (True, False):
        kw = dict(precision=precision, resident=resident)
        p, st = jk.step(dev(wl.p0), en, wl.gamma, wl.tau, max_iters=23, check_every=4, absorb_threshold=60.0, **kw)
        _, _, ck = jk.flow(dev(wl.p0), en, wl.gamma, wl.tau, 2, max_iters=5, checkpoints=True, **kw)
        gw, gp = jk.backward(ck, [5, 5], dev(wl.w), en, wl.gamma, wl.tau, **kw)
        out.append(((p, ck, gw, gp), st))
    for a, b in zip(out[0][0], out[1][0]):
        assert torch.equal(a, b), f"max |diff| {float((a - b).abs().max()):.3e}"
    for k in KEYS:
        assert out[0][1][k] == out[1][1][k], k


@pytest.mark.parametrize("precision", ["fp32", "split_bf16"])
@pytest.mark.parametrize("shape", [(64, 64), (48, 40), (33, 61), (200,)])
def test_values_that_are_not_finite_stay_where_they_are(shape, precision):
    """An infinite scaling reaches the tiles whose halo holds its cell, and no other: the one-block kernel's rows
    go on past a tile's halo, where the tile kernel has zeros (every cell the same, NaN for NaN)."""
    banner(f"small non-finite {shape} {precision}")
    n = max(shape)
    gamma = (1.2 / n) ** 2
    rng = np.random.default_rng(5)
    p = dev(rng.uniform(0.5, 1.5, shape) / np.prod(shape))
    for cell in rng.choice(int(np.prod(shape)), 12, replace=False):
        w, kappa = np.zeros(shape), np.full(shape, 2.0)
        w.flat[cell], kappa.flat[cell] = -1e30, np.inf     # p = s exp(-sigma w) = inf there, and a = p / s
        en = jk.EnergySpec(kind="congestion", w=dev(w), kappa=dev(kappa))
        got, ref = [host64(jk.step(p, en, gamma, 4 * gamma, max_iters=2, precision=precision, with_stats=False,
                                   resident=r)[0]) for r in (True, False)]
        assert not np.isfinite(ref).all()
        np.testing.assert_array_equal(got, ref)


def _us(shapes, kind, precision, **kw):
    """The fastest of several steps of 50 iterations on each of the shapes, taken in turn, in microseconds."""
    runs = []
    for shape in shapes:
        p = np.random.default_rng(3).uniform(0.5, 1.5, shape)
        p = dev(p / p.sum())
        en = jk.EnergySpec(kind=kind, kappa_scalar=float(p.max()), m=1.5, density_scale=float(np.prod(shape)))
        runs.append((p, en, (3.0 / max(shape)) ** 2))
    best = [np.inf] * len(shapes)
    for _ in range(30):
        for i, (p, en, gamma) in enumerate(runs):
            torch.cuda.synchronize()
            t = time.perf_counter()
            jk.step(p, en, gamma, 2 * gamma, max_iters=50, precision=precision, **kw)
            torch.cuda.synchronize()
            best[i] = min(best[i], 1e6 * (time.perf_counter() - t))
    return best


@pytest.mark.parametrize("kind,kw", [("gen_entropy", {}), ("porous", {}), ("congestion", dict(tol=1e-30, check_every=1))])
def test_a_smaller_grid_is_not_slower(kind, kw):
    """16 tiles against the 20 of a grid that only the tile kernel takes (a fifth more is the clock's)."""
    small, large = _us(((64, 64), (64, 80)), kind, "split_bf16", **kw)
    banner(f"small {kind} {kw}: 64 x 64 {small:.0f} us, 64 x 80 {large:.0f} us")
    assert small <= 1.2 * large
