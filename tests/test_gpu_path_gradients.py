"""Gradients on the paths of 1D grids (the tile kernels, as one column of cells:
resident and as launches) and of ragged 3D grids (the plane and axis-0 passes),
in the initial density and in the energy's field, against float64 autograd
through the oracle's iteration (1e-3, as every gradient) and against the axis
passes.  The crowd's capacity keeps away from its kinks: every cell is either
far under it or far over it in all iterations."""
import numpy as np
import pytest
import torch

import paper_1502_06216_amd as jk
from oracle.grad import loss_and_grads
from workloads import small_case

from _util import banner, dev, energies, f32, host64

pytestmark = pytest.mark.gpu

GRAD_TOL = 1e-3
# The same sums in another order: 2 x 6 iterations of two products forward and
# two back, each a sum of at most 3 x 500 positive terms, in FP32 of the order of
# 2^-24 sqrt(1500) a product; 2^-16 more split.
SUM_TOL = {"fp32": 48 * 40 * 2.0 ** -24, "split_bf16": 48 * (40 * 2.0 ** -24 + 2.0 ** -16)}
SHAPES = [(40,), (130,), (467,), (17, 33, 31), (33, 18, 40)]


def _rel(x, ref):
    return float(np.linalg.norm(np.asarray(x, np.float64) - ref) / np.linalg.norm(ref))


def _case(kind, shape):
    gamma = (3.0 / max(shape)) ** 2
    wl = small_case(shape, "entropy" if kind == "gen_entropy" else kind, seed=4, gamma=gamma, tau=2.5 * gamma, n_boxes=0)
    rng = np.random.default_rng(11)
    wl.p0 = rng.uniform(0.5, 1.5, shape)
    wl.p0 /= wl.p0.sum()
    if kind == "gen_entropy":
        wl.kind, wl.density_scale = kind, float(wl.N)
        wl.coef, wl.m_field = 0.2 + 0.3 * rng.uniform(size=shape), 1.0 + rng.uniform(size=shape)
    if kind == "congestion":
        wl.w = 0.3 * rng.uniform(size=shape)
        over = rng.uniform(size=shape) < 0.2
        wl.kappa = np.where(over, 0.02, 50.0) / wl.N
    return wl


@pytest.mark.parametrize("precision", ["fp32", "split_bf16"])
@pytest.mark.parametrize("kind", ["congestion", "entropy", "gen_entropy", "zero"])
@pytest.mark.parametrize("shape", SHAPES)
def test_gradients(shape, kind, precision):
    banner(f"path gradients {shape} {kind} {precision}")
    wl = _case(kind, shape)
    g_en, o_en = energies(wl)
    target = np.random.default_rng(9).uniform(size=shape)
    target /= target.sum()
    iters = [6, 6]
    want_w = kind in ("congestion", "gen_entropy")
    out = []
    for kw in (dict(), dict(resident=False), dict(planes=False)):
        kw["precision"] = precision
        pT, _, ck = jk.flow(dev(wl.p0), g_en, wl.gamma, wl.tau, 2, max_iters=6, checkpoints=True, **kw)
        dL = 2.0 * (pT - dev(target))
        gw, gp = jk.backward(ck, iters, dL.contiguous(), g_en, wl.gamma, wl.tau, want_w=want_w, **kw)
        out.append((host64(pT), host64(gp), host64(gw) if want_w else None))
    coef = o_en._coef(shape) if kind in ("entropy", "gen_entropy") else None
    m = o_en._m(shape) if kind == "gen_entropy" else None
    w = f32(wl.w).astype(np.float64) if kind == "congestion" else np.zeros(shape)
    kappa = f32(wl.kappa).astype(np.float64) if kind == "congestion" else np.inf
    _, rw, rp, _ = loss_and_grads(f32(wl.p0).astype(np.float64), w, kappa, wl.gamma, wl.tau, iters, target, kind=kind,
                                  coef=coef, m=m, density_scale=wl.density_scale)
    for (p, gp, gw), name in zip(out, ("default", "launches", "axis passes")):
        ep, ew = _rel(gp, rp), _rel(gw, rw) if want_w else 0.0
        print(f"[gpu-test] {shape} {kind} {precision} {name}: dL/dp0 {ep:.1e}, dL/dfield {ew:.1e}", flush=True)
        assert ep <= GRAD_TOL and ew <= GRAD_TOL
        assert _rel(p, out[2][0]) <= SUM_TOL[precision]
        assert _rel(gp, out[2][1]) <= 4 * SUM_TOL[precision]
        if want_w:
            assert _rel(gw, out[2][2]) <= 4 * SUM_TOL[precision]
