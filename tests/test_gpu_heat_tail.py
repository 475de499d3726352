"""The far tail of the heat kernel.  The scaling iteration divides by the
operator's products, so its entries count relative to their own size down to
float32's smallest normal value, not to the product's norm: columns entry by
entry, and steps of a localised density whose far cells live on that tail,
against the oracle's LU solves (an M-matrix's solves add positive terms only,
so each entry is accurate to FP64 rounding)."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_1502_06216_amd as jk

from _util import banner, host64, rel_l1

pytestmark = pytest.mark.gpu

# An entry is the series' value rounded to float32 once (6e-8); the series is
# cut 21 decades per L below the norm, at most 46 (stored) or 85, and six
# decades above the cut what it drops is below 1e-8 of an entry.
TOL_ENTRY = 1e-6
# the flows' bound: float32 scalings and prox against FP64
TOL_FLOW = 1e-5


@pytest.mark.parametrize("per_product", [False, True])
@pytest.mark.parametrize("shape,src", [((1, 300), (0, 3)), ((90, 1), (70, 0)), ((100, 84), (30, 40))])
@pytest.mark.parametrize("L,nu", [(1, 1.0), (2, 1.0), (3, 0.1), (10, 0.1), (10, 1.0), (10, 9.0), (20, 1.0)])
def test_columns_keep_their_tail(shape, src, L, nu, per_product):
    banner(f"heat tail {shape} L={L} nu={nu} per_product={per_product}")
    rng = np.random.default_rng(1)
    mask = np.ones(shape, bool) if 1 in shape else rng.uniform(size=shape) < 0.85
    mask[src] = True
    gamma = nu * L / max(shape) ** 2
    x = np.zeros(shape, np.float32)
    x[src] = 1.0
    ref = O.HeatKernel(mask, gamma, L)(x.astype(np.float64))
    op = jk.HeatOperator(shape, gamma, L, mask=torch.from_numpy(mask.astype(np.uint8)).cuda(), per_product=per_product)
    y = host64(op.apply(torch.from_numpy(x).cuda()))
    seen = ref >= max(1e-37, 10.0 ** (6 - 21 * L))
    err = float((np.abs(y - ref)[seen] / ref[seen]).max())
    print(f"[gpu-test] heat tail {shape} L={L}: {int(seen.sum())} entries down to {ref[seen].min():.0e}, "
          f"relative {err:.1e}", flush=True)
    assert err <= TOL_ENTRY
    assert (y >= 0).all()


def _line(n=128, width=2.0):
    """A bump of a few cells on a line: everything else is far tail."""
    x = np.arange(n) - 0.15 * n
    p = np.exp(-x * x / (2 * width * width))
    p[p < 1e-6 * p.max()] = 0.0
    return (p / p.sum()).astype(np.float32)[None, :]


@pytest.mark.parametrize("per_product", [False, True])
@pytest.mark.parametrize("ratio", [2.5, 4.0])
def test_localised_density(ratio, per_product):
    banner(f"heat tail flow tau={ratio} gamma per_product={per_product}")
    p0 = _line()
    gamma = 10.0 / p0.size ** 2
    op = jk.HeatOperator(p0.shape, gamma, 10, per_product=per_product)
    p, _ = op.step(torch.from_numpy(p0).cuda(), jk.EnergySpec(kind="entropy"), ratio * gamma, max_iters=100)
    ref, _ = O.jko_step(p0.astype(np.float64), O.Energy(kind="entropy"), gamma, ratio * gamma, 100,
                        op=O.HeatKernel(np.ones(p0.shape, bool), gamma, 10))
    err = rel_l1(host64(p), ref)
    print(f"[gpu-test] heat tail flow tau={ratio} gamma: {err:.2e}", flush=True)
    assert err <= TOL_FLOW


@pytest.mark.parametrize("per_product", [False, True])
def test_overflow_is_reported(per_product):
    """At ten times gamma the far cells' scalings leave float32: an operator whose tail is cut off would
    hide that."""
    banner(f"heat tail overflow per_product={per_product}")
    p0 = _line()
    gamma = 10.0 / p0.size ** 2
    op = jk.HeatOperator(p0.shape, gamma, 10, per_product=per_product)
    with pytest.raises(jk.JKOError):
        op.step(torch.from_numpy(p0).cuda(), jk.EnergySpec(kind="entropy"), 10.0 * gamma, max_iters=100)
