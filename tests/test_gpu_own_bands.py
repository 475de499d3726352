"""A 2D product of a caller's field (whose memory may start at any float and may
not be read past its end) against the same product inside a step, whose fields
lie in the workspace: one iteration under the zero energy from a = 1 is
b = q / (xi 1), p = xi b, so two products give the step's density bit for bit.
Grids at the edges of the tiles of both sizes, narrow and wide bands, and bands
cut by both edges of the grid."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_1502_06216_amd as jk

from _util import banner, dev, f32, host64
from workloads import small_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp32", "split_bf16"])
@pytest.mark.parametrize("shape,cells", [((16, 16), 2.0), ((1, 250), 3.0), ((17, 33), 1.0), ((45, 70), 3.0),
                                         ((201, 161), 3.0), ((256, 256), 4.0), ((64, 48), 5.0), ((300, 270), 2.5),
                                         ((511, 500), 4.0)])
def test_same_bits_as_in_a_step(shape, cells, precision):
    banner(f"own bands {shape} {cells} {precision}")
    gamma = (cells / max(shape)) ** 2
    q = dev(small_case(shape, "zero", seed=2).p0)
    p, _ = jk.step(q, jk.EnergySpec(kind="zero"), gamma, 2.5 * gamma, max_iters=1, precision=precision,
                   resident=False)
    t = jk.gibbs_apply(torch.ones_like(q), gamma, precision)
    b = torch.where(q == 0, torch.zeros_like(q), q / t)
    assert torch.equal(jk.gibbs_apply(b, gamma, precision), p)
    # the same input one float later, with values behind it that no output may see
    buf = torch.full((b.numel() + 5,), float("nan"), device=b.device)
    buf[1:1 + b.numel()] = b.reshape(-1)
    assert torch.equal(jk.gibbs_apply(buf[1:1 + b.numel()].view(*shape), gamma, precision), p)
    # a value that isn't finite stays out of the row before its own
    if min(shape) > 1 and cells * 11 < shape[0] / 4:
        x = torch.ones_like(q)
        r = shape[0] // 2
        x[r, 0] = float("inf")
        y = jk.gibbs_apply(x, gamma, precision)
        assert not torch.isfinite(y[r, 0])
        if cells * 11 + 20 < shape[1]:
            assert torch.isfinite(y[:, -1]).all()


@pytest.mark.parametrize("precision", ["fp32", "split_bf16"])
@pytest.mark.parametrize("shape", [(64, 1), (65,), (300, 2), (70, 3), (3, 3), (1, 1), (40, 5), (18, 6), (50, 17),
                                   (33, 34), (80, 47), (20, 18, 21), (17, 16, 33)])
@pytest.mark.parametrize("cells", [0.4, 1.0, 2.0])
def test_the_last_values_of_a_callers_field(shape, cells, precision):
    """The copies that cross the end of a caller's field, whose last three values are read one by one: rows of one
    to three cells, tiles whose halo ends just before the last cell, every start of the field in its memory; against
    the oracle's products, with values behind the field that no output may see."""
    banner(f"field end {shape} {cells} {precision}")
    gamma = (cells / max(shape)) ** 2
    rng = np.random.default_rng(9)
    x = f32(rng.uniform(0.5, 1.5, shape))
    ref = O.gibbs_apply(x.astype(np.float64), gamma)
    for off in range(4):
        buf = torch.full((x.size + 8,), float("nan"), device="cuda")
        buf[off:off + x.size] = dev(x).reshape(-1)
        y = host64(jk.gibbs_apply(buf[off:off + x.size].view(*shape), gamma, precision))
        # sums of positive terms in FP32, two roundings an axis; 16-bit pairs split
        np.testing.assert_allclose(y, ref, rtol={"fp32": 1e-5, "split_bf16": 1e-4}[precision], atol=0)
