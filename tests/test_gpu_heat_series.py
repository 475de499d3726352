"""The heat kernel's Chebyshev series (per-product form and the stored
operator's columns) against the oracle's sparse LU solves, at the edges of the
series kernel's 16 x 32 tiles and 16-sweep launches."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_1502_06216_amd as jk
from tests._util import banner

pytestmark = pytest.mark.gpu

# One product: the series' error is below 1e-15 of the input's norm, so what
# is left is the rounding of the result (and of the stored operator's entries
# and float32 sums) to float32: a few 2^-24 in the L1 norm.
TOL = 1e-6


@pytest.mark.parametrize("shape", [(1, 1), (1, 70), (5, 1), (16, 32), (17, 33), (15, 31), (33, 65), (40, 97)])
@pytest.mark.parametrize("L,nu", [(1, 1.0), (10, 1.0), (10, 0.01), (10, 9.0), (37, 0.3)])
def test_products_match_the_oracle(shape, L, nu):
    banner(f"heat series {shape} L={L} nu={nu}")
    rng = np.random.default_rng(shape[0] * 1000 + shape[1])
    mask = rng.uniform(size=shape) < 0.85
    mask.flat[0] = True
    gamma = nu * L / max(shape) ** 2
    H = O.HeatKernel(mask, gamma, L)
    x = np.where(mask, rng.uniform(size=shape), 0.0).astype(np.float32)
    ref = H(x.astype(np.float64))
    m = torch.from_numpy(mask.astype(np.uint8)).cuda()
    for per_product in (False, True):
        op = jk.HeatOperator(shape, gamma, L, mask=m, per_product=per_product)
        y = op.apply(torch.from_numpy(x).cuda()).cpu().numpy().astype(np.float64)
        err = np.abs(y - ref).sum() / np.abs(ref).sum()
        print(f"[gpu-test] heat series {shape} L={L} nu={nu} per_product={per_product}: {err:.2e}", flush=True)
        assert err <= TOL
        assert not y[~mask].any()
