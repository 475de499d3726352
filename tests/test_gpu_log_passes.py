"""The log-domain passes at the edges of their work items (256 outputs along a
contiguous axis, 16 x 16 along a strided one): short, odd and long axes, fewer
fibres than an item holds, more items than blocks, against the exact
log-sum-exp oracle."""
import numpy as np
import pytest

import oracle as O
import paper_1502_06216_amd as jk
from tests._util import banner, dev, energies, f32, host64, rel_l1
from workloads import small_case

pytestmark = pytest.mark.gpu

# As the other log-domain tests: the scalings' logs (up to about 100) carry a
# rounding of 2^-24 of themselves per product, relative in the density.
TOL = 1e-5


@pytest.mark.parametrize("shape", [(300,), (1024,), (2, 257), (257, 3), (16, 16), (15, 33), (17, 256), (1024, 20),
                                   (20, 1024), (7, 5, 70), (40, 33, 31), (1, 1, 40)])
def test_step_matches_the_log_oracle(shape):
    banner(f"log passes {shape}")
    wl = small_case(shape, "congestion", seed=3, n_boxes=0, projected=False)
    g_en, o_en = energies(wl)
    p, _ = jk.step(dev(wl.p0), g_en, wl.gamma, wl.tau, max_iters=12, check_every=5, absorb_threshold=0.0)
    ref, _ = O.jko_step_log(f32(wl.p0).astype(np.float64), o_en, wl.gamma, wl.tau, 12)
    err = rel_l1(host64(p), ref)
    print(f"[gpu-test] log passes {shape}: rel-L1 {err:.2e}", flush=True)
    assert err <= TOL
