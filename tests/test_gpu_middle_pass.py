"""The one-pass middle of the mesh product (planes up to 64 x 64) against the
separate axis passes, on planes at the edges of its three tile sizes.

Both are FP32 transforms of the same N points, each within 4 log2(N) 2^-24 of
the exact product's norm (two roundings per butterfly level, there and back).
"""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid", [(12, 12, 12), (32, 12, 20), (12, 32, 16), (36, 24, 12), (20, 48, 36), (48, 48, 24),
                                  (64, 12, 32), (12, 64, 60), (60, 64, 12), (64, 64, 100)])
def test_one_pass_equals_separate_passes(grid):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2607_17978_amd import qeq
    rng = np.random.default_rng([80, *grid])
    n, cell = 37, np.diag([0.75 * k for k in grid]) @ np.array([[1.0, 0.0, 0.0], [0.2, 1.0, 0.0], [-0.15, 0.1, 1.0]])
    T = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")
    pos, sigma, v = T(rng.uniform(0, 1, (n, 3)) @ cell), T(np.full(n, 1.2)), T(rng.normal(0.0, 1.0, n))
    plan = qeq.Plan(n, eta=2.0, r_cut=7.0, grid=grid)
    out = []
    for one in (True, False):
        plan.use_fused_inverse(one)
        for interp in (True, False):
            plan.use_fused_interp(interp)
            out.append(plan.matvec(pos, cell, sigma, v, qeq.PART_RECIP))
    plan.close()
    tol = 8 * math.log2(grid[0] * grid[1] * grid[2]) * 2.0 ** -24
    for y in out[1:]:
        assert float((y - out[0]).norm() / out[0].norm()) <= tol
