"""Self-correction tables at axis lengths around their 64-column steps.

The mesh reproduces an atom's own reciprocal term as theta^T Theta theta, which
depends on its place in the grid cell; with the correction the sum does not.
What is left is the FP32 rounding of the mesh product, 4 log2(N) 2^-24 of the
term for each of the two products compared.
"""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid,p", [((16, 16, 16), 4), ((12, 60, 20), 6), ((20, 64, 16), 6), ((16, 72, 24), 8),
                                    ((100, 128, 12), 6), ((24, 36, 160), 6)])
def test_corrected_self_term_does_not_move(grid, p):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2607_17978_amd import qeq
    rng = np.random.default_rng([82, *grid])
    cell = np.diag([0.8 * k for k in grid]) @ np.array([[1.0, 0.0, 0.0], [0.25, 1.0, 0.0], [-0.2, 0.15, 1.0]])
    T = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")
    sigma, v = T([1.2]), T([1.0])
    plan = qeq.Plan(1, eta=2.0, r_cut=7.0, grid=grid, spline_order=p)
    raw, fixed = [], []
    for _ in range(6):
        pos = T(rng.uniform(0, 1, (1, 3)) @ cell)
        raw.append(float(plan.matvec(pos, cell, sigma, v, qeq.PART_RECIP)))
        fixed.append(float(plan.matvec(pos, cell, sigma, v, qeq.PART_RECIP | qeq.PART_SELF)))
    plan.close()
    print(grid, p, "raw spread", np.ptp(raw), "corrected", np.ptp(fixed), "term", raw[0])
    tol = 2 * 4 * math.log2(grid[0] * grid[1] * grid[2]) * 2.0 ** -24 * max(abs(r) for r in raw)
    assert np.ptp(fixed) <= tol
    assert np.ptp(raw) > np.ptp(fixed)
