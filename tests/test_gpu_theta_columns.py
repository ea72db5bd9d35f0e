"""Self-correction tables whose columns are split over blocks.

As in the tables' other test, the corrected self term of one atom does not depend
on its place in the grid cell, and neither does its virial (the strain tables),
up to the FP32 rounding of the mesh product: 4 log2(N) 2^-24 of the term or of the
virial's largest entry for each of the two compared.  Axis 2 has two to eight
groups of 64 columns, with a last group of four to 64, and fewer blocks than
groups where axis 3 is long.
"""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid,p", [((12, 72, 12), 6), ((16, 128, 16), 8), ((12, 192, 40), 6), ((12, 200, 12), 4),
                                    ((12, 320, 512), 6), ((16, 512, 20), 8)])
def test_corrected_terms_do_not_move(grid, p):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2607_17978_amd import qeq
    rng = np.random.default_rng([97, *grid])
    cell = np.diag([0.8 * k for k in grid]) @ np.array([[1.0, 0.0, 0.0], [0.02, 1.0, 0.0], [-0.03, 0.01, 1.0]])
    T = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")
    one = T([1.0])
    spread = {}
    for correct in (True, False):
        plan = qeq.Plan(1, eta=2.0, r_cut=7.0, grid=grid, spline_order=p, self_correction=correct)
        terms, virials = [], []
        at = rng.uniform(0, 1, (6, 1, 3)) if correct else at
        for x in at:
            pos = T(x @ cell)
            terms.append(float(plan.matvec(pos, cell, T([1.2]), one, qeq.PART_RECIP | qeq.PART_SELF)))
            plan.solve(pos, cell, T([1.2]), one, T([0.1]), 1.0)
            virials.append(plan.virial().cpu().numpy())
        plan.close()
        spread[correct] = np.ptp(terms), np.ptp(virials, axis=0).max(), np.abs(terms).max(), np.abs(virials).max()
    print(grid, p, spread)
    bar = 2 * 4 * math.log2(grid[0] * grid[1] * grid[2]) * 2.0 ** -24
    assert spread[True][0] <= bar * spread[True][2]
    assert spread[True][1] <= bar * spread[True][3]
    assert spread[False][0] > spread[True][0] and spread[False][1] > spread[True][1]
