"""The Gaussian-on-grid operator's tile lists.

Cells far smaller than the supports (an atom meets a tile through several
periodic images), one atom alone, odd atom counts and strongly skewed cells
against the dense FP64 oracle at the parity bars of the other solves; and the
lists against the per-atom walks, which 32-row tiles select, on the same grid:
both add the same FP32 terms, so the charges agree to FP32 rounding amplified by
the solve (1e-6 e, as between any two mesh paths).
"""
import numpy as np
import pytest

from inputs import gen
from oracle import ewald

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def T(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


@pytest.mark.parametrize("n,length,skew,q_tot", [(1, 9.3, 0.0, 1.0), (5, 9.3, 0.3, 0.0), (13, 11.9, 0.2, -1.0),
                                                 (65, 18.6, 0.35, 0.0)])
def test_small_and_skewed_cells_match_oracle(n, length, skew, q_tot):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2607_17978_amd import qeq
    rng = np.random.default_rng([77, n])
    cell = length * (np.eye(3) + skew * np.array([[0.0, 0.0, 0.0], [1.0, 0.0, 0.0], [0.6, -0.8, 0.0]]))
    pos = rng.uniform(0, 1, (n, 3)) @ cell
    sigma, J, chi = rng.uniform(1.0, 1.6, n), rng.uniform(0.3, 0.6, n), rng.normal(0.0, 0.1, n)
    ref = ewald.qeq_dense(pos, cell, sigma, J, chi, q_tot)
    plan = qeq.Plan(n, eta=2.0, r_cut=11.0, max_spacing=0.8, tol=1e-9, max_iter=3000)
    plan.use_planewave(True)
    q, en, f, st = plan.solve(T(pos), cell, T(sigma), T(J), T(chi), q_tot)
    plan.close()
    assert st["rc"] == 0
    assert np.abs(q.cpu().numpy() - ref.q).max() <= 1e-5
    assert abs(float(en[0]) - ref.e_qeq) <= 1e-6 * max(abs(ref.e_qeq), 1e-2)
    assert np.sqrt(np.mean((f.cpu().numpy() - ref.forces) ** 2)) <= 1e-4 * max(np.sqrt(np.mean(ref.forces ** 2)), 1e-2)


def test_lists_equal_walks():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2607_17978_amd import qeq
    s = gen.system_4096()
    out = []
    for rows in (0, 32):
        plan = qeq.Plan(s.n, eta=2.0, r_cut=11.0, grid=s.grid, tol=1e-8, max_iter=3000)
        plan.use_planewave(True)
        plan.set_tiles(0, rows, 0)
        q, en, f, st = plan.solve(T(s.pos), s.cell, T(s.sigma), T(s.J), T(s.chi), 0.0)
        assert st["rc"] == 0
        out.append((q, en, f))
        plan.close()
    (q0, e0, f0), (q1, e1, f1) = out
    assert float((q0 - q1).abs().max()) <= 1e-6
    assert float((e0 - e1).abs().max() / e1.abs().max()) <= 1e-6
    assert float((f0 - f1).norm() / f1.norm()) <= 1e-5
