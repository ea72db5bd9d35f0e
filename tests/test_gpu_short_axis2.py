"""Grids whose axis 2 has 16 points, with an axis 1 or 3 that has no uniform
tiles of its own: two tiles of eight rows.  The header's range of grids holds
them; the uniform 16-row tiles that served other lengths refused them.  Parity
bars of the other solves against the dense FP64 oracle.
"""
import numpy as np
import pytest

from inputs import gen
from oracle import ewald

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid", [(288, 16, 32), (16, 16, 60), (20, 16, 36), (60, 16, 12)])
@pytest.mark.parametrize("q_tot", [0.0, 1.0])
def test_matches_oracle(grid, q_tot):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2607_17978_amd import qeq
    rng = np.random.default_rng([31, *grid])
    cell = np.diag([0.75 * k for k in grid])
    side = np.maximum(1, (np.diag(cell) / 5.0).astype(int))
    sites = np.stack(np.meshgrid(*map(np.arange, side), indexing="ij"), -1).reshape(-1, 3)
    n = len(sites)
    pos = (sites + 0.5 + rng.uniform(-0.1, 0.1, (n, 3))) / side @ cell
    sp = rng.integers(0, 2, n)
    sigma, J = np.asarray(gen.SIGMA_2EL)[sp], np.asarray(gen.J_2EL)[sp]
    chi = np.asarray(gen.CHI_MEAN_2EL)[sp] + rng.normal(0.0, gen.CHI_SD, n)
    ref = ewald.qeq_dense(pos, cell, sigma, J, chi, q_tot)
    T = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")
    plan = qeq.Plan(n, eta=2.0, r_cut=11.0, grid=grid, tol=1e-8, max_iter=3000)
    q, en, f, st = plan.solve(T(pos), cell, T(sigma), T(J), T(chi), q_tot)
    plan.close()
    assert st["rc"] == 0
    assert np.abs(q.cpu().numpy() - ref.q).max() <= 1e-5
    assert abs(float(en[0]) - ref.e_qeq) <= 1e-6 * max(abs(ref.e_qeq), 1e-2)
    assert np.sqrt(np.mean((f.cpu().numpy() - ref.forces) ** 2)) <= 1e-4 * max(np.sqrt(np.mean(ref.forces ** 2)), 1e-2)
