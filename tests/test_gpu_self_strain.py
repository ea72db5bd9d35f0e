"""Virial across the split of its self-correction tables over blocks (up to
4,096 atoms): a cell of 2,100 atoms and its double along one axis, on a grid
that doubles with it, have the same charges and twice the virial.

Bar: the charges of both solves are within the CG tolerance 1e-8 and the FP32
mesh and pair rounding of the product, a few 1e-7 of the virial's norm; 1e-5
is what the mesh virial is held to against the oracle elsewhere.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_double_cell_has_twice_the_virial():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2607_17978_amd import qeq
    rng = np.random.default_rng(83)
    n, L = 2100, 60.0
    sites = np.stack(np.meshgrid(*[np.arange(13)] * 3, indexing="ij"), -1).reshape(-1, 3)[rng.permutation(2197)[:n]]
    pos = (sites + 0.5 + rng.uniform(-0.2, 0.2, (n, 3))) * (L / 13)
    sigma, J, chi = rng.uniform(1.0, 1.6, n), rng.uniform(0.3, 0.6, n), rng.normal(0.0, 0.1, n)
    T = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")
    w = []
    for copies in (1, 2):
        cell = np.diag([L, L, L * copies])
        p = np.concatenate([pos + np.array([0.0, 0.0, L * c]) for c in range(copies)])
        plan = qeq.Plan(n * copies, eta=2.0, r_cut=11.0, grid=(80, 80, 80 * copies), tol=1e-8, max_iter=3000)
        st = plan.solve(T(p), cell, *[T(np.tile(a, copies)) for a in (sigma, J, chi)], 0.0)[3]
        assert st["rc"] == 0
        w.append(np.asarray(plan.virial().cpu()))
        plan.close()
    print(w[0], w[1])
    assert np.linalg.norm(w[1] - 2 * w[0]) <= 1e-5 * np.linalg.norm(w[1])
