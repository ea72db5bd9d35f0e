"""Isolated solves with and without stored kernel values: the same bits, and the
matrix goes back when its bound or the plan's next call says so."""
import numpy as np
import pytest

from inputs import gen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def T(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


def cluster(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    s = gen.cluster_system(n, q_tot=1.0, seed=n)
    return s, (T(s.pos), T(s.sigma), T(s.J), T(s.chi), s.q_tot)


# one and several tiles of 256 atoms, the last one full or partial; 12,289 atoms:
# splits of two tiles
@pytest.mark.parametrize("n", [2, 255, 256, 257, 513, 1000, 4097, 12289])
def test_stored_and_evaluated_values_agree(n):
    from paper_2607_17978_amd import qeq
    s, args = cluster(n)
    species = torch.as_tensor(s.species, dtype=torch.int32, device="cuda")
    out = []
    for bound in (-1, 0):
        plan = qeq.Plan(n, tol=1e-8, max_iter=3000)
        plan.use_stored_kernel(bound)
        q, en, f, st = plan.solve_nonperiodic(*args)
        assert st["rc"] == 0
        out.append((q, en, f, plan.element_potentials(species, 2)))
        if bound < 0:      # products after the matrix has gone
            plan.use_stored_kernel(0)
            assert torch.equal(plan.element_potentials(species, 2), out[0][3])
        plan.close()
    for a, b in zip(*out):
        assert torch.equal(a, b)


def free_bytes():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


@pytest.mark.parametrize("leave", ["bound", "solve", "batch"])
def test_large_matrix_is_given_back(leave):
    from paper_2607_17978_amd import qeq
    n = 12289                                      # 12,289 x 12,352 floats: 607 MB
    s, args = cluster(n)
    d = gen.system_64()
    periodic = (T(d.pos), d.cell, T(d.sigma), T(d.J), T(d.chi), 0.0)
    batch = dict(pos=T(d.pos), offsets=[0, d.n], cells=d.cell[None], sigma=T(d.sigma), J=T(d.J), chi=T(d.chi),
                 q_tot=[0.0])
    plan = qeq.Plan(n, max_iter=20)
    plan.solve(*periodic)
    plan.solve_batched(**batch)                    # what these calls allocate once
    plan.use_stored_kernel(0)
    plan.solve_nonperiodic(*args, check=False)
    before = free_bytes()
    plan.use_stored_kernel()
    plan.solve_nonperiodic(*args, check=False)
    assert before - free_bytes() >= 500 << 20
    {"bound": lambda: plan.use_stored_kernel(256 << 20), "solve": lambda: plan.solve(*periodic),
     "batch": lambda: plan.solve_batched(**batch)}[leave]()
    assert before - free_bytes() < 100 << 20
    plan.close()
