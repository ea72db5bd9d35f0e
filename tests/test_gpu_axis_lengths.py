"""Mesh product for every supported axis length against plain FP64 torch.

Each of the 36 lengths takes each axis in turn, the other two axes being short
lengths whose rows do not divide into equal tiles, with spline orders 4, 6 and 8
in turn, in a triclinic cell.  The reference is the same discretisation in 64
bits (B-spline spreading, torch.fft, Green's function with the spline moduli,
interpolation), so what is left is FP32 rounding: two transforms of N points,
each value passing log2 N butterfly levels there and back with about two
roundings per level, bounded by 4 log2(N) 2^-24 of the result's norm.
"""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LENGTHS = [k for k in range(12, 513, 4) if all(k % f for f in (7, 11, 13, 17, 19, 23, 29, 31, 37, 41, 43, 47, 53, 59,
                                                              61, 67, 71, 73, 79, 83, 89, 97, 101, 103, 107, 109,
                                                              113, 127))]
ETA = 2.0


def spline(w, p):
    """M_p(w + k), k = 0 .. p - 1, for w in [0, 1)."""
    x = w[:, None] + torch.arange(p, dtype=torch.float64, device=w.device)
    m = [torch.clamp(1.0 - (x - j - 1.0).abs(), min=0.0) for j in range(p)]   # M_2(x - j)
    for n in range(3, p + 1):
        m = [((x - j) * m[j] + (n - x + j) * m[j + 1]) / (n - 1) for j in range(p + 1 - n + 1)]
    return m[0]


def reference(pos, cell, v, grid, p):
    H = torch.as_tensor(cell, dtype=torch.float64, device=pos.device)
    Hi = torch.linalg.inv(H)
    s = pos @ Hi
    s = s - torch.floor(s)
    idx, wts = [], []
    for a in range(3):
        u = s[:, a] * grid[a]
        h = torch.floor(u)
        idx.append((h[:, None].long() - torch.arange(p, device=pos.device)) % grid[a])
        wts.append(spline(u - h, p))
    at = (idx[0][:, :, None, None] * grid[1] + idx[1][:, None, :, None]) * grid[2] + idx[2][:, None, None, :]
    w = wts[0][:, :, None, None] * wts[1][:, None, :, None] * wts[2][:, None, None, :]
    Q = torch.zeros(grid[0] * grid[1] * grid[2], dtype=torch.float64, device=pos.device)
    Q.index_add_(0, at.reshape(-1), (w * v[:, None, None, None]).reshape(-1))
    ms, mod = [], []
    for a in range(3):
        K = grid[a]
        m = torch.arange(K, dtype=torch.float64, device=pos.device)
        ints = spline(torch.zeros(1, dtype=torch.float64, device=pos.device), p)[0]   # M_p(0), M_p(1), ...
        ph = torch.exp(2j * math.pi * m[:, None] * torch.arange(p - 1, device=pos.device) / K)
        mod.append(1.0 / ((ph * ints[1:p]).sum(1).abs() ** 2))
        ms.append(torch.where(m <= K // 2, m, m - K))
    m = torch.stack(torch.meshgrid(*ms, indexing="ij"), -1)
    k2 = ((2 * math.pi * (m @ Hi.T)) ** 2).sum(-1)
    G = 4 * math.pi / float(torch.linalg.det(H)) * torch.exp(-0.5 * ETA ** 2 * k2) / k2
    G = G * mod[0][:, None, None] * mod[1][None, :, None] * mod[2][None, None, :]
    G[0, 0, 0] = 0.0
    G[grid[0] // 2] = 0.0
    G[:, grid[1] // 2] = 0.0
    G[:, :, grid[2] // 2] = 0.0
    phi = torch.fft.ifftn(torch.fft.fftn(Q.reshape(grid)) * G).real * Q.numel()
    return (w * phi.reshape(-1)[at]).sum((1, 2, 3))


@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("i", range(len(LENGTHS)))
def test_every_length(i, axis):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2607_17978_amd import qeq
    assert len(LENGTHS) == 36
    K = LENGTHS[i]
    p = (4, 6, 8)[(i + axis) % 3]
    if K < 2 * p:
        p = 6
    grid = [20, 36, 24]
    grid[axis] = K
    rng = np.random.default_rng([36, i, axis])
    n = 70
    cell = np.diag([0.75 * g for g in grid]) @ np.array([[1.0, 0.05, 0.1], [0.0, 1.0, -0.1], [0.08, 0.0, 1.0]])
    dev = torch.device("cuda")
    pos = torch.as_tensor(rng.uniform(0, 1, (n, 3)) @ cell, device=dev)
    v = torch.as_tensor(rng.normal(0, 0.3, n), device=dev)
    sigma = torch.full((n,), 1.2, dtype=torch.float64, device=dev)
    ref = reference(pos, cell, v, grid, p)
    tol = 4.0 * math.log2(np.prod(grid)) * 2.0 ** -24
    plan = qeq.Plan(n, eta=ETA, r_cut=6.0, grid=grid, spline_order=p)
    for fused in (True, False):
        plan.use_fused_interp(fused)
        y = plan.matvec(pos, cell, sigma, v, parts=qeq.PART_RECIP)
        err = float((y - ref).norm() / ref.norm())
        print("K", K, "axis", axis, "order", p, "fused", fused, "relative error", err, "bound", tol)
        assert err <= tol
    plan.close()
