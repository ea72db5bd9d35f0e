"""Plans of several host threads, each on a stream of its own, at the same time:
the CG loops are captured and replayed as graphs while other threads build grids,
allocate and copy.  Every thread gets the bits that its calls give one after the
other."""
import threading

import numpy as np
import pytest

from inputs import gen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

KINDS = ("solve64", "solve512", "cell", "ewald", "planewave", "virial4096", "batch", "cluster")


def T(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


def calls(kind, rounds, out):
    from paper_2607_17978_amd import qeq
    torch.cuda.set_device(0)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        if kind == "batch":
            ss = [gen.batch_structure(k) for k in range(16)]
            cat = lambda f: T(np.concatenate([getattr(s, f) for s in ss]))
            args = dict(pos=cat("pos"), offsets=np.cumsum([0] + [s.n for s in ss]), cells=np.stack([s.cell for s in ss]),
                        sigma=cat("sigma"), J=cat("J"), chi=cat("chi"), q_tot=[s.q_tot for s in ss])
            plan = qeq.Plan(512, r_cut=12.0, stream=stream)
            call = lambda i: plan.solve_batched(**args)[0]
        elif kind == "cluster":
            c = gen.cluster_system(1500, q_tot=1.0)
            args = (T(c.pos), T(c.sigma), T(c.J), T(c.chi), c.q_tot)
            plan = qeq.Plan(c.n, stream=stream)
            call = lambda i: plan.solve_nonperiodic(*args)[0]
        else:
            s = {"solve64": gen.system_64, "virial4096": gen.system_4096}.get(kind, gen.system_512)()
            args = [T(a) for a in (s.pos, s.sigma, s.J, s.chi)]
            plan = qeq.Plan(s.n, stream=stream)
            if kind == "ewald":
                plan.use_ewald(True)
            if kind == "planewave":
                plan.use_planewave(True)

            def call(i):
                # another cell, and every third time another grid, in each call
                cell = s.cell * (1.0 + (1e-3, 2e-3, 0.1)[i % 3]) if kind == "cell" else s.cell
                q = plan.solve(args[0], cell, args[1], args[2], args[3], 0.0)[0]
                return torch.cat([q, plan.virial().ravel()]) if kind in ("cell", "virial4096") else q

        for i in range(rounds):
            r = call(i)
            stream.synchronize()
            out.append(r.cpu().numpy())
        plan.close()


def test_threads_get_their_own_results():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    alone = {k: [] for k in KINDS}
    for k in KINDS:
        calls(k, 6, alone[k])
    for repeat in range(3):
        together, errors = {k: [] for k in KINDS}, []

        def run(k):
            try:
                calls(k, 6, together[k])
            except Exception as e:      # reported by the main thread
                errors.append((k, repr(e)))

        threads = [threading.Thread(target=run, args=(k,)) for k in KINDS]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        assert not errors, errors
        for k in KINDS:
            assert all(np.array_equal(a, b) for a, b in zip(alone[k], together[k])), k
