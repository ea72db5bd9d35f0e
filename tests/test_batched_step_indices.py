"""Host replay of the batched kernels' index arithmetic (csrc/batched.hip).

For every combination of the ten axis lengths and the three spline orders: the
planes of a block (pb), its LDS buffers, the accumulator rows, the half-spectrum
columns and the axis-1 line blocks stay inside their allocations and cover every
row, plane and line exactly once.  The formulas are transcribed from the source;
no kernel runs.
"""
import itertools

import numpy as np
import pytest

LENGTHS = (12, 16, 20, 24, 32, 36, 40, 48, 60, 64)
NC, KS, NC2, KS2, NT, PB, KAX = 64, 65, 56, 57, 512, 8, 64


ACC = 38400


def planes_per_block(K, km, p):
    """pf, pb: planes of a block of the forward and of the inverse kernel."""
    pb = max(1, min(2 * NC // K[1], NC2 // km, K[0] - p + 1, PB))
    return max(1, min(pb, ACC // (8 * K[1] * K[2]))), pb


def walk(nm2, km, K2, kept):
    """BqWalk: (m2, plane) of the rows tid >> 5, + NT / 32, ..., by its carries."""
    out = {}
    step = NT // 32
    for first in range(step):
        row, j, e = first, 0, first
        while True:
            while e >= nm2:
                e, j = e - nm2, j + 1
            if row >= kept:
                break
            assert row not in out
            out[row] = (e if e < (nm2 + 1) // 2 else e + K2 - nm2, j)
            row, e = row + step, e + step
    assert kept <= step * (2 * NC // step)      # register slots of the loads
    return [out[r] for r in range(kept)]


@pytest.mark.parametrize("p", [4, 6, 8])
def test_blocks_stay_inside_their_buffers(p):
    # kept modes: all of them, the usual four fifths, and very few
    shares = (1.0, 0.8, 0.1)
    for (K, share) in itertools.product(itertools.product([k for k in LENGTHS if k >= 2 * p], repeat=3), shares):
        K1, K2, K3 = K
        km = min(K3 // 2 + 1, int(share * K3 / 2) + 1)
        nm2 = min(K2, 2 * int(share * K2 / 2) + 1)
        assert (nm2 == K2 or nm2 % 2 == 1) and 1 <= nm2 <= K2
        pf, pb = planes_per_block(K, km, p)
        assert 1 <= pf <= pb
        rw = pf * K2
        assert pb * K2 <= 2 * NC and rw <= 2 * NC and rw % 2 == 0 and pb * km <= NC2 < KS2 and NC2 <= 64 and pb <= PB
        assert pb + p - 1 <= K1                        # a block's candidate planes never overlap themselves
        lds = max(K3 * KS * 8, K2 * KS2 * 8, K3 * rw * 8)   # lines, columns and accumulator share their place
        assert lds <= ACC
        # unpacking / packing slots: m = tid / 128 + 4 q, q < 9
        assert 4 * ((KAX // 2 + 4) // 4) > K3 // 2
        # clears (int4), conversion (t -> (g3, c)), unpacking and packing
        assert (K3 * rw) % 2 == 0
        t = np.arange(KAX * NC)
        g3, c = t // NC, t % NC
        ok = (g3 < K3) & (c < rw // 2)
        assert (g3 * rw + 2 * c + 1)[ok].max() < K3 * rw and ok.sum() == K3 * rw // 2
        assert (g3 * KS + c)[g3 < K3].max() < K3 * KS
        fwd = np.zeros(K1, dtype=int)
        for y in range(-(-K1 // pf)):
            fwd[y * pf:y * pf + min(pf, K1 - y * pf)] += 1
        assert np.all(fwd == 1)
        done = np.zeros(K1, dtype=int)
        for y in range(-(-K1 // pb)):
            g1a, planes = y * pb, min(pb, K1 - y * pb)
            done[g1a:g1a + planes] += 1
            rows = planes * K2
            kept = planes * nm2
            assert km <= 64                                # two steps of 32 lanes
            r = np.arange(rows)
            j, g2 = r // K2, r % K2
            cols = j[:, None] * km + np.arange(km)[None, :]
            assert cols.max() < NC2 and (g2[:, None] * KS2 + cols).max() < K2 * KS2
            # packed rows: row pairs stay in one plane (K2 even)
            assert np.all((r[0::2] // K2) == (r[1::2] // K2)) and rows // 2 <= NC
            assert (g1a + planes) * nm2 * km <= K1 * nm2 * km
            if y == 0 and K1 == K3:
                rr = np.arange(kept)
                e = rr % nm2
                m2 = np.where(e < (nm2 + 1) // 2, e, e + K2 - nm2)
                assert walk(nm2, km, K2, kept) == list(zip(m2.tolist(), (rr // nm2).tolist()))
                # kept rows and cleared rows together are all rows
                half = (nm2 + 1) // 2
                assert sorted(set(m2.tolist()) | set(range(half, half + K2 - nm2))) == list(range(K2))
        assert np.all(done == 1)
        # potential reads of the interpolation: 2 (g3 KS + (r >> 1)) + (r & 1)
        assert 2 * ((K3 - 1) * KS + ((pb * K2 - 1) >> 1)) + 1 < 2 * K3 * KS
        # axis-1 line blocks
        nl = nm2 * km
        nb = -(-nl // NC)
        L = np.arange(nb * NC)
        assert np.array_equal(L[L < nl], np.arange(nl))
        kstep = NT // NC
        maxit = KAX // kstep
        k = (np.arange(NT) // NC)[:, None] + kstep * np.arange(maxit)[None, :]
        for cc in (0, NC - 1):
            hits = np.sort(k[np.arange(NT) % NC == cc].ravel())
            assert np.array_equal(hits[hits < K1], np.arange(K1))


def test_plane_ranges_wrap():
    """bq_ranges: the atoms (sorted by home plane) with home planes g1 .. g1 + p - 1."""
    rng = np.random.default_rng(0)
    for K1, p, n in ((12, 6, 1), (12, 6, 40), (24, 8, 500), (64, 4, 1024), (16, 8, 7)):
        h = np.sort(rng.integers(0, K1, n))
        hs = np.concatenate([[0], np.cumsum(np.bincount(h, minlength=K1))])
        for g in range(K1):
            e = g + p
            cnt = hs[e] - hs[g] if e <= K1 else n - hs[g] + hs[e - K1]
            i = hs[g] + np.arange(cnt)
            i = np.where(i >= n, i - n, i)
            want = [a for a in range(n) if (h[a] - g) % K1 < p]
            assert sorted(i.tolist()) == want
            k1 = h[i] - g
            k1 = np.where(k1 < 0, k1 + K1, k1)
            assert np.all((k1 >= 0) & (k1 < p))
