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
NC, KS, NC2, KS2, NT, PB, KAX = 64, 65, 66, 67, 512, 8, 64


def planes_per_block(K, p):
    return max(1, min(2 * NC // K[1], NC2 // (K[2] // 2 + 1), K[0] - p + 1, PB))


@pytest.mark.parametrize("p", [4, 6, 8])
def test_blocks_stay_inside_their_buffers(p):
    for K in itertools.product([k for k in LENGTHS if k >= 2 * p], repeat=3):
        K1, K2, K3 = K
        K3h, pb = K3 // 2 + 1, planes_per_block(K, p)
        rw = pb * K2
        assert rw <= 2 * NC and rw % 2 == 0 and pb * K3h <= NC2 < KS2 and pb <= PB
        assert pb + p - 1 <= K1                        # a block's candidate planes never overlap themselves
        two = K3 * KS + K2 * KS2                       # buf + X2, complex
        lds_fwd = max(two * 8, K3 * rw * 8)
        assert lds_fwd <= 160 * 1024 - 4096
        # clears (int4), conversion (t -> (g3, c)), unpacking and packing
        assert (K3 * rw) % 2 == 0
        t = np.arange(KAX * NC)
        g3, c = t // NC, t % NC
        ok = (g3 < K3) & (c < rw // 2)
        assert (g3 * rw + 2 * c + 1)[ok].max() < K3 * rw and ok.sum() == K3 * rw // 2
        assert (g3 * KS + c)[g3 < K3].max() < K3 * KS
        done = np.zeros(K1, dtype=int)
        for y in range(-(-K1 // pb)):
            g1a, planes = y * pb, min(pb, K1 - y * pb)
            done[g1a:g1a + planes] += 1
            rows = planes * K2
            # loads and stores of the half spectra: PER register slots cover rows * K3h elements
            per = -(-KAX * NC2 // NT)
            assert rows * K3h <= per * NT
            r = np.arange(rows)
            j, g2 = r // K2, r % K2
            cols = j[:, None] * K3h + np.arange(K3h)[None, :]
            assert cols.max() < NC2 and (g2[:, None] * KS2 + cols).max() < K2 * KS2
            # packed rows: row pairs stay in one plane (K2 even)
            assert np.all((r[0::2] // K2) == (r[1::2] // K2)) and rows // 2 <= NC
            assert (g1a * K2 * K3h + rows * K3h) <= K1 * K2 * K3h
        assert np.all(done == 1)
        # potential reads of the interpolation: 2 (g3 KS + (r >> 1)) + (r & 1)
        assert 2 * ((K3 - 1) * KS + ((pb * K2 - 1) >> 1)) + 1 < 2 * K3 * KS
        # axis-1 line blocks
        nl = K2 * K3h
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
