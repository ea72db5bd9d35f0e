"""Sizes and index rules of the batched solve, from the header that its kernels
use (csrc/batched_layout.h), compiled for the host: what changes there is what is
checked here."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_17978_amd", "csrc")

# bytes of each array of a slot of n atoms, h half-spectrum points and c pairs, in order
ARRAYS = (("C", lambda n, h, c: 8 * h), ("G", lambda n, h, c: 4 * h), ("wts", lambda n, h, c: 96 * n),
          ("dwts", lambda n, h, c: 96 * n), ("home", lambda n, h, c: 16 * n), ("frac", lambda n, h, c: 24 * n),
          ("vec", lambda n, h, c: 88 * n), ("selfgrad", lambda n, h, c: 24 * n), ("row", lambda n, h, c: 8 * n),
          ("col", lambda n, h, c: 4 * c), ("kval", lambda n, h, c: 4 * c), ("pdr", lambda n, h, c: 16 * c),
          ("tab", lambda n, h, c: 8 * 15 ** 3), ("mpart", lambda n, h, c: 128 * n), ("hstart", lambda n, h, c: 260),
          ("perm", lambda n, h, c: 4 * n), ("fpair", lambda n, h, c: 24 * n))


def host_program(tmp_path, body):
    """Path of a program that includes the header and runs body."""
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    src, exe = tmp_path / "layout.cpp", tmp_path / "layout"
    src.write_text('#include <cstdio>\n#include <cstdlib>\n#include <initializer_list>\n#include "batched_layout.h"\nusing namespace qeqb;\n'
                   "int main(int argc, char** argv) {\n" + body + "\nreturn 0;}\n")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    return str(exe)


def run(exe, *args):
    out = subprocess.run([exe, *map(str, args)], capture_output=True, text=True, check=True)
    return [int(x) for x in out.stdout.split()]


# smallest and largest structures at ordinary cutoffs; 1,024 atoms on 60 points
# an axis with r_cut = 170 bohr (2.1e8 pairs, 4.7 GiB); the most pairs that the
# limit of four cell widths lets through
@pytest.mark.parametrize("n,nhalf,pairs", [(1, 12 * 12 * 7, 16), (512, 48 * 39 * 20, 40960),
                                           (1024, 60 * 60 * 31, 178956970), (1024, 60 * 60 * 31, 210000000),
                                           (1024, 64 * 64 * 33, 281000000)])
def test_slot_arrays_do_not_overlap(tmp_path, n, nhalf, pairs):
    members = ", ".join(f"slot_bytes(L.{name})" for name, _ in ARRAYS)
    exe = host_program(tmp_path, """
        BSlot L{};
        const size_t end = slot_layout(L, strtoull(argv[1], 0, 10), strtoull(argv[2], 0, 10), strtoull(argv[3], 0, 10));
        const size_t all[] = {MEMBERS, end};
        for (size_t at : all) std::printf("%zu ", at);""".replace("MEMBERS", members))
    at = run(exe, n, nhalf, pairs)
    assert at[0] == 0
    for (name, size), lo, hi in zip(ARRAYS, at[:-1], at[1:]):
        assert lo % 256 == 0 and lo + size(n, nhalf, pairs) <= hi, name


# every combination of axis lengths and kept modes: a block's LDS stays below the
# 64 KB that a launch gets without asking (and four forward blocks share 160 KB),
# its planes, rows and columns inside the buffers, every plane in one block, and
# the walk over the kept rows meets each once, at its place
PLANES = """
    const int len[] = {12, 16, 20, 24, 32, 36, 40, 48, 60, 64}, p = atoi(argv[1]);
    long cases = 0, bad = 0;
    for (int K1 : len) for (int K2 : len) for (int K3 : len) for (int share = 1; share <= 10; share += 3) {
        if (K1 < 2 * p || K2 < 2 * p || K3 < 2 * p) continue;
        ++cases;
        const int km = bq_min(K3 / 2 + 1, share * K3 / 20 + 1), nm2 = bq_min(K2, 2 * (share * K2 / 20) + 1);
        const int pb = bq_planes_inv(K1, K2, km, p), pf = bq_planes_fwd(pb, K2, K3);
        bool ok = 1 <= pf && pf <= pb && pb <= BQ_PB && pb + p - 1 <= K1;
        ok = ok && pb * K2 <= 2 * BQ_NC && (pb * K2) % 2 == 0 && pb * km <= BQ_NC2 && BQ_NC2 < BQ_KS2 && BQ_NC < BQ_KS;
        const size_t fwd = bq_lds_fwd(K2, K3, pf), inv = bq_lds_inv(K2, K3);
        ok = ok && fwd <= 40960 && inv <= fwd && bq_lds_lines(K1) <= 65536 && 8 * (size_t)K3 * pf * K2 <= fwd;
        ok = ok && 8 * ((size_t)(K3 - 1) * BQ_KS + (pb * K2 - 1) / 2 + 1) <= inv && km <= 64;
        for (int planes : {pf, pb}) {
            const int kept = planes * nm2;
            ok = ok && kept <= BqWalk::ROWS * (2 * BQ_NC / BqWalk::ROWS);   // register slots
            int seen = 0;
            for (int first = 0; first < BqWalk::ROWS; ++first)
                for (BqWalk w(32 * first + 31, nm2, km, K2); w.row < kept; w.next(), ++seen) {
                    const int j = w.row / nm2, m2 = bq_m2(w.row % nm2, nm2, K2);
                    ok = ok && w.row % BqWalk::ROWS == first && w.at() == m2 * BQ_KS2 + j * km;
                    ok = ok && 0 <= m2 && m2 < K2 && 8 * (size_t)(w.at() + km) <= inv;
                }
            ok = ok && seen == kept;
        }
        // kept indices: the lowest and the highest, without a repeat
        int last = -1;
        for (int e = 0; e < nm2; ++e) {
            const int m2 = bq_m2(e, nm2, K2);
            ok = ok && m2 > last && (m2 <= (nm2 - 1) / 2 || m2 >= K2 - (nm2 - 1) / 2 || nm2 == K2);
            last = m2;
        }
        ok = ok && last == (nm2 == 1 ? 0 : K2 - 1);
        if (!ok && ++bad < 5) std::fprintf(stderr, "%d %d %d share %d\\n", K1, K2, K3, share);
    }
    std::printf("%ld %ld", cases, bad);"""


@pytest.mark.parametrize("p", [4, 6, 8])
def test_blocks_stay_inside_their_buffers(tmp_path, p):
    lengths = sum(k >= 2 * p for k in (12, 16, 20, 24, 32, 36, 40, 48, 60, 64))
    assert run(host_program(tmp_path, PLANES), p) == [4 * lengths ** 3, 0]
