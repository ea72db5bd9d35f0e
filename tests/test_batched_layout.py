"""Memory layout of the batched solve, from the header that its kernels use
(csrc/batched_layout.h), compiled for the host."""
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
    src.write_text('#include <cstdio>\n#include <cstdlib>\n#include "batched_layout.h"\nusing namespace qeqb;\n'
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
