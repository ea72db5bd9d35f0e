"""Growth of buffers that share a capacity (csrc/grow.h), compiled for the host
with an allocator that fails on demand: after a failure no buffer is left and no
capacity either, so that the next request allocates instead of using nothing."""
import os
import re
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_17978_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "grow.h"
int main(int, char** argv) {
    // requests in turn: items, number of the allocation that fails (0: none)
    void *a = nullptr, *b = nullptr, *c = nullptr;
    size_t cap = 0;
    int live = 0;
    for (int r = 1; argv[r]; r += 2) {
        const int fail = atoi(argv[r + 1]);
        int calls = 0;
        size_t bytes = 0;
        const bool ok = grow_together(cap, strtoull(argv[r], 0, 10), {{&a, 4, 1, false}, {&b, 8, 0, true}, {&c, 16, 2, false}},
            [&](const GrowBuf&, size_t n) {
                if (++calls == fail) return (void*)nullptr;
                bytes += n;
                ++live;
                return malloc(n);
            },
            [&](void* p) { --live; free(p); });
        std::printf("%d %zu %d %d %d %zu\n", (int)ok, cap, (a != nullptr) + (b != nullptr) + (c != nullptr), live, calls, bytes);
    }
}
"""


@pytest.mark.parametrize("fail", [1, 2, 3])
def test_failed_growth_leaves_no_capacity(tmp_path, fail):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    src, exe = tmp_path / "grow.cpp", tmp_path / "grow"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    # first request, larger one that fails, one below the first, one that fits
    out = subprocess.run([str(exe), "100", "0", "1000", str(fail), "50", "0", "50", "0"], capture_output=True,
                         text=True, check=True).stdout.split("\n")
    ok, cap, held, live, calls, size = zip(*(map(int, line.split()) for line in out if line))
    assert ok == (1, 0, 1, 1)
    assert cap == (100, 0, 50, 50)
    assert held == (3, 0, 3, 3) and live == held          # all or none, and nothing leaks
    assert calls == (3, fail, 3, 0)                       # the small request allocates again
    assert size[0] == 4 * 101 + 8 * 100 + 16 * 102 and size[2] == 4 * 51 + 8 * 50 + 16 * 52


# buffers whose capacity decides whether they are allocated grow through it
@pytest.mark.parametrize("cap,source", [("pw_cap_t", "planewave.hip"), ("pw_cap_a", "planewave.hip"),
                                        ("pw_cap_e", "planewave.hip"), ("pw_cap_k", "planewave.hip"),
                                        ("ncell_alloc", "api.hip")])
def test_shared_capacities_grow_through_it(cap, source):
    with open(os.path.join(CSRC, source)) as fh:
        text = fh.read()
    assert re.search(r"device_grow\(pl->" + cap + r"\b", text)
    assigned = re.findall(r"pl->" + cap + r" = ([^;]*);", text)
    assert all(re.fullmatch(r"(pl->pw_cap_\w = )*0", v) for v in assigned), assigned
