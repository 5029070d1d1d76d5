"""The grid barrier's arrival test where its 32-bit counter wraps, compiled for
the host (no GPU needed)."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(__file__)), "paper_1905_09598_amd", "csrc")

# Barrier number n of G workgroups: not reached by the arrivals of barrier
# n - 1 nor by all but one of its own, reached by all of them and still
# reached while workgroups already arrive at barrier n + 1.
SOURCE = """
#include "som_barrier.h"
#include <cstdio>
int main() {
    const unsigned grids[] = {2, 33, 511, 512, 4096};
    for (unsigned G : grids) {
        const unsigned long long wrap = (1ull << 32) / G, half = wrap / 2;
        const unsigned long long around[] = {2, half, wrap, 2 * wrap};
        for (unsigned long long at : around)
            for (unsigned long long n = at - 1; n <= at + 2; ++n) {
                const unsigned long long done = n * G;
                const unsigned target = (unsigned)n * G;
                for (unsigned k = 0; k < G; ++k)
                    if (som::arrivals_reached((unsigned)(done - G + k), target)) {
                        std::printf("G %u: barrier %llu passed early\\n", G, n);
                        return 1;
                    }
                for (unsigned k = 0; k < G; ++k)
                    if (!som::arrivals_reached((unsigned)(done + k), target)) {
                        std::printf("G %u: barrier %llu missed\\n", G, n);
                        return 1;
                    }
            }
    }
    return 0;
}
"""


def test_arrivals_are_counted_across_the_wrap(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "arrivals.cpp", tmp_path / "arrivals"
    src.write_text(SOURCE)
    subprocess.run([cxx, "-std=c++17", "-O1", f"-I{CSRC}", str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
