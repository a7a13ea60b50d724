"""The check that a call's outputs are disjoint from its inputs and from each
other sees every array, however many a call has (host code, compiled here)."""
import os
import subprocess

import pytest

from paper_2505_06703_amd import build as hsbuild

PROGRAM = r"""
#include "hs_ranges.h"
#include <cstdio>
#include <cstdlib>
int main(int, char **argv)
{
    const int n = std::atoi(argv[1]), at = std::atoi(argv[2]);
    const bool input = argv[3][0] == 'i';
    static char mem[64 * 100];
    hs::Ranges outs, ins;
    for (int k = 0; k < n; ++k) {  // 16 bytes each, 64 apart: outputs, then inputs
        outs.push_back({mem + 64 * k, 16, "out"});
        ins.push_back({mem + 64 * k + 32, 16, "in"});
    }
    hs::Clash c;
    if (hs::find_clash(outs, ins, c)) return 1;
    // one more, on the last byte of number `at`
    (input ? ins : outs).push_back({mem + 64 * at + 15, 1, "last"});
    if (!hs::find_clash(outs, ins, c)) return 2;
    if (c.input != input) return 3;
    return outs.size() + ins.size() == 2 * (size_t)n + 1 ? 0 : 4;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("ranges")
    src, exe = d / "t.cpp", d / "t"
    src.write_text(PROGRAM)
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-O1", "-Wall", "-I", hsbuild.CSRC, str(src), "-o", str(exe)],
                   check=True, timeout=120)
    return str(exe)


@pytest.mark.parametrize("arrays", [1, 15, 16, 17, 40])
@pytest.mark.parametrize("kind", ["input", "output"])
def test_the_last_array_counts(program, arrays, kind):
    for at in {0, arrays - 1}:
        assert subprocess.run([program, str(arrays), str(at), kind], timeout=30).returncode == 0
