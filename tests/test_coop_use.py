"""When a solver takes its cooperative form again after launches that other
work kept from coming together: the rule alone, compiled for the host."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1602_03643_amd", "csrc")

MAIN = r"""
#include "coop_use.hpp"
#include <cstdio>
static int until(oasis::CoopUse &u) {   // solves in the launched form before the next cooperative one
    int n = 0;
    while (!u.next() && n < 5000) ++n;
    return n;
}
int main() {
    oasis::CoopUse u;
    std::printf("%d", until(u));
    for (int k = 0; k < 9; ++k) {
        u.gave_up();
        std::printf(" %d", until(u));
    }
    u.worked();
    std::printf(" %d", until(u));
    u.gave_up();
    std::printf(" %d", until(u));
    u.never = true;
    std::printf(" %d\n", until(u));
}
"""


def test_rests_and_comes_back(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "use.cpp", tmp_path / "use"
    src.write_text(MAIN)
    subprocess.run([cxx, "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    got = [int(v) for v in subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()]
    # at once; 16, doubled to 1024 while it fails; at once and 16 again after a success; never
    assert got == [0, 16, 32, 64, 128, 256, 512, 1024, 1024, 1024, 0, 16, 5000]
