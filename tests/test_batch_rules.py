"""Rules on the number of requests in a batch (csrc/batch_rules.h)."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_08151_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "batch_rules.h"
using namespace specv;
#define CHECK(ok, ...) do { if (!(ok)) { std::printf(__VA_ARGS__); return 1; } } while (0)
int main()
{
    // many positions per round trip where few pairs wait for it; elsewhere little is read behind an early difference; only shapes that are built
    for (int cus = 8; cus <= 304; cus += 8) for (int B = 1; B <= 9 * cus; ++B) {
        const DivergenceShape s = divergence_shape(B, cus);
        CHECK(s.threads * s.per == (B <= cus ? 4096 : 1024), "B=%d: %d x %d", B, s.threads, s.per);
        CHECK((s.threads == 512 && (s.per == 8 || s.per == 2)) || (s.threads == 256 && s.per == 4), "B=%d: %d x %d", B, s.threads, s.per);
    }
    std::puts("ok");
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_rules(tmp_path):
    src, exe = tmp_path / "rules.cpp", tmp_path / "rules"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    done = subprocess.run([str(exe)], capture_output=True, text=True)
    assert done.returncode == 0 and done.stdout.strip() == "ok", done.stdout
