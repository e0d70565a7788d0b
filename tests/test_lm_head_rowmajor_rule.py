"""Which shapes of row-major weights go through the large-tile kernel: the rule at measured shapes on both sides, and the logits where the other kernel serves them."""
import math
import os
import shutil
import subprocess

import numpy as np
import pytest
import torch

from paper_2605_08151_amd import workloads as wl
from test_gpu_parity import sv  # noqa: F401

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_08151_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "lm_head_tiles.h"
using namespace specv;
#define CHECK(ok, ...) do { if (!(ok)) { std::printf(__VA_ARGS__); return 1; } } while (0)
int main()
{
    const struct { int M, H, V; bool large; } measured[] = {
        {192, 4096, 151936, true}, {200, 2560, 64000, true}, {300, 1024, 64000, true}, {400, 2048, 50021, true}, {768, 2560, 50021, true}, {1152, 4096, 151936, true}, {2048, 1024, 100000, true},
        {576, 4096, 151936, true}, {576, 6144, 151936, true}, {576, 8192, 151936, true}, {1152, 6144, 151936, true}, {768, 6144, 128256, true}, {576, 6144, 128256, false},
        {576, 2560, 64000, false}, {576, 4096, 64000, false}, {576, 1280, 128256, false}, {576, 2560, 128256, false}, {576, 2048, 151936, false}, {576, 5120, 128256, false},
        {768, 2560, 64000, false}, {1152, 2048, 64000, false}, {1152, 2560, 32000, false}, {1152, 3072, 100000, false}, {1206, 2560, 50021, false},
        {177, 256, 4000, false}, {192, 256, 12001, false}, {208, 256, 12001, true}, {177, 512, 4000, true}, {300, 256, 28002, false}, {1152, 256, 8000, false}, {257, 256, 20001, true},
        {128, 1280, 24001, true}, {160, 2048, 20001, true}, {128, 2560, 24001, false}, {160, 2560, 20001, false}, {128, 2048, 28001, false}, {128, 4096, 28001, true}, {128, 4096, 8001, false},
        {128, 2560, 24000, false}, {128, 2560, 64000, false}, {128, 2560, 64001, true}, {128, 4096, 151936, true}, {112, 4096, 151936, false}};
    for (const auto& m : measured) CHECK(lm_rowmajor_large_tile(m.M, m.H, m.V, 256) == m.large, "M=%d H=%d V=%d", m.M, m.H, m.V);
    const int Vs[] = {1, 17, 999, 8200, 32000, 50021, 128256, 151937}, cuss[] = {8, 64, 256, 304}, Hs[] = {64, 256, 320, 512, 2560, 4096};
    int taken = 0;
    for (int M = 1; M <= 3000; M += M < 400 ? 1 : 13) for (int V : Vs) for (int cus : cuss) for (int H : Hs) {
        if (!lm_rowmajor_large_tile(M, H, V, cus)) continue;
        ++taken;
        const MfmaLayout L = mfma_layout_for(M, V, cus, 0);
        CHECK(M > 112 && H % 256 == 0 && L.tm >= 8 && L.tm <= 16, "M=%d H=%d V=%d: %d tiles", M, H, V, L.tm);
    }
    CHECK(taken > 1000, "%d", taken);
    CHECK(!lm_rowmajor_large_tile(300, 1024, 4000000, 256), "beyond 32-bit row offsets");
    std::puts("ok");
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_rule(tmp_path):
    src, exe = tmp_path / "rule.cpp", tmp_path / "rule"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    done = subprocess.run([str(exe)], capture_output=True, text=True)
    assert done.returncode == 0 and done.stdout.strip() == "ok", done.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("M,V,H", [(300, 28002, 256), (177, 4000, 256), (576, 64000, 512), (1152, 8000, 256)])
def test_shapes_of_the_other_kernel(sv, oracle, M, V, H):
    g = torch.Generator(device="cuda").manual_seed(V + M)
    hidden = torch.randn((M, H), generator=g, device="cuda").to(torch.bfloat16)
    W = torch.randn((V, H), generator=g, device="cuda").to(torch.bfloat16)
    logits = torch.full((M + 1, V), 7.0, device="cuda")
    sv.spec_lm_head(hidden, W, logits[:M])
    rows = torch.tensor(sorted({0, M // 2, M - 1}), device="cuda")
    ref = oracle.lm_head(wl.bf16_bits(hidden[rows]), wl.bf16_bits(W))
    assert np.abs(logits[rows].cpu().numpy() - ref).max() <= 1e-5 * math.sqrt(H) * np.abs(ref).max()
    assert (logits[M] == 7.0).all()
    exact = hidden.double() @ W.double().t()
    assert ((logits[:M].double() - exact).abs() <= (hidden.double().abs() @ W.double().abs().t()) * H * 2.0 ** -24).all()
