"""The last pass of a panel range in the large-tile LM head: 1..16 panels, served by code for two, three or four panels per wave."""
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
int main()
{
    for (int n_own = 1; n_own <= 200; ++n_own) {
        const int slots = mf_last_slots(n_own), npass = (n_own + kMfPassPanels - 1) / kMfPassPanels;
        if (slots < 2 || slots > kMfTN) { std::printf("%d panels: %d slots", n_own, slots); return 1; }
        for (int wave = 0; wave < kMfWaves; ++wave)
            if (mf_panel_share(0, n_own, npass - 1, wave).np > slots) { std::printf("%d panels: wave %d has more than %d", n_own, wave, slots); return 1; }
        for (int V = n_own * 16; V > n_own * 16 - 16; --V) {
            const int full = mf_full_passes(0, n_own, V);
            if (full < npass - 1 || (full == npass && slots != kMfTN)) { std::printf("%d panels: %d full passes of %d", n_own, full, npass); return 1; }
        }
    }
    std::puts("ok");
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_the_last_pass_has_a_slot_for_every_panel_of_a_wave(tmp_path):
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    done = subprocess.run([str(exe)], capture_output=True, text=True)
    assert done.returncode == 0 and done.stdout.strip() == "ok", done.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("M", [177, 400])
@pytest.mark.parametrize("panels", [2, 5, 8, 9, 12, 13, 17, 20, 24, 28, 31])
def test_large_tile_lm_head_last_passes(sv, oracle, M, panels):
    """Every panel count of a last pass at which the code changes, alone and after a full pass (ranges are one per CU and row group; the
    last range is short and its last panel ragged).  Same order of additions as the weight-streaming kernel: same bits."""
    H = 256
    ranges = torch.cuda.get_device_properties(0).multi_processor_count // (1 if M <= 256 else 2) // 8 * 8
    V = panels * ranges * 16 - 16 * (panels // 2) - 5
    g = torch.Generator(device="cuda").manual_seed(panels + M)
    hidden = torch.randn((M, H), generator=g, device="cuda").to(torch.bfloat16)
    W = torch.randn((V, H), generator=g, device="cuda").to(torch.bfloat16)
    Wp = torch.empty(sv.spec_lm_head_packed_bytes(V, H) // 2, dtype=torch.bfloat16, device="cuda")
    sv.spec_lm_head_pack(W, Wp)
    logits = torch.full((M + 1, V), 7.0, device="cuda")
    sv.spec_lm_head_packed(hidden, Wp, logits[:M])
    rows = torch.tensor([0, M // 2, M - 1], device="cuda")
    ref = oracle.lm_head(wl.bf16_bits(hidden[rows]), wl.bf16_bits(W))
    assert np.abs(logits[rows].cpu().numpy() - ref).max() <= 1e-5 * math.sqrt(H) * np.abs(ref).max()
    assert (logits[M] == 7.0).all()
    other = torch.empty((M, V), device="cuda")
    sv.spec_set_tuning("lm_packed_tile", 1)
    try:
        sv.spec_lm_head_packed(hidden, Wp, other)
        torch.cuda.synchronize()
    finally:
        sv.spec_set_tuning("lm_packed_tile", 0)
    assert torch.equal(other, logits[:M])
