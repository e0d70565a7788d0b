"""Row groups of 17 and 18 tiles of the large-tile LM head: the rule, its geometry, and the logits."""
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
#include <initializer_list>
#include <vector>
#include "lm_head_tiles.h"
using namespace specv;
#define CHECK(ok, ...) do { if (!(ok)) { std::printf(__VA_ARGS__); std::printf("\n"); return 1; } } while (0)
int main()
{
    const struct { int M, V, groups; } expected[] = {{272, 151936, 1}, {576, 151936, 2}, {1152, 151936, 4}, {576, 100000, 0}, {288, 32000, 0}, {1204, 151936, 0}, {256, 151936, 0}, {161, 500, 0}};
    for (const auto& e : expected) CHECK(mfma_tall_layout_for(e.M, e.V, 256).groups == e.groups, "M=%d V=%d: %d groups", e.M, e.V, mfma_tall_layout_for(e.M, e.V, 256).groups);
    const struct { int M, H, V; bool pays; } short_rows[] = {{260, 256, 64000, false}, {288, 512, 128256, false}, {257, 768, 60021, true}, {288, 1024, 62003, true},
        {560, 256, 32000, false}, {576, 256, 130000, true}, {560, 512, 32000, true}, {1152, 256, 128256, true}};
    for (const auto& e : short_rows) CHECK(mfma_tall_layout_for(e.M, e.V, 256).groups > 0 && mfma_tall_pays(mfma_tall_layout_for(e.M, e.V, 256), e.H) == e.pays, "M=%d H=%d V=%d", e.M, e.H, e.V);
    const int Vs[] = {1, 17, 999, 8200, 32000, 50021, 128256, 151937}, cuss[] = {8, 64, 256, 304};
    int tall = 0;
    for (int M = 161; M <= 2000; M += 7) for (int V : Vs) for (int cus : cuss) {
        const MfmaLayout L = mfma_tall_layout_for(M, V, cus);
        if (L.groups == 0) continue;
        ++tall;
        CHECK(L.tm == 17 || L.tm == 18, "M=%d V=%d: %d tiles", M, V, L.tm);
        CHECK(L.tm - L.tiles_lo <= 1 && 16 * (L.groups * L.tiles_lo + L.groups_hi) >= M && 16 * (L.groups * L.tiles_lo + L.groups_hi) < M + 16, "M=%d: rows", M);
        std::vector<int> owner((V + 15) / 16, 0);
        for (int range = 0; range < L.ranges; ++range) {
            const int p_begin = range * L.per_range, p_end = (int)owner.size() < p_begin + L.per_range ? (int)owner.size() : p_begin + L.per_range;
            for (int pass = 0; pass * kMfPassPanels < p_end - p_begin; ++pass)
                for (int wave = 0; wave < kMfWaves; ++wave) {
                    const PanelShare s = mf_panel_share(p_begin, p_end, pass, wave);
                    CHECK(s.p0 >= p_begin && s.p0 < p_end && s.p0 + s.np <= p_end, "M=%d V=%d: panels %d + %d", M, V, s.p0, s.np);
                    for (int k = 0; k < s.np; ++k) ++owner[s.p0 + k];
                }
        }
        for (int n : owner) CHECK(n == 1, "M=%d V=%d: a panel owned %d times", M, V, n);
    }
    CHECK(tall > 100, "%d layouts", tall);
    // every call reaches an instantiation that is built; what is not built is refused
    for (int tm = 1; tm <= 20; ++tm)
        for (MfmaLoads loads : {kBufferLoads, kGlobalLoads, kStreamLoads, kRowLoads, kRowStreamLoads}) {
            const bool built = loads <= kStreamLoads && (tm == 17 || tm == 18 || (tm == 8 && loads != kGlobalLoads) || ((tm == 9 || tm == 10) && loads == kStreamLoads));
            CHECK(mf_tile_built(loads, tm) == built, "loads %d, %d tiles", (int)loads, tm);
        }
    for (int M = 113; M <= 2000; M += M < 320 ? 1 : 7) for (int V : Vs) for (int cus : cuss) for (int H : {256, 768, 2048, 4096}) {
        if (M <= 160 && !lm_packed_large_tile(M, H, V, cus)) continue;
        MfmaLayout L = mfma_tall_layout_for(M, V, cus);
        const bool tall_one = L.groups > 0 && mfma_tall_pays(L, H);
        if (!tall_one) L = mfma_layout_for(M, V, cus, 0);
        const MfmaLoads loads = mfma_loads_for(L.groups, H, V);
        const bool in_tile_file = tall_one || (loads == kStreamLoads ? L.tm < 11 : loads == kBufferLoads && L.tm < 9);
        CHECK(in_tile_file ? mf_tile_built(loads, L.tm) : L.tm >= (loads == kStreamLoads ? 11 : 9) && L.tm <= 16, "M=%d V=%d H=%d: loads %d, %d tiles", M, V, H, (int)loads, L.tm);
    }
    std::puts("ok");
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_tall_layouts_own_every_row_and_panel_once(tmp_path):
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    done = subprocess.run([str(exe)], capture_output=True, text=True)
    assert done.returncode == 0 and done.stdout.strip() == "ok", done.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("M,V,H", [(257, 60021, 768), (272, 64000, 2560), (273, 64016, 1280), (288, 62003, 1024), (288, 100000, 768), (529, 32000, 1024), (561, 32000, 2048),
                                   (576, 31003, 512), (560, 32000, 512), (576, 130000, 256), (576, 137001, 256), (1057, 31000, 1024), (1152, 31999, 2048)])
def test_tall_groups(sv, oracle, M, V, H):
    """One, two and four groups; 17 and 18 tiles, the last one whole and ragged, groups of one tile fewer beside them; the three kinds of loads of W, stores nontemporal and
    not; one full pass, ragged last passes of two and of four panels per wave.  Same order of additions as the weight-streaming kernel: same bits."""
    g = torch.Generator(device="cuda").manual_seed(V + M)
    hidden = torch.randn((M, H), generator=g, device="cuda").to(torch.bfloat16)
    W = torch.randn((V, H), generator=g, device="cuda").to(torch.bfloat16)
    Wp = torch.empty(sv.spec_lm_head_packed_bytes(V, H) // 2, dtype=torch.bfloat16, device="cuda")
    sv.spec_lm_head_pack(W, Wp)
    logits = torch.full((M + 1, V), 7.0, device="cuda")
    sv.spec_lm_head_packed(hidden, Wp, logits[:M])
    rows = torch.tensor(sorted({0, M // 2, M - 17, M - 1}), device="cuda")
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


LINES_M, LINES_VH = [112, 113, 128, 129, 144, 145, 160], [(999, 4096), (36864, 1280), (36880, 2048), (50021, 1280), (57344, 256), (70000, 256), (64013, 1024)]

LINES_PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "lm_head_tiles.h"
int main(int, char** a) { std::puts(specv::lm_packed_large_tile(std::atoi(a[1]), std::atoi(a[2]), std::atoi(a[3]), 256) ? "large tile" : "weight-streaming"); return 0; }
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_which_kernel_the_lines_choose(tmp_path):
    """For 256 CUs, and the library's own choices (no tuning key set): the shapes that the next test runs, and measured ones on both sides of the other lines."""
    src, exe = tmp_path / "lines.cpp", tmp_path / "lines"
    src.write_text(LINES_PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    expected = {(M, H, V): M > 112 and (V, H) not in ((36864, 1280), (57344, 256)) for M in LINES_M for V, H in LINES_VH}
    assert sum(expected.values()) == 30
    expected |= {(128, 1024, 40000): True, (128, 512, 40000): False, (160, 512, 40000): False, (144, 512, 44000): False, (144, 256, 2000): False, (144, 512, 2000): True, (128, 256, 16000): True,
                 (128, 2560, 32000): False, (160, 2560, 32000): True, (113, 4096, 151936): True, (160, 2560, 64000): False, (161, 4096, 151936): False}
    for (M, H, V), large in expected.items():
        got = subprocess.run([str(exe), str(M), str(H), str(V)], capture_output=True, text=True, check=True).stdout.strip()
        assert got == ("large tile" if large else "weight-streaming"), (M, H, V)


@pytest.mark.gpu
@pytest.mark.parametrize("M", LINES_M)
@pytest.mark.parametrize("V,H", LINES_VH)
def test_lines_between_the_weight_streaming_and_the_large_tile_kernel(sv, oracle, M, V, H):
    """8, 9 and 10 row tiles, whole and ragged; less than a panel, 9 (ordinary and nontemporal loads), 13, 14, 16 and 18 panels per CU, aligned rows of logits and not."""
    g = torch.Generator(device="cuda").manual_seed(V + M)
    hidden = torch.randn((M, H), generator=g, device="cuda").to(torch.bfloat16)
    W = torch.randn((V, H), generator=g, device="cuda").to(torch.bfloat16)
    Wp = torch.empty(sv.spec_lm_head_packed_bytes(V, H) // 2, dtype=torch.bfloat16, device="cuda")
    sv.spec_lm_head_pack(W, Wp)
    logits = torch.full((M + 1, V), 7.0, device="cuda")
    sv.spec_lm_head_packed(hidden, Wp, logits[:M])
    rows = torch.tensor(sorted({0, M // 2, M - 1}), device="cuda")
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


@pytest.mark.gpu
@pytest.mark.parametrize("M", [113, 128, 160, 161, 256, 257, 400])
@pytest.mark.parametrize("V,H", [(999, 4096), (20001, 256), (32001, 512), (37003, 512), (49152, 1280), (70000, 256), (64013, 1024)])
def test_row_major_weights_through_the_large_tile_kernel(sv, oracle, M, V, H):
    """Ragged last panels (rows past the matrix repeat its last one), one group and two, ordinary and nontemporal loads, aligned rows of logits and not.  Same
    order of additions as on packed weights: same bits."""
    g = torch.Generator(device="cuda").manual_seed(V + M)
    hidden = torch.randn((M, H), generator=g, device="cuda").to(torch.bfloat16)
    W = torch.randn((V, H), generator=g, device="cuda").to(torch.bfloat16)
    logits = torch.full((M + 1, V), 7.0, device="cuda")
    sv.spec_lm_head(hidden, W, logits[:M])
    rows = torch.tensor(sorted({0, M // 2, M - 1}), device="cuda")
    ref = oracle.lm_head(wl.bf16_bits(hidden[rows]), wl.bf16_bits(W))
    assert np.abs(logits[rows].cpu().numpy() - ref).max() <= 1e-5 * math.sqrt(H) * np.abs(ref).max()
    assert (logits[M] == 7.0).all()
    Wp = torch.empty(sv.spec_lm_head_packed_bytes(V, H) // 2, dtype=torch.bfloat16, device="cuda")
    sv.spec_lm_head_pack(W, Wp)
    other = torch.empty((M, V), device="cuda")
    sv.spec_lm_head_packed(hidden, Wp, other)
    torch.cuda.synchronize()
    assert torch.equal(other, logits[:M])
