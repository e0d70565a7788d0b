"""Geometry of the large-tile LM head, on the CPU: a C++ program that includes the kernel's own arithmetic (csrc/lm_head_tiles.h) walks every
row group, panel range, pass and wave of a matrix.  No device code runs."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_08151_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "lm_head_tiles.h"
using namespace specv;

#define CHECK(ok, ...) do { if (!(ok)) { std::printf(__VA_ARGS__); std::printf("\n"); return 1; } } while (0)

static int walk(int M, int V, int H, int cus, int cap)
{
    const MfmaLayout L = mfma_layout_for(M, V, cus, cap);
    CHECK(L.tm >= 9 && L.tm <= 16 && L.tm - L.tiles_lo <= 1, "M=%d: %d tiles per group", M, L.tm);
    CHECK(16 * (L.groups * L.tiles_lo + L.groups_hi) >= M && 16 * (L.groups * L.tiles_lo + L.groups_hi) < M + 16, "M=%d: rows", M);
    const int n_panels = (V + 15) / 16;
    const uint32_t panel_bytes = (uint32_t)H * 32u;
    const uint64_t matrix = (uint64_t)n_panels * panel_bytes;
    std::vector<int> owner(n_panels, 0);
    for (int range = 0; range < L.ranges; ++range) {
        const int p_begin = range * L.per_range, p_end = n_panels < p_begin + L.per_range ? n_panels : p_begin + L.per_range;
        if (p_begin >= p_end) continue;
        const int npass = (p_end - p_begin + kMfPassPanels - 1) / kMfPassPanels;
        CHECK(npass <= L.passes_per_range, "M=%d V=%d: %d passes", M, V, npass);
        const int full = mf_full_passes(p_begin, p_end, V);
        CHECK(full == npass || full == npass - 1, "M=%d V=%d range %d: %d full of %d passes", M, V, range, full, npass);
        CHECK(full == npass || (p_end - p_begin) % kMfPassPanels != 0 || p_end * 16 > V, "M=%d V=%d range %d: the last pass is a full one", M, V, range);
        for (int pass = 0; pass < npass; ++pass)
            for (int wave = 0; wave < kMfWaves; ++wave) {
                const PanelShare s = mf_panel_share(p_begin, p_end, pass, wave);
                CHECK(s.np >= 0 && s.np <= kMfTN && s.p0 >= p_begin && s.p0 + s.np <= p_end && s.p0 < p_end, "M=%d V=%d range %d pass %d wave %d: panels %d + %d", M, V, range, pass, wave, s.p0, s.np);
                if (pass < full) CHECK(s.np == kMfTN && (s.p0 + s.np) * 16 <= V, "M=%d V=%d range %d pass %d wave %d: not a full pass", M, V, range, pass, wave);
                for (int k = 0; k < s.np; ++k) ++owner[s.p0 + k];
                for (int tn = 0; tn < kMfTN; ++tn) {
                    // the requests of a slot cover one whole panel, slab by slab
                    const uint64_t from = (uint64_t)s.p0 * panel_bytes + mf_slot_bytes(s.np, tn, panel_bytes);
                    CHECK(from + panel_bytes <= matrix, "M=%d V=%d H=%d range %d pass %d wave %d slot %d: bytes up to %llu of %llu",
                          M, V, H, range, pass, wave, tn, (unsigned long long)(from + panel_bytes), (unsigned long long)matrix);
                    if (tn < s.np) CHECK(from == (uint64_t)(s.p0 + tn) * panel_bytes, "slot %d reads another panel", tn);
                }
            }
    }
    for (int p = 0; p < n_panels; ++p) CHECK(owner[p] == 1, "M=%d V=%d: panel %d owned %d times", M, V, p, owner[p]);
    return 0;
}

// one more group where fewer leave much of a range's last pass, or of the chip, without panels; else as few as 16 tiles each allow
static int groups_chosen()
{
    const struct { int M, V, groups; } expected[] = {
        {188, 151936, 1}, {576, 151936, 3}, {1152, 151936, 5}, {640, 32000, 4}, {768, 32000, 4}, {512, 32000, 2}, {704, 64000, 4}, {1600, 151936, 8}};
    for (const auto& e : expected) {
        const int g = mfma_layout_for(e.M, e.V, 256, 0).groups;
        CHECK(g == e.groups, "M=%d V=%d: %d groups", e.M, e.V, g);
    }
    return 0;
}

int main()
{
    if (groups_chosen()) return 1;
    const int Ms[] = {161, 192, 208, 209, 256, 257, 416, 417, 466, 576, 640, 1152, 1204, 1600, 4000};
    const int Vs[] = {1, 5, 16, 17, 999, 2000, 4095, 8200, 32000, 33000, 50021, 70003, 139281, 151936, 151937};
    const int Hs[] = {256, 1280, 4096}, cuss[] = {8, 64, 256, 304}, caps[] = {0, 144, 208, 256};
    for (int M : Ms) for (int V : Vs) for (int H : Hs) for (int cus : cuss) for (int cap : caps)
        if (walk(M, V, H, cus, cap)) return 1;
    std::puts("ok");
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_every_request_of_the_vocabulary_matrix_lies_inside_it(tmp_path):
    """Every panel is owned by one wave of one pass, a full pass has four panels per wave and no entry past the matrix, and the bytes that any panel slot of any wave requests (slots past a wave's share
    included) are bytes of the packed matrix."""
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    done = subprocess.run([str(exe)], capture_output=True, text=True)
    assert done.returncode == 0 and done.stdout.strip() == "ok", done.stdout
