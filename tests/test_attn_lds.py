"""The attention kernels' small arrays in LDS (csrc/attn_lds.h): room for every page id, and masks on multiples of 8 bytes, whatever the chunk."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_08151_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "attn_lds.h"
using namespace specv;
int main()
{
    for (int keys = 1; keys <= 16384; ++keys) {
        const int slots = attn_page_slots(keys), pages = (keys + 15) / 16;
        if (slots < pages || slots < keys / 16 + 1 || slots > keys / 16 + 2) { std::printf("%d keys: %d slots", keys, slots); return 1; }
        if (attn_mask_offset(keys) % 8 != 0 || attn_mask_offset(keys) < (slots + 64) * 4) { std::printf("%d keys: masks at %d", keys, attn_mask_offset(keys)); return 1; }
    }
    std::puts("ok");
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_every_array_has_its_room_and_alignment(tmp_path):
    src, exe = tmp_path / "lds.cpp", tmp_path / "lds"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    done = subprocess.run([str(exe)], capture_output=True, text=True)
    assert done.returncode == 0 and done.stdout.strip() == "ok", done.stdout
