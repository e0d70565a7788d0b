"""Rules on the number of requests in a batch (csrc/batch_rules.h)."""
import os
import shutil
import subprocess

import numpy as np
import pytest
import torch

from test_gpu_parity import sv  # noqa: F401

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_08151_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "batch_rules.h"
using namespace specv;
#define CHECK(ok, ...) do { if (!(ok)) { std::printf(__VA_ARGS__); return 1; } } while (0)
int main()
{
    // many positions per round trip where few pairs wait for it; elsewhere little is read behind an early difference; only shapes that are built
    for (int B = 1; B <= 9 * 256; ++B) {
        const DivergenceShape s = divergence_shape(B);
        CHECK(s.threads * s.per == (B <= 256 ? 4096 : 1024), "B=%d: %d x %d", B, s.threads, s.per);
        CHECK((s.threads == 512 && (s.per == 8 || s.per == 2)) || (s.threads == 256 && s.per == 4), "B=%d: %d x %d", B, s.threads, s.per);
    }
    CHECK(kMergeCounted >= 256 && kMergeCounted <= 2048, "requests are counted up to %d", kMergeCounted);
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


@pytest.mark.gpu
@pytest.mark.parametrize("B", [1024, 1025, 9001])
def test_merge_finds_its_request(sv, B):
    """Requests of one and two rows, split by the bound they state: every row merged with its own request's keys, on both
    sides of the line between counting and searching.  V holds the number of its page's request, so that every output row names its request."""
    rng = np.random.default_rng(B)
    rows = rng.integers(1, 3, B)
    qo = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    M, lens = int(qo[-1]), rng.integers(0, 14, B).astype(np.int32)
    bound = 16 * 321                                          # (5136 keys: two chunks)
    table = torch.zeros((B, 321), dtype=torch.int32, device="cuda")
    table[:, 0] = torch.arange(B, dtype=torch.int32)
    k = torch.zeros((B, 1, 16, 128), dtype=torch.bfloat16, device="cuda")
    v = torch.empty_like(k)
    v[:] = (torch.arange(B, device="cuda") % 251).to(torch.bfloat16).view(B, 1, 1, 1)
    v[..., 64:] = (torch.arange(B, device="cuda") // 251).to(torch.bfloat16).view(B, 1, 1, 1)
    q = torch.zeros((M, 2, 128), dtype=torch.bfloat16, device="cuda")
    out = torch.full_like(q, -5.0)
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = torch.empty(sv.spec_verify_attn_workspace_bytes(B, M, 2, 1, 128, bound, 2), dtype=torch.uint8, device="cuda")
    dev = lambda a: torch.from_numpy(a).cuda()                # noqa: E731
    sv.spec_verify_attn(q, k, v, table, dev(lens), dev(qo), out, None, bound, 2, 1.0, status, ws)
    got, owner = out.float().cpu().numpy(), np.repeat(np.arange(B), rows)
    assert int(status.cpu()) == 0
    assert np.abs(got[:, :, :64] - (owner % 251)[:, None, None]).max() < 0.5 and np.abs(got[:, :, 64:] - (owner // 251)[:, None, None]).max() < 0.5
