"""Rules on the number of requests in a batch (csrc/batch_rules.h)."""
import os
import shutil
import subprocess

import numpy as np
import pytest
import torch

from paper_2605_08151_amd import workloads as wl
from test_gpu_parity import _close, _oracle_attn, _step, sv  # noqa: F401

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_08151_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
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
    // attention's places: every request's pieces once each; requests that fill part of their places use all 8 XCDs x 4 shader engines alike (workgroups go round them in grid order)
    for (int Hkv = 1; Hkv <= 16; ++Hkv) for (int splits = 1; splits <= 33; ++splits) {
        const PieceTurn t = piece_turn(Hkv, splits);
        const int B = 32 * splits;
        for (int pieces = 1; pieces <= splits; ++pieces) {
            long load[32] = {}, sum = 0;
            for (int i = 0; i < B; ++i) for (int place = 0; place < splits; ++place) {
                const int k = splits == 1 ? place : piece_of_place(t, splits, place, i);
                CHECK(k >= 0 && k < splits, "Hkv=%d splits=%d: piece %d", Hkv, splits, k);
                for (int h = 0; k < pieces && h < Hkv; ++h, ++sum) ++load[(h + (long)Hkv * (place + (long)splits * i)) % 32];
            }
            for (long l : load) CHECK(l * 32 == sum || Hkv * splits > 32, "Hkv=%d splits=%d pieces=%d: %ld of %ld", Hkv, splits, pieces, l, sum);
        }
    }
    for (int splits = 2; splits <= 32; ++splits) for (int i = 0; i < 65536; ++i) {
        const PieceTurn t = piece_turn(1, splits);
        const int turn = (i >> t.shift) % splits;
        CHECK(piece_of_place(t, splits, turn, i) == 0 && piece_of_place(t, splits, turn == 0 ? splits - 1 : turn - 1, i) == splits - 1, "splits=%d i=%d", splits, i);
    }
    for (int splits : {33, 65535, 65536, 1 << 22}) for (int i : {0, 1, 4096, 65534})
        CHECK(piece_of_place(piece_turn(1, splits), splits, splits - 2, i) == splits - 2, "more than 32 workgroups: as they are");
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


@pytest.mark.gpu
@pytest.mark.parametrize("Hkv,gammas", [(1, (0,)), (2, (0, 3)), (4, (4,)), (4, (15,))], ids=["1_head", "2_heads", "4_heads", "row_split"])
@pytest.mark.parametrize("B", [9, 70])
def test_pieces_begin_a_place_on_with_every_request(sv, oracle, B, Hkv, gammas):
    """Chunks of 256 keys, one to three of three places filled: against the oracle, and bit for bit each request alone (request 0 of its batch: no turn)."""
    cfg = wl.VerifyConfig("turn", 60 + B + Hkv, B, gammas, ("uniform", 0, 700), 4 * Hkv, Hkv, 64, 64, sigma_qkv=1.0)
    b = wl.make_batch(cfg, device="cuda", with_lm_head=False)
    sv.spec_set_tuning("attn_plan", 2)
    sv.spec_set_tuning("attn_chunk", 256)
    step = _step(b, cfg)
    out = step.attn(b["q"], b["k_cache"], b["v_cache"], b["page_table"], b["seq_lens"], b["qo_indptr"], b["scale"]).clone()
    assert int(step.status.cpu()) == 0
    _close(out.float().cpu().numpy(), _oracle_attn(oracle, b), "turn", sharp=True)
    qo = b["qo_indptr"].cpu().numpy()
    for i in (1, 2, B - 1):
        one = slice(qo[i], qo[i + 1])
        single = torch.empty_like(b["q"][one])
        sv.spec_verify_attn(b["q"][one], b["k_cache"], b["v_cache"], b["page_table"][i:i + 1], b["seq_lens"][i:i + 1],
                            torch.tensor([0, qo[i + 1] - qo[i]], dtype=torch.int32, device="cuda"), single, None, b["max_kv_len"],
                            b["gamma_max"] + 1, b["scale"], step.status, step.attn_ws)
        assert torch.equal(single, out[one]), i
