"""Attention with the requests taken longest first (at most 64 requests, fixed chunks, more workgroups than CUs): right, and the same bits as in the order given."""
import numpy as np
import pytest
import torch

from paper_2605_08151_amd import workloads as wl
from test_gpu_parity import _close, _oracle_attn, _step, sv  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [33, 64, 65])
@pytest.mark.parametrize("gammas,Hq", [((0,), 8), ((4,), 32), ((0, 3, 8), 64)], ids=["decode", "two_tiles", "row_split"])
def test_longest_first(sv, oracle, B, gammas, Hq):
    """33 x 8 and 64 x 8 workgroups by length, 65 in the order given; contexts of zero, equal ones among them, and one request with lengths out of range."""
    cfg = wl.VerifyConfig("by_length", 90 + B, B, gammas, ("uniform", 0, 600), Hq, 8, 64, 64, sigma_qkv=1.0)
    b = wl.make_batch(cfg, device="cuda", with_lm_head=False)
    lens = b["seq_lens"].clone()
    lens[3] = lens[7] = lens[B - 1]                       # (cut to what their pages hold)
    lens = torch.minimum(lens, b["seq_lens"])
    lens[5] = 0
    b = dict(b, seq_lens=lens)
    step = _step(b, cfg)
    out = step.attn(b["q"], b["k_cache"], b["v_cache"], b["page_table"], lens, b["qo_indptr"], b["scale"]).clone()
    _close(out.float().cpu().numpy(), _oracle_attn(oracle, b), "by length", sharp=True)
    assert int(step.status.cpu()) == 0
    qo = b["qo_indptr"].cpu().numpy()
    for i in (0, 3, 5, B - 1):                            # alone: few workgroups, the order given
        one = slice(qo[i], qo[i + 1])
        single = torch.empty_like(b["q"][one])
        status = torch.zeros(1, dtype=torch.int32, device="cuda")
        sv.spec_verify_attn(b["q"][one], b["k_cache"], b["v_cache"], b["page_table"][i:i + 1], lens[i:i + 1],
                            torch.tensor([0, qo[i + 1] - qo[i]], dtype=torch.int32, device="cuda"), single, None, b["max_kv_len"],
                            b["gamma_max"] + 1, b["scale"], status, step.attn_ws)
        assert int(status.cpu()) == 0
        _close(single.float().cpu().numpy(), out[one].float().cpu().numpy(), "alone", sharp=True)
    bad = lens.clone()
    bad[9], bad[11] = -1, 1 << 30
    again = step.attn(b["q"], b["k_cache"], b["v_cache"], b["page_table"], bad, b["qo_indptr"], b["scale"])
    keep = np.ones(qo[-1], bool)
    for i in (9, 11):
        keep[qo[i]:qo[i + 1]] = False
    keep = torch.from_numpy(keep).cuda()
    assert torch.equal(again[keep], out[keep]) and int(step.status.cpu()) == sv.FLAG_BAD_LENGTH


@pytest.mark.parametrize("B", [33, 64])
@pytest.mark.parametrize("chunk", [256, 1024], ids=["split", "whole"])
@pytest.mark.parametrize("gammas,Hq", [((0,), 8), ((4,), 32), ((0, 3, 8), 64)], ids=["decode", "two_tiles", "row_split"])
def test_same_bits_as_in_the_order_given(sv, B, chunk, gammas, Hq):
    """The same requests and chunks, once as a batch of at most 64 and once with requests of one row and no context behind them, 65 in all, which takes the order given."""
    cfg = wl.VerifyConfig("by_length_bits", 190 + B, B, gammas, ("uniform", 0, 900), Hq, 8, 64, 64, sigma_qkv=1.0, pool_slack=1.5)
    b = wl.make_batch(cfg, device="cuda", with_lm_head=False)
    assert int(b["free_count"].cpu()) >= 65 - B and b["max_kv_len"] > 512
    sv.spec_set_tuning("attn_plan", 2)
    sv.spec_set_tuning("attn_chunk", chunk)
    try:
        step = _step(b, cfg)                              # (the workspace is that of these chunks)
        out = step.attn(b["q"], b["k_cache"], b["v_cache"], b["page_table"], b["seq_lens"], b["qo_indptr"], b["scale"]).clone()
        lse = step.lse.clone()
        more = 65 - B
        table = torch.cat([b["page_table"], torch.full((more, b["page_table"].shape[1]), -1, dtype=torch.int32, device="cuda")])
        table[B:, 0] = b["free_list"][:more]
        qo = torch.cat([b["qo_indptr"], b["qo_indptr"][-1] + 1 + torch.arange(more, dtype=torch.int32, device="cuda")])
        long = dict(b, B=65, M=b["M"] + more, q=torch.cat([b["q"], b["q"][:more]]), seq_lens=torch.cat([b["seq_lens"], torch.zeros(more, dtype=torch.int32, device="cuda")]))
        given = _step(long, cfg)
        other = given.attn(long["q"], b["k_cache"], b["v_cache"], table, long["seq_lens"], qo, b["scale"])
        assert int(step.status.cpu()) == 0 and int(given.status.cpu()) == 0
        torch.cuda.synchronize()
    finally:
        sv.spec_set_tuning("attn_plan", 0)
        sv.spec_set_tuning("attn_chunk", 0)
    assert torch.equal(out, other[:b["M"]]) and torch.equal(lse, given.lse[:b["M"]])
