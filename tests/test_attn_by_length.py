"""Attention with the requests taken longest first (at most 64 requests, fixed chunks, more workgroups than CUs): same bits as in the order given."""
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
