"""The order in which attention deals (piece, kv head) to workgroups: heads first up to 65535 pieces, pieces first beyond."""
import pytest
import torch

from paper_2605_08151_amd import workloads as wl
from test_gpu_parity import _close, _oracle_attn, _step, sv  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gammas,Hq", [((0,), 4), ((0, 3), 32)], ids=["key_split", "row_split"])
def test_heads_first_and_pieces_first(sv, oracle, gammas, Hq):
    """1024 requests whose stated bound makes a work list of 64512 pieces at most, and of 65536: same cuts, same bits."""
    cfg = wl.VerifyConfig("order", 81, 1024, gammas, ("uniform", 1, 90), Hq, 2, 64, 64, sigma_qkv=1.0)
    b = wl.make_batch(cfg, device="cuda", with_lm_head=False)
    outs = []
    for bound in (8192 * 63, 8192 * 64):
        table = torch.full((1024, bound // 16), -1, dtype=torch.int32, device="cuda")
        table[:, :b["page_table"].shape[1]] = b["page_table"]
        step = _step(dict(b, max_kv_len=bound), cfg)
        outs.append(step.attn(b["q"], b["k_cache"], b["v_cache"], table, b["seq_lens"], b["qo_indptr"], b["scale"]))
        torch.cuda.synchronize()
        assert int(step.status.cpu()) == 0
        del step, table
    assert torch.equal(outs[0], outs[1])
    _close(outs[0].float().cpu().numpy(), _oracle_attn(oracle, b), "order", sharp=True)
