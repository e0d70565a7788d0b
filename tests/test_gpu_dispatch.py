"""GPU parity at the lines of the launch rules: both sides of a rule on sizes against the CPU oracle, at sizes where the variant behind
the line can go wrong.  Tolerances as in test_gpu_parity.py."""
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2605_08151_amd import workloads as wl  # noqa: E402
from test_gpu_parity import _accept_both, _assert_same, _close, _oracle_attn, _qo, _step, sv  # noqa: E402,F401


@pytest.mark.parametrize("gammas,Hq", [((0,), 8), ((4,), 32), ((0, 3, 8), 64)], ids=["decode", "two_tiles", "row_split"])
def test_attention_streaming_and_cached_loads(sv, oracle, gammas, Hq):
    """Where the stated bound exceeds 3/4 of the memory-side cache (here 3 requests x 8 kv heads x 16384 keys) the kernels look at the batch before
    they choose how to load K/V, up to it they do not (this batch is a small one, ordinary loads).  Same bits on both sides of the line."""
    cfg = wl.VerifyConfig("stream", 71, 3, gammas, ("uniform", 200, 2500), Hq, 8, 64, 64, sigma_qkv=1.0)
    b = wl.make_batch(cfg, device="cuda", with_lm_head=False)
    table = torch.full((3, 1040), -1, dtype=torch.int32, device="cuda")
    table[:, :b["page_table"].shape[1]] = b["page_table"]
    outs = []
    for bound in (16384, 16385):
        step = _step(dict(b, max_kv_len=bound), cfg)
        outs.append(step.attn(b["q"], b["k_cache"], b["v_cache"], table, b["seq_lens"], b["qo_indptr"], b["scale"]))
        torch.cuda.synchronize()
        assert int(step.status.cpu()) == 0
    assert torch.equal(outs[0], outs[1])
    _close(outs[1].float().cpu().numpy(), _oracle_attn(oracle, b), "stream", sharp=True)


@pytest.mark.parametrize("gammas,Hq", [((0,), 8), ((4,), 32), ((0, 3, 8), 64)], ids=["decode", "two_tiles", "row_split"])
def test_attention_over_more_keys_than_the_cache_holds(sv, oracle, gammas, Hq):
    """3 requests x 8 kv heads x 16450..16800 keys (more than 3/4 of the memory-side cache: nontemporal loads), each also alone under the same
    bounds (ordinary loads) and all with the first pages of request 0 mapped into the others (a common prefix: ordinary loads where it is
    shared).  Same cuts, so same bits alone and together."""
    cfg = wl.VerifyConfig("many_keys", 72, 3, gammas, ("uniform", 16450, 16800), Hq, 8, 64, 64, sigma_qkv=1.0)
    b = wl.make_batch(cfg, device="cuda", with_lm_head=False)
    assert int(b["seq_lens"].sum()) * 8 * 512 > 192 << 20
    sv.spec_set_tuning("attn_plan", 2)
    sv.spec_set_tuning("attn_chunk", 2048)
    try:
        step = _step(b, cfg)
        together = step.attn(b["q"], b["k_cache"], b["v_cache"], b["page_table"], b["seq_lens"], b["qo_indptr"], b["scale"]).clone()
        qo = b["qo_indptr"].cpu().numpy()
        for i in range(3):
            one = slice(qo[i], qo[i + 1])
            out, status = torch.empty_like(b["q"][one]), torch.zeros(1, dtype=torch.int32, device="cuda")
            sv.spec_verify_attn(b["q"][one], b["k_cache"], b["v_cache"], b["page_table"][i:i + 1], b["seq_lens"][i:i + 1],
                                torch.tensor([0, qo[i + 1] - qo[i]], dtype=torch.int32, device="cuda"), out, None, b["max_kv_len"],
                                b["gamma_max"] + 1, b["scale"], status, step.attn_ws)
            assert torch.equal(out, together[one]) and int(status.cpu()) == 0
        _close(together.float().cpu().numpy(), _oracle_attn(oracle, b), "many keys", sharp=True)
        table = b["page_table"].clone()
        table[1:, :300] = table[0, :300]
        shared = dict(b, page_table=table)
        out = step.attn(b["q"], b["k_cache"], b["v_cache"], table, b["seq_lens"], b["qo_indptr"], b["scale"])
        assert torch.equal(out[:qo[1]], together[:qo[1]])
        _close(out.float().cpu().numpy(), _oracle_attn(oracle, shared), "shared prefix", sharp=True)
        assert int(step.status.cpu()) == 0
    finally:
        sv.spec_set_tuning("attn_plan", 0)
        sv.spec_set_tuning("attn_chunk", 0)


@pytest.mark.parametrize("M", [1, 37, 160])
@pytest.mark.parametrize("V", [196608, 196612, 196625])
def test_packed_lm_head_streaming_and_cached_weights(sv, oracle, M, V):
    """The vocabulary matrix by nontemporal loads above 3/8 of the memory-side cache (H = 256: more than 196608 entries)."""
    g = torch.Generator(device="cuda").manual_seed(V + M)
    hidden = torch.randn((M, 256), generator=g, device="cuda").to(torch.bfloat16)
    W = torch.randn((V, 256), generator=g, device="cuda").to(torch.bfloat16)
    Wp = torch.empty(sv.spec_lm_head_packed_bytes(V, 256) // 2, dtype=torch.bfloat16, device="cuda")
    sv.spec_lm_head_pack(W, Wp)
    logits = torch.full((M, V), 7.0, device="cuda")
    sv.spec_lm_head_packed(hidden, Wp, logits)
    ref = oracle.lm_head(wl.bf16_bits(hidden), wl.bf16_bits(W))
    err = np.abs(logits.cpu().numpy() - ref).max()
    assert err <= 1e-5 * math.sqrt(256) * np.abs(ref).max(), err


@pytest.mark.parametrize("M", [1, 17, 80, 160])
@pytest.mark.parametrize("V", [5, 4099, 32768, 32769, 70003])
def test_row_major_lm_head_through_the_packed_kernel(sv, oracle, M, V):
    """Up to 160 rows and H a multiple of 256 a row-major matrix goes through the packed kernel (128 bytes of 8 rows per load): last panels of
    1 .. 15 entries, up to 8 panels per CU (4 waves) and more (8 waves).  Same order of additions as from packed weights: same bits."""
    g = torch.Generator(device="cuda").manual_seed(V + M)
    hidden = torch.randn((M, 512), generator=g, device="cuda").to(torch.bfloat16)
    W = torch.randn((V, 512), generator=g, device="cuda").to(torch.bfloat16)
    logits = torch.full((M + 1, V), 7.0, device="cuda")
    sv.spec_lm_head(hidden, W, logits[:M])
    ref = oracle.lm_head(wl.bf16_bits(hidden), wl.bf16_bits(W))
    err = np.abs(logits[:M].cpu().numpy() - ref).max()
    assert err <= 1e-5 * math.sqrt(512) * np.abs(ref).max(), err
    assert (logits[M] == 7.0).all()                        # nothing past the last row
    Wp = torch.empty(sv.spec_lm_head_packed_bytes(V, 512) // 2, dtype=torch.bfloat16, device="cuda")
    sv.spec_lm_head_pack(W, Wp)
    packed = torch.empty((M, V), device="cuda")
    sv.spec_lm_head_packed(hidden, Wp, packed)
    assert torch.equal(packed, logits[:M])


def _both_layouts(sv, hidden, W):
    """logits of the row-major and of the packed matrix"""
    M, V, H = hidden.shape[0], W.shape[0], W.shape[1]
    logits, packed = torch.full((M, V), 7.0, device="cuda"), torch.full((M, V), 7.0, device="cuda")
    sv.spec_lm_head(hidden, W, logits)
    Wp = torch.empty(sv.spec_lm_head_packed_bytes(V, H) // 2, dtype=torch.bfloat16, device="cuda")
    sv.spec_lm_head_pack(W, Wp)
    sv.spec_lm_head_packed(hidden, Wp, packed)
    return logits, packed


@pytest.mark.parametrize("M", [1, 32, 33, 160])
@pytest.mark.parametrize("V", [28672, 28673, 32768, 32769, 40960, 40961])
def test_row_major_lm_head_at_the_lines_of_its_routes(sv, oracle, M, V):
    """7, 8, 9 and 10, 11 panels per CU (of 256), up to 32 rows and more: the 4-wave kernel on one side, the packed kernel's row-major form on the other."""
    g = torch.Generator(device="cuda").manual_seed(V + M)
    hidden = torch.randn((M, 256), generator=g, device="cuda").to(torch.bfloat16)
    W = torch.randn((V, 256), generator=g, device="cuda").to(torch.bfloat16)
    logits, packed = _both_layouts(sv, hidden, W)
    ref = oracle.lm_head(wl.bf16_bits(hidden), wl.bf16_bits(W))
    assert np.abs(logits.cpu().numpy() - ref).max() <= 1e-5 * math.sqrt(256) * np.abs(ref).max()
    assert torch.equal(packed, logits)


@pytest.mark.parametrize("M", [5, 80, 160])
@pytest.mark.parametrize("V,H", [(32000, 1792), (32767, 2048)])
def test_few_panels_and_a_matrix_beyond_the_cache(sv, oracle, V, H, M):
    """At most 8 panels per CU (4 waves, two slabs in the ring) and nontemporal weights, both layouts."""
    assert V * H * 2 > 96 << 20
    g = torch.Generator(device="cuda").manual_seed(V + M)
    hidden = torch.randn((M, H), generator=g, device="cuda").to(torch.bfloat16)
    W = torch.randn((V, H), generator=g, device="cuda").to(torch.bfloat16)
    logits, packed = _both_layouts(sv, hidden, W)
    rows = torch.tensor(sorted({0, M // 2, M - 1}), device="cuda")
    ref = oracle.lm_head(wl.bf16_bits(hidden[rows]), wl.bf16_bits(W))
    assert np.abs(logits[rows].cpu().numpy() - ref).max() <= 1e-5 * math.sqrt(H) * np.abs(ref).max()
    assert torch.equal(packed, logits)
    try:
        for waves in (4, 8):
            sv.spec_set_tuning("lm_packed_waves", waves)
            assert torch.equal(_both_layouts(sv, hidden, W)[1], logits)
    finally:
        sv.spec_set_tuning("lm_packed_waves", 0)


@pytest.mark.parametrize("M", [1, 80, 160])
@pytest.mark.parametrize("V,H", [(50000, 1280), (62000, 1280), (62000, 1024)])
def test_row_major_lm_head_by_ordinary_and_nontemporal_loads(sv, oracle, M, V, H):
    """A matrix beyond 3/8 of the memory-side cache: rows of whole 2 KB or panel slots nearly all filled (13 and 16 of 16 per CU)."""
    assert V * H * 2 > 96 << 20
    g = torch.Generator(device="cuda").manual_seed(V + M)
    hidden = torch.randn((M, H), generator=g, device="cuda").to(torch.bfloat16)
    W = torch.randn((V, H), generator=g, device="cuda").to(torch.bfloat16)
    logits, packed = _both_layouts(sv, hidden, W)
    rows = torch.tensor(sorted({0, M // 2, M - 1}), device="cuda")
    ref = oracle.lm_head(wl.bf16_bits(hidden[rows]), wl.bf16_bits(W))
    assert np.abs(logits[rows].cpu().numpy() - ref).max() <= 1e-5 * math.sqrt(H) * np.abs(ref).max()
    assert torch.equal(packed, logits)


@pytest.mark.parametrize("V,B", [(1, 3), (4095, 5), (4096, 5), (4097, 5), (8193, 5), (50021, 7), (50021, 60), (300, 1366), (300, 1367)])
def test_sampled_acceptance_of_small_batches(sv, oracle, V, B):
    """Up to 8 Mi logits every row is summed in fp64 and the decision is taken by every workgroup of the residual launch (180 rows x 50021
    are just beyond), in up to 4096 rows (1366 requests have 4096, 1367 have 4100).  Rows that start at odd multiples of 4 bytes, last segments of 1, 4095 and 4096 entries."""
    rng = np.random.default_rng(V + B)
    gammas = np.full(B, 3)
    gammas[::3] = 0
    qo = _qo(gammas)
    logits = rng.normal(0, 2.0, (qo[-1], V)).astype(np.float32)
    cfg = wl.VerifyConfig("s", V, B, (3,), ("const", 1), 8, 1, 64, V)
    dp, tokens = wl.draft_probs_noisy(cfg, torch.from_numpy(qo), torch.from_numpy(logits), noise_std=0.5)
    temp = np.full(B, 0.8, np.float32)
    temp[1::4] = 0.0
    got, ref = _accept_both(sv, oracle, logits, tokens.numpy(), dp.numpy(), temp, rng.integers(0, 2 ** 63, B, dtype=np.uint64), 9, qo, 3)
    _assert_same(got, ref, gammas)
    assert got["status"] == 0


@pytest.mark.parametrize("V,H", [(2000, 256), (33000, 512), (70003, 256), (139281, 256)])
@pytest.mark.parametrize("M", [161, 256, 257, 466])
def test_large_tile_lm_head_passes(sv, oracle, M, V, H):
    """More than 160 rows: a range of one short pass, of full passes before it (whole tiles stored without tests, their stores pending
    over the next steps), passes of as few slabs as the ring has, rows of logits that start at odd multiples of 4 bytes, whole and ragged row
    tiles.  Same order of additions as the weight-streaming kernel over row groups: same bits."""
    g = torch.Generator(device="cuda").manual_seed(V + M)
    hidden = torch.randn((M, H), generator=g, device="cuda").to(torch.bfloat16)
    W = torch.randn((V, H), generator=g, device="cuda").to(torch.bfloat16)
    Wp = torch.empty(sv.spec_lm_head_packed_bytes(V, H) // 2, dtype=torch.bfloat16, device="cuda")
    sv.spec_lm_head_pack(W, Wp)
    logits = torch.full((M + 1, V), 7.0, device="cuda")
    sv.spec_lm_head_packed(hidden, Wp, logits[:M])
    rows = torch.tensor(sorted({0, 15, 16, M // 2, M - 17, M - 1}), device="cuda")
    ref = oracle.lm_head(wl.bf16_bits(hidden[rows]), wl.bf16_bits(W))
    err = np.abs(logits[rows].cpu().numpy() - ref).max()
    assert err <= 1e-5 * math.sqrt(H) * np.abs(ref).max(), err
    assert (logits[M] == 7.0).all()                        # nothing past the last row
    sv.spec_set_tuning("lm_packed_tile", 1)
    try:
        other = torch.empty((M, V), device="cuda")
        sv.spec_lm_head_packed(hidden, Wp, other)
        torch.cuda.synchronize()
    finally:
        sv.spec_set_tuning("lm_packed_tile", 0)
    assert torch.equal(other, logits[:M])
