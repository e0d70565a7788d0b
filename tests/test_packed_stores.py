"""Logits rows that start at any multiple of 4 bytes, from the weight-streaming LM head: vector stores, the last 1 to 3 entries of a row one by one, nothing beside them."""
import pytest
import torch

from test_gpu_parity import sv  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [1, 16, 57, 112])
@pytest.mark.parametrize("V", [1, 2, 3, 5, 18, 1003, 32001, 50021])
@pytest.mark.parametrize("row_major", [False, True])
def test_rows_of_any_length(sv, M, V, row_major):
    H = 256
    g = torch.Generator(device="cuda").manual_seed(V + M)
    hidden = torch.randn((M, H), generator=g, device="cuda").to(torch.bfloat16)
    W = torch.randn((V, H), generator=g, device="cuda").to(torch.bfloat16)
    buf = torch.full((M * V + 64,), 7.0, device="cuda")
    logits = buf[:M * V].view(M, V)
    if row_major:
        sv.spec_lm_head(hidden, W, logits)
    else:
        Wp = torch.empty(sv.spec_lm_head_packed_bytes(V, H) // 2, dtype=torch.bfloat16, device="cuda")
        sv.spec_lm_head_pack(W, Wp)
        sv.spec_lm_head_packed(hidden, Wp, logits)
    ref = hidden.double() @ W.double().t()
    # products are exact in fp32, H additions round by 2^-24 of partial sums of at most sum |h w|
    bound = (hidden.double().abs() @ W.double().abs().t()) * H * 2.0 ** -24
    assert ((logits.double() - ref).abs() <= bound).all()
    assert (buf[M * V:] == 7.0).all()
