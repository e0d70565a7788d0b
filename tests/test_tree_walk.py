"""Greedy acceptance on the largest trees (64 rows, a lane each) and on one row: chains, stars with equal children, random trees, and requests with every kind of fault."""
import numpy as np
import pytest
import torch

from test_gpu_parity import sv  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", [5, 4097, 64 * 4096 + 3])
def test_walks_of_64_rows(sv, oracle, V):
    rng = np.random.default_rng(V)
    sizes = [64, 64, 64, 1, 63, 17, 64, 64, 64, 64, 65, 0, 2]  # (65 rows are more than gamma_max + 1, none are too few)
    qo = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    M, B, gmax = int(qo[-1]), len(sizes), 63
    logits = rng.normal(0, 1, (M, V)).astype(np.float32)
    am = logits.argmax(1)
    parent, tokens = np.full(M, -1, np.int32), rng.integers(0, V, M).astype(np.int32)
    for i, n in enumerate(sizes):
        for j in range(1, n):
            r = qo[i] + j
            parent[r] = j - 1 if i == 0 else (0 if i == 1 else rng.integers(max(0, j - 6), j))
            if i < 2 or rng.random() < 0.8:                     # a full chain; a star of equal children (the lowest row wins); deep walks
                tokens[r] = am[qo[i] + parent[r]]
    logits[qo[6] + 40, V // 2] = np.nan
    tokens[qo[7] + 63] = V
    parent[qo[8] + 20] = 20
    parent[qo[9]] = 0
    ref = oracle.accept_tree(logits, tokens, parent, qo, gmax)
    dev = lambda a: torch.from_numpy(a).cuda()                  # noqa: E731
    full = lambda shape, dtype: torch.full(shape, 9, dtype=dtype, device="cuda")    # noqa: E731
    al, ot, pth, rb = full((B,), torch.int32), full((B, gmax + 1), torch.int32), full((B, gmax + 1), torch.int32), full((B,), torch.uint8)
    st, status = full((4,), torch.int32), torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = torch.empty(max(256, sv.spec_accept_workspace_bytes(B, M, V, gmax)), dtype=torch.uint8, device="cuda")
    sv.spec_accept_tree(dev(logits), dev(tokens), dev(parent), dev(qo), al, ot, pth, rb, st, gmax, status, ws)
    ref["rollback"][10] = 0                                     # a request of a length that is refused: nothing is rolled back (the oracle: n > 1)
    for got, name in ((al, "accept_len"), (ot, "out_tokens"), (pth, "path"), (rb, "rollback")):
        assert np.array_equal(got.cpu().numpy(), ref[name]), name
    assert ref["accept_len"][0] == 63 and int(status.cpu()) == sv.FLAG_BAD_LOGITS | sv.FLAG_BAD_TOKEN | sv.FLAG_BAD_TREE | sv.FLAG_BAD_LENGTH
    for i in (10, 11):
        assert int(al[i]) == 0 and (ot[i] == -1).all() and pth[i].tolist() == [0] + [-1] * gmax
    flagged = [6, 7, 8, 9, 10, 11]
    sound = [i for i in range(B) if i not in flagged]
    assert st.tolist() == [int(ref["rollback"].sum()), int((ref["accept_len"][sound] + 1).sum()), B, 0]
