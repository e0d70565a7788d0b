"""Divergence points at the edges of what one memory round trip compares (512 threads x 8 positions)."""
import numpy as np
import pytest
import torch

from test_gpu_parity import sv  # noqa: F401

pytestmark = pytest.mark.gpu


def test_divergence_at_the_edges_of_a_trip(sv, oracle):
    at = [0, 63, 64, 511, 512, 4095, 4096, 4097, 8191, 8192, 9000]
    lens = [max(1, t + 1) for t in at] + [4096, 4097, 9001, 0, 5]
    rng = np.random.default_rng(5)
    p = [rng.integers(0, 9, n).astype(np.int32) for n in lens]
    h = [np.concatenate([x, x[:1]]) for x in p]                  # the longer one agrees all the way ...
    for k, t in enumerate(at):
        h[k][t] += 1                                             # ... but for one position, and everything behind it
        h[k][t + 1:] += 1
    indptr = lambda rows: np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)  # noqa: E731
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    delta = torch.full((len(p),), -7, dtype=torch.int32, device="cuda")
    sv.spec_divergence(dev(np.concatenate(p)), dev(indptr(p)), dev(np.concatenate(h)), dev(indptr(h)), delta)
    expected = at + lens[len(at):]
    assert delta.cpu().tolist() == expected
    assert oracle.divergence(np.concatenate(p), indptr(p), np.concatenate(h), indptr(h)).tolist() == expected


@pytest.mark.parametrize("per_cu", [1, 4])
def test_divergence_of_many_sequences(sv, oracle, per_cu):
    """More pairs than 256 CUs, and more than four per CU: trips of 1024 positions by 512 threads and by 256, a difference at every edge."""
    edges = [0, 1, 63, 64, 255, 256, 511, 512, 513, 1023, 1024, 1025, 2047, 2048, 3000]
    rng = np.random.default_rng(6)
    B = per_cu * 256 + 5
    at = [edges[i % len(edges)] for i in range(B)]
    p = [rng.integers(0, 9, t + 1 + i % 3).astype(np.int32) for i, t in enumerate(at)]
    h = [x.copy() for x in p]
    for i, t in enumerate(at):
        if i % 5:                                                # (every fifth agrees to its end)
            h[i][t:] += 1
    indptr = lambda rows: np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)  # noqa: E731
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    delta = torch.full((B,), -7, dtype=torch.int32, device="cuda")
    sv.spec_divergence(dev(np.concatenate(p)), dev(indptr(p)), dev(np.concatenate(h)), dev(indptr(h)), delta)
    assert delta.cpu().tolist() == oracle.divergence(np.concatenate(p), indptr(p), np.concatenate(h), indptr(h)).tolist()
    assert delta.cpu().tolist() == [len(x) if i % 5 == 0 else t for i, (x, t) in enumerate(zip(p, at))]
