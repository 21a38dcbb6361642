"""Bags times lanes per row beyond the threads that one launch holds: the backward of the rows with one lookup, bag by bag,
with 16384 tables of 64 lanes and batch 4096 (2^32 lanes)."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_more_bag_lanes_than_2_to_32():
    from paper_2305_01515_amd.tbe import TBE, pinned_empty
    n_tab, dim, batch, lr, eps = 16384, 256, 4096, 0.1, 1e-8  # pooled vectors: 64 GiB, also handed in as the gradient
    gen = torch.Generator().manual_seed(1)
    w = pinned_empty((n_tab, dim), torch.float32).copy_(torch.randn(n_tab, dim, generator=gen))
    m = pinned_empty((n_tab,), torch.float32).zero_()
    want, acc = w.clone(), m.clone()
    g = TBE([w[t:t + 1] for t in range(n_tab)], [m[t:t + 1] for t in range(n_tab)], [0] * n_tab, 4, batch, 16, overlap=False)
    at = [(0, 5), (4095, 4095), (4096, 0), (9001, 77), (n_tab - 1, batch - 1)]  # (table, sample) of the lookups, one each
    off = torch.zeros(n_tab * batch + 1, dtype=torch.int64, device="cuda")
    for t, b in at:
        off[t * batch + b + 1:] += 1
    idx = torch.zeros(len(at), dtype=torch.int64, device="cuda")
    out = g.forward(idx, off)
    for t, b in at:
        assert torch.equal(out[b, t * dim:(t + 1) * dim].cpu(), want[t])
    g.backward_update(out, lr, eps)
    g.flush()
    for t, _ in at:
        acc[t] = want[t].double().square().mean()
        want[t] -= lr * want[t] / (acc[t].sqrt() + eps)
    assert torch.allclose(w, want, rtol=0, atol=1e-6) and torch.allclose(m, acc, rtol=1e-6, atol=0)
    g.close()
    del out, off
    torch.cuda.empty_cache()
