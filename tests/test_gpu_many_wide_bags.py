"""More bags than the threads of one launch serve: the backward of the rows with one lookup, bag by bag, with 16384 tables of 64
lanes and batch 4096 (2^32 lanes); the key generation with 2^29 bags (8 lanes each); one table whose bags alone are too many."""
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


def test_two_to_the_29_bags():
    from paper_2305_01515_amd.tbe import TBE, TbeError, pinned_empty
    n_tab, dim, batch, lr, eps = 8, 4, 1 << 26, 0.1, 1e-8
    w = [pinned_empty((3, dim), torch.float32).copy_(torch.randn(3, dim, generator=torch.Generator().manual_seed(t))) for t in range(n_tab)]
    m = [pinned_empty((3,), torch.float32).zero_() for _ in range(n_tab)]
    want = [x.clone() for x in w]
    g = TBE(w, m, [0] * n_tab, 4, batch, 16, overlap=False)
    at = [(0, 5, 2), (1, batch - 1, 0), (2, 0, 1), (5, 77, 1), (7, 0, 0), (7, batch - 1, 2)]  # (table, sample, row), one lookup each
    off = torch.zeros(n_tab * batch + 1, dtype=torch.int64, device="cuda")
    for t, b, _ in at:
        off[t * batch + b + 1:] += 1
    idx = torch.tensor([r for _, _, r in at], device="cuda")
    out = g.forward(idx, off)
    for t, b, r in at:
        assert torch.equal(out[b, t * dim:(t + 1) * dim].cpu(), want[t][r])
    assert int(torch.count_nonzero(out)) == len(at) * dim
    g.backward_update(out, lr, eps)
    g.flush()
    for t, b, r in at:
        want[t][r] -= lr * want[t][r] / (want[t][r].square().mean().sqrt() + eps)
    assert all(torch.allclose(a, b, rtol=0, atol=1e-6) for a, b in zip(w, want))
    idx[-1] = 3  # no such row: seen in the last bag too
    g.forward(idx, off, out)
    with pytest.raises(TbeError) as e:
        g.stats()
    assert e.value.code == -2
    g.close()
    del out, off
    torch.cuda.empty_cache()


def test_one_table_with_too_many_bags_is_refused():
    from paper_2305_01515_amd.tbe import TBE, lib, pinned_empty
    g = TBE([pinned_empty((3, 256), torch.float32).zero_()], [pinned_empty((3,), torch.float32).zero_()], [0], 4, 1 << 26, 16)
    some = torch.zeros(64, dtype=torch.int64, device="cuda")
    assert lib().tbe_prefetch(g._h, some.data_ptr(), some.data_ptr(), 1 << 26, 0) == -5
    g.close()
