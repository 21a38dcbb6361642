"""tbe_flush writes the accumulators of small tables by a kernel and those of large ones by copies: tables of one row, on
either side of the line and many at once, each array whole on the host afterwards, also with several flushes in a run."""
import numpy as np
import pytest
import torch

from paper_2305_01515_amd import synth
from parity_util import run_parity

pytestmark = pytest.mark.gpu
T = synth.TableCfg


def test_tables_around_the_line():
    tabs = [T(1, 8, synth.FP32, None, "fixed", 1), T(255, 4, synth.FP32, 1.0, "fixed", 2, cache_slots=32), T(262143, 4, synth.FP32, 0.9, "fixed", 3, cache_slots=320),
            T(262144, 4, synth.FP32, None, "fixed", 3, cache_slots=320), T(262145, 4, synth.FP32, None, "fixed", 3, cache_slots=320)]
    run_parity(synth.WorkloadCfg("line", tabs, batch=40, ways=16, steps=4, seed=2, init_std=0.05, lr=0.05), steps=4, order="inline",
               flush_every=2)


def test_many_tables_and_rows_no_batch_touched():
    from paper_2305_01515_amd.tbe import TBE, pinned_empty
    g = torch.Generator().manual_seed(3)
    rows = [3 + 7 * t for t in range(1100)]
    W = [pinned_empty((r, 4), torch.float32).zero_() for r in rows]
    M = [pinned_empty((r,), torch.float32).copy_(torch.rand(r, generator=g)) for r in rows]
    want = [m.clone() for m in M]
    t = TBE(W, M, [0] * len(rows), 4, 2, 64)
    for m in M:
        m.zero_()
    t.flush()
    assert all(np.array_equal(m.numpy(), w.numpy()) for m, w in zip(M, want))
    t.close()


def test_state_in_memory_that_kernels_cannot_write():
    """accumulators in ordinary, not pinned memory through the C boundary: read at creation and written by every flush, beside
    tables whose arrays lie inside one pinned block"""
    import ctypes as C
    from oracle import Oracle
    from paper_2305_01515_amd.tbe import TableSpec, lib
    from parity_util import compare_backing, make_backing
    tabs = [T(300, 8, synth.FP32, 1.0, "fixed", 3, cache_slots=64), T(5000, 4, synth.FP32, 1.0, "fixed", 2, cache_slots=0),
            T(77, 16, synth.FP32, None, "fixed", 2, cache_slots=32), T(1, 4, synth.FP32, None, "fixed", 1)]
    cfg = synth.WorkloadCfg("pageable", tabs, batch=30, ways=8, steps=4, seed=8, init_std=0.05, lr=0.05)
    Wn, _, Wp, _ = make_backing(cfg)
    block = torch.empty(300 + 77 + 5, dtype=torch.float32, pin_memory=True)
    Mp = [block[1:301], torch.empty(5000), block[301:378], torch.empty(1)]
    assert [m.is_pinned() for m in Mp] == [True, False, True, False]
    for m in Mp:
        m.copy_(torch.rand(m.numel(), generator=torch.Generator().manual_seed(m.numel())))
    Mn = [m.numpy().copy() for m in Mp]
    edges = (float(block[0].fill_(-1.0)), block[378:].fill_(-2.0).tolist())
    slots = [t.cache_slots for t in tabs]
    o = Oracle(Wn, Mn, slots, cfg.ways)
    specs = (TableSpec * 4)(*[TableSpec(t.rows, t.dim, 0, w.data_ptr(), m.data_ptr(), t.cache_slots) for t, w, m in zip(tabs, Wp, Mp)])
    h = C.c_void_p()
    assert lib().tbe_create(C.byref(h), specs, 4, cfg.ways, cfg.batch, 1024, None, None) == 0
    for m in Mp:
        m.zero_()  # what the flush does not write stays zero
    stream = synth.BatchStream(cfg)
    for s in range(4):
        idx, off = stream.next()
        di, df, out, go = idx.cuda(), off.cuda(), torch.empty(cfg.batch, cfg.sum_dim, device="cuda"), synth.grad_out(cfg, s + 1)
        dg = go.cuda()
        assert lib().tbe_forward(h, di.data_ptr(), df.data_ptr(), cfg.batch, di.numel(), out.data_ptr()) == 0
        assert lib().tbe_backward_update(h, dg.data_ptr(), cfg.lr, cfg.eps) == 0
        o.prefetch(idx.numpy(), off.numpy())
        o.forward()
        o.backward_update(go.numpy(), cfg.lr, cfg.eps)
        if s % 2:
            assert lib().tbe_flush(h) == 0
            o.flush()
            compare_backing(cfg, Wn, Mn, Wp, Mp, f"flush after step {s + 1}")
        torch.cuda.synchronize()
    assert (float(block[0]), block[378:].tolist()) == edges
    assert lib().tbe_destroy(h) == 0
    o.close()


@pytest.mark.parametrize("second_level", [0, 2])
def test_a_flush_writes_every_cached_row_whatever_became_of_its_copy(second_level):
    """the caller writes over the host copies of cached rows and over all accumulators between two flushes, with no batch and with a
    batch of other rows in between: every flush leaves the whole model in the host arrays"""
    from oracle import Oracle
    from paper_2305_01515_amd.tbe import TBE
    from parity_util import compare_backing, make_backing
    slots = 160 if second_level else 480  # with a second level most rows have moved down into it
    tabs = [T(400, 16, synth.FP32, None, "fixed", 4, cache_slots=slots)]
    cfg = synth.WorkloadCfg("scribble", tabs, batch=64, ways=8, steps=4, seed=2, init_std=0.05, lr=0.05)
    Wn, Mn, Wp, Mp = make_backing(cfg)
    o = Oracle(Wn, Mn, [slots], 8, second_level_slots=[slots * second_level] if second_level else None)
    g = TBE(Wp, Mp, [slots], 8, 64, 256, second_level_factor=second_level)
    off = torch.arange(0, 257, 4, dtype=torch.int64)
    for step, rows in enumerate(([0, 150], [150, 400], None, [40, 90], None)):
        if rows:
            idx = torch.arange(256, dtype=torch.int64) % (rows[1] - rows[0]) + rows[0]
            go = synth.grad_out(cfg, step + 1)
            di, df, dg = idx.cuda(), off.cuda(), go.cuda()
            g.forward(di, df)
            g.backward_update(dg, cfg.lr, cfg.eps)
            o.prefetch(idx.numpy(), off.numpy())
            o.forward()
            o.backward_update(go.numpy(), cfg.lr, cfg.eps)
        o.flush()
        g.flush()
        compare_backing(cfg, Wn, Mn, Wp, Mp, f"flush {step}")
        tags = [g.cache_state(0)[0]] + ([g.second_level_state(0)[0]] if second_level else [])
        cached = torch.from_numpy(np.concatenate([x.ravel() for x in tags]))
        cached = cached[cached >= 0]
        assert cached.numel() > 100
        Wp[0][cached] = 7.0
        Mp[0].fill_(7.0)
    if second_level:
        assert g.second_level_stats()[1]["demotions"] > 100
    g.close()
    o.close()
