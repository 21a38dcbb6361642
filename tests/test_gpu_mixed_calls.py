"""Batches of unlike size, some prefetched ahead, some prefetched by the forward itself, in one program: a batch's kernels go to
the compute, the prefetch or the link stream by its size and by who prefetches it, and every change from one stream to another
must keep the order of what was given before.  Half of the rows bypass the caches, so that copies of bypassed rows are on their
way at most of these changes."""
import numpy as np
import pytest
import torch

from oracle import Oracle
from paper_2305_01515_amd import synth
from parity_util import compare_backing, make_backing

pytestmark = pytest.mark.gpu
T = synth.TableCfg


def drawn(rng, tabs, sizes):
    """one batch per entry of sizes (bags a table, mean lookups a bag): indices, offsets, output gradient"""
    host = []
    for batch, mean in sizes:
        lens = rng.poisson(mean, (len(tabs), batch))
        off = np.concatenate([[0], np.cumsum(lens.ravel())]).astype(np.int64)
        idx = np.concatenate([rng.randint(0, t.rows, int(n.sum())) for t, n in zip(tabs, lens)]).astype(np.int64)
        host.append((idx, off, rng.randn(batch, sum(t.dim for t in tabs)).astype(np.float32)))
    return host


def run(cfg, host, rng, ready, depth=1, level2=0, own=(), ahead_of=(), flush_behind=()):
    """Trains on the batches in order, each prefetched at a moment that rng chooses -- but those in `own` by the forward, those in
    `ahead_of` before the update of the batch in front -- and compares with the oracle, which takes them one by one: values,
    counters and cache state.  flush_behind: steps behind which nothing is prefetched before a flush."""
    from paper_2305_01515_amd.tbe import TBE
    Wn, Mn, Wp, Mp = make_backing(cfg)
    slots = [t.cache_slots for t in cfg.tables]
    g = TBE(Wp, Mp, slots, cfg.ways, cfg.batch, max(1, max(b[0].size for b in host)), second_level_factor=level2)
    if depth > 1:
        g.set_prefetch_depth(depth)
    dev = [tuple(torch.from_numpy(x).cuda() for x in b) for b in host]
    torch.cuda.synchronize()
    g.set_inputs_ready(ready)
    ahead, outs = 0, []
    for s in range(len(dev)):
        def prefetch(most, certain=False):
            nonlocal ahead
            while ahead < min(len(dev), s + most) and ahead not in own and not (ahead - 1 in flush_behind and ahead > s):
                if rng.rand() >= 0.6 and not (certain and ahead in ahead_of):
                    break
                g.prefetch(*dev[ahead][:2])
                ahead += 1
        ahead = max(ahead, s)
        prefetch(depth + 1)      # before the forward: the batch itself and those that the pipeline takes ahead of it
        outs.append(g.forward(*dev[s][:2]))
        ahead = max(ahead, s + 1)
        prefetch(depth + 1, certain=True)  # between forward and update
        g.backward_update(dev[s][2], cfg.lr, cfg.eps)
        if s in flush_behind:
            g.flush()
    g.flush()
    outs = [o.cpu().numpy() for o in outs]
    o = Oracle(Wn, Mn, slots, cfg.ways, prefetch_lock=depth if depth > 1 else 0,
               second_level_slots=[level2 * (n // cfg.ways) * cfg.ways for n in slots] if level2 else None)
    for (idx, off, grad), out in zip(host, outs):
        o.prefetch(idx, off)
        ref = o.forward()
        assert np.abs(out - ref).max() <= 1e-5 * np.abs(ref).max()  # fp32 sums of a few terms
        o.backward_update(grad, cfg.lr, cfg.eps)
    st = g.stats()
    assert st["total"] == o.stats()[1]
    for t in range(len(slots)):
        for x, y in zip(o.cache_state(t), g.cache_state(t)):
            assert np.array_equal(x, y)
    o.flush()
    compare_backing(cfg, Wn, Mn, Wp, Mp, "at the end")
    st["rows_from_copies"] = g.prefetch_depth()[1]
    g.close()
    o.close()
    return st


@pytest.mark.parametrize("seed", range(6))
@pytest.mark.parametrize("ready", [False, True], ids=["inputs_ordered", "inputs_ready"])
@pytest.mark.parametrize("depth,level2", [(1, 0), (1, 1), (2, 0), (3, 0)])
def test_sizes_and_orders_in_turn(seed, ready, depth, level2):
    """a handful of lookups, around the lines of one kernel, beyond them, and, twice, above 65536: once prefetched by the forward
    itself, once ahead, both times between smaller ones"""
    rng = np.random.RandomState(1000 * depth + seed)
    tabs = [T(4001, 16, synth.FP32, None, "poisson", 1.0, cache_slots=4 * 100), T(900, 8, synth.FP32, None, "poisson", 1.0, cache_slots=0),
            T(50, 32, synth.FP32, None, "poisson", 1.0, cache_slots=52 * 4)]
    sizes = [(int(rng.choice([1, 3, 40, 500, 1300, 1400, 2500], p=[.1, .1, .25, .2, .15, .1, .1])), 1.0) for _ in range(24)]
    sizes[5], sizes[12] = (9000, 2.9), (9000, 2.9)
    host = drawn(rng, tabs, sizes)
    lookups = [b[0].size for b in host]
    assert lookups[5] > 65536 and lookups[12] > 65536 and min(lookups) < 1024 and any(4096 < n < 65536 for n in lookups)
    cfg = synth.WorkloadCfg("mixed", tabs, batch=9000, ways=4, steps=24, seed=seed, init_std=0.05, lr=0.05)
    st = run(cfg, host, rng, ready, depth, level2, own=(5,), ahead_of=(12,))
    assert st["total"]["bypasses"] > 0 and st["total"]["evictions"] > 0
    assert st["late_fetches"] > 0


@pytest.mark.parametrize("ready", [False, True], ids=["inputs_ordered", "inputs_ready"])
@pytest.mark.parametrize("depth", [1, 2])
@pytest.mark.parametrize("seed", range(2))
def test_wide_rows_in_turn(seed, depth, ready):
    """rows of 1 KB, most of them bypassed: batches of 40 to 35000 lookups, around 1024 rows, 4 MB and 32 MB of them, prefetched by the
    forward and ahead"""
    rng = np.random.RandomState(77 + seed)
    tabs = [T(9000, 256, synth.FP32, None, "poisson", 1.0, cache_slots=4 * 50), T(9000, 256, synth.FP32, None, "poisson", 1.0, cache_slots=0)]
    sizes = [(b, 1.0) for b in (20, 490, 530, 1900, 17500, 20, 2200, 15000, 500, 17500, 17500, 2200, 540, 480)]
    host = drawn(rng, tabs, sizes)
    cfg = synth.WorkloadCfg("wide", tabs, batch=17500, ways=4, steps=len(sizes), seed=seed, init_std=0.05, lr=0.05)
    st = run(cfg, host, rng, ready, depth, own=(3, 4, 5, 7, 8, 9, 11), ahead_of=(2, 6, 10))
    assert st["total"]["bypasses"] > 0 and st["total"]["evictions"] > 0


@pytest.mark.parametrize("ready", [False, True], ids=["inputs_ordered", "inputs_ready"])
@pytest.mark.parametrize("depth", [1, 2, 3])
@pytest.mark.parametrize("seed", range(2))
def test_models_that_never_bypass(seed, depth, ready):
    """every table has a way for each of its rows: no update is followed by a write-back, and what follows it on the other streams
    goes by the marks that other batches left; flushes in mid-stream, with batches before and behind them"""
    rng = np.random.RandomState(500 + 10 * depth + seed)
    tabs = [T(4001, 16, synth.FP32, None, "poisson", 1.0, cache_slots=4001 + 4), T(900, 256, synth.FP32, None, "poisson", 1.0, cache_slots=900 + 4),
            T(50, 32, synth.FP32, None, "poisson", 1.0, cache_slots=50 + 4)]
    sizes = [(int(rng.choice([1, 3, 40, 300, 500, 1400, 3000])), 1.0) for _ in range(24)]
    sizes[6], sizes[13] = (9000, 2.9), (9000, 2.9)
    host = drawn(rng, tabs, sizes)
    cfg = synth.WorkloadCfg("resident", tabs, batch=9000, ways=4, steps=24, seed=seed, init_std=0.05, lr=0.05)
    st = run(cfg, host, rng, ready, depth, own=(3, 6, 16, 17), ahead_of=(7, 10, 11, 13, 14), flush_behind=(8, 15))
    assert st["total"]["bypasses"] == 0 and st["total"]["evictions"] == 0 and st["total"]["hits"] > 0
