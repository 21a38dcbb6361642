"""Rows whose backing-tier copy is stale are found through map entries that are never taken out: an entry counts only
while the list it points into is still alive and holds the row there.  Long runs of small models, in which the same
rows are evicted, bypassed and wanted again over and over, so that entries many batches old point at positions that
later batches' lists fill with other rows."""
import pytest
import torch

from paper_2305_01515_amd import synth
from parity_util import run_parity

pytestmark = pytest.mark.gpu


def churn(seed, slots=(16, 8, 0), wide=False):
    """wide: sixteen times the rows and lookups, of 1 KB: their transfers and commits have the link's stream to themselves, those of
    the others follow the stage on its own"""
    T = synth.TableCfg
    f, d = (16, 16) if wide else (1, 1)
    tabs = [T(60 * f, 16 * d, synth.FP32, 0.7, "poisson", 2, 0, 20, cache_slots=slots[0] * f),
            T(45 * f, 8 * d, synth.FP32, None, "poisson", 1, 0, 20, cache_slots=slots[1] * f),
            T(30 * f, 4 * d, synth.FP32, None, "fixed", 1, cache_slots=slots[2] * f)]
    return synth.WorkloadCfg("churn", tabs, batch=19 * f, ways=4, steps=30, seed=seed, init_std=0.05, lr=0.05)


@pytest.mark.parametrize("kw", [dict(order="early"), dict(order="ahead", vary_batch=3), dict(order="serial", flush_every=4),
                                dict(order="early", second_level_factor=1), dict(order="early", second_level_factor=2, policy="lfu"),
                                dict(order="pipe2"), dict(order="pipe5"), dict(order="deep3", vary_batch=5)],
                         ids=["early", "ahead", "flush", "two_level", "two_level_lfu", "pipe2", "pipe5", "queue"])
@pytest.mark.parametrize("seed", [1, 2])
def test_thirty_batches_over_the_same_rows(seed, kw):
    st = run_parity(churn(seed), steps=30, **kw)
    assert st["total"]["bypasses"] > 0 and st["total"]["inserts"] > 0
    assert st["late_fetches"] > 0


@pytest.mark.parametrize("kw", [dict(order="early"), dict(order="ahead", vary_batch=3), dict(order="serial", flush_every=4),
                                dict(order="early", second_level_factor=1), dict(order="pipe2"), dict(order="pipe3", vary_batch=2),
                                dict(order="deep3", vary_batch=5)],
                         ids=["early", "ahead", "flush", "two_level", "pipe2", "pipe3", "queue"])
def test_thirty_batches_of_wide_rows(kw):
    """vary_batch: batches on both sides of the line in turn"""
    st = run_parity(churn(1, wide=True), steps=30, **kw)
    assert st["total"]["bypasses"] > 0 and st["total"]["inserts"] > 0
    assert st["late_fetches"] > 0


@pytest.mark.parametrize("wide", [False, True], ids=["narrow", "wide"])
@pytest.mark.parametrize("ready", [True, False], ids=["inputs_ready", "inputs_ordered"])
@pytest.mark.parametrize("burst", [2, 3, 4])
def test_bursts_that_begin_with_two_batches_prefetched(burst, ready, wide):
    """A loop that trains `burst` batches, the last of them with nothing behind it, and then prefetches two before the next
    forward: the second takes the buffer of the batch whose overflow copies the burst's last commit parked, while they go
    home.  Values, and the backing tier at the end, as trained one by one."""
    from oracle import Oracle
    from paper_2305_01515_amd.tbe import TBE
    from parity_util import compare_backing, compare_forward, make_backing
    cfg = churn(7 + burst, slots=(8, 4, 0), wide=wide)
    Wn, Mn, Wp, Mp = make_backing(cfg)
    slots = [t.cache_slots for t in cfg.tables]
    o = Oracle(Wn, Mn, slots, cfg.ways)
    stream = synth.BatchStream(cfg)
    host = [stream.next() for _ in range(8 * burst)]
    dev = [(i.cuda(), f.cuda()) for i, f in host]
    grads = [synth.grad_out(cfg, s + 1) for s in range(len(host))]
    dgrads = [x.cuda() for x in grads]
    g = TBE(Wp, Mp, slots, cfg.ways, cfg.batch, max(i.numel() for i, _ in host))
    g.set_inputs_ready(ready)
    torch.cuda.synchronize()
    outs = []
    for s in range(len(host)):
        if s % burst == 0:
            g.prefetch(*dev[s])
        if s % burst + 1 < burst:
            g.prefetch(*dev[s + 1])
        outs.append(g.forward(*dev[s]))
        g.backward_update(dgrads[s], cfg.lr, cfg.eps)
    g.flush()
    for s, (i, f) in enumerate(host):
        o.prefetch(i.numpy(), f.numpy())
        compare_forward(cfg, o.forward(), outs[s].cpu().numpy(), f"step {s + 1}")
        o.backward_update(grads[s].numpy(), cfg.lr, cfg.eps)
    o.flush()
    compare_backing(cfg, Wn, Mn, Wp, Mp, "after flush")
    st = g.stats()
    assert st["total"] == o.stats()[1] and st["total"]["bypasses"] > 0 and st["late_fetches"] > 0
    g.close()
    o.close()
