"""A batch that the device refuses (an index out of range), with more batches behind it that the caller issues before a
synchronising call tells of the refusal: none of them does anything, the error is there however many follow, and the
flush leaves the backing tier as the last batch in front of the refused one left it.

The prefetch stage of a batch has several forms, and each raises a refusal and hears of one in kernels of its own.  LOOKUPS names a
batch size (samples) for each: about four lookups a sample."""
import numpy as np
import pytest
import torch

from oracle import Oracle
from paper_2305_01515_amd import synth
from parity_util import compare_backing, first_bags, make_backing

pytestmark = pytest.mark.gpu
T = synth.TableCfg


LOOKUPS = {"one_workgroup": 12,     # one kernel of one workgroup
           "few_workgroups": 150,   # ... of 3
           "many_workgroups": 500,  # ... of 10, several of them with lists
           "kernel_a_pass": 1500,   # 4097 to 524288 lookups
           "large": 21846}          # > 65536 bags: no small batch, its stage behind training


def model(seed, dtype, batch=19):
    f = max(1, batch // 19)
    tabs = [T(60 * f, 16, dtype, 0.7, "poisson", 2, 0, 20, cache_slots=16 * f), T(45 * f, 8, dtype, None, "poisson", 1, 0, 20, cache_slots=8 * f),
            T(30 * f, 8, dtype, None, "fixed", 1, cache_slots=0)]
    return synth.WorkloadCfg("refused", tabs, batch=batch, ways=4, steps=12, seed=seed, init_std=0.05, lr=0.05)


def start(cfg, n, samples=None, **kw):
    """library, oracle and the first n batches; the last of them with an index that no table has.  samples[i]: batch i has only
    the first so many bags of each table"""
    from paper_2305_01515_amd.tbe import TBE
    Wn, Mn, Wp, Mp = make_backing(cfg)
    slots = [t.cache_slots for t in cfg.tables]
    o = Oracle(Wn, Mn, slots, cfg.ways)
    stream = synth.BatchStream(cfg)
    host = [stream.next() for _ in range(n)]
    if samples:
        host = [first_bags(i, f, cfg.num_tables, x) for (i, f), x in zip(host, samples)]
    bad = host[-1][0].clone()
    bad[bad.numel() // 2] = cfg.tables[0].rows  # the largest table's
    dev = [(i.cuda(), f.cuda()) for i, f in host[:-1]] + [(bad.cuda(), host[-1][1].cuda())]
    g = TBE(Wp, Mp, slots, cfg.ways, cfg.batch, max(i.numel() for i, _ in host) + 1, **kw)
    return g, o, host, dev, (Wn, Mn, Wp, Mp)


def train(g, o, cfg, s, host, dev, ahead=()):
    for b in ahead:
        g.prefetch(*b)
    g.forward(*dev[s])
    go = synth.grad_out(cfg, s + 1)[:(len(host[s][1]) - 1) // cfg.num_tables]
    g.backward_update(go.cuda(), cfg.lr, cfg.eps)
    o.prefetch(host[s][0].numpy(), host[s][1].numpy())
    o.forward()
    o.backward_update(go.numpy(), cfg.lr, cfg.eps)


def expect_refusal(call, code=-2):
    from paper_2305_01515_amd.tbe import TbeError
    with pytest.raises(TbeError) as e:
        call()
    assert e.value.code == code


def refuse_and_go_on(cfg, behind, ahead, level2, samples=None, good=5, bad_offsets=False):
    """`good` batches that train, a refused one, and `behind` of the good ones again; samples[i]: of batch i (the last: the refused)"""
    g, o, host, dev, (Wn, Mn, Wp, Mp) = start(cfg, good + 1, samples, second_level_factor=level2)
    if bad_offsets:
        off = host[-1][1].clone()
        off[len(off) // 2] = off[-1] + 1
        dev[-1] = (host[-1][0].cuda(), off.cuda())
    if ahead:
        g.prefetch(*dev[0])
    for s in range(good):
        train(g, o, cfg, s, host, dev, dev[s + 1:s + 2] if ahead else ())
    assert o.stats()[0]["bypasses"] > 0
    late = [dev[good]] + [dev[s % good] for s in range(behind)]  # the bad batch, then rows that were bypassed just before
    ones = torch.ones(cfg.batch, cfg.sum_dim, device="cuda")
    for n, b in enumerate(late):
        if ahead and n + 1 < len(late):
            g.prefetch(*late[n + 1])
        g.forward(*b)
        g.backward_update(ones[:(len(b[1]) - 1) // cfg.num_tables], cfg.lr, cfg.eps)
    code = -1 if bad_offsets else -2
    expect_refusal(g.flush, code)
    expect_refusal(g.flush, code)
    expect_refusal(lambda: g.prefetch(*dev[0]), code)
    o.flush()
    compare_backing(cfg, Wn, Mn, Wp, Mp, "after the refused batch")
    g.close()
    o.close()


@pytest.mark.parametrize("behind", [1, 2, 3, 4, 7])
@pytest.mark.parametrize("ahead", [True, False], ids=["ahead", "one_by_one"])
@pytest.mark.parametrize("dtype,level2", [(synth.FP32, 0), (synth.FP16, 0), (synth.FP32, 2)])
def test_nothing_behind_a_refused_batch_trains(behind, ahead, dtype, level2):
    """behind: good batches after the bad one, each forwarded and updated by a caller that does not know yet"""
    refuse_and_go_on(model(3 + behind, dtype), behind, ahead, level2)


@pytest.mark.parametrize("size", ["one_workgroup", "many_workgroups", "kernel_a_pass", "large"])
@pytest.mark.parametrize("behind,ahead,level2,bad_offsets", [(1, True, 0, False), (4, True, 0, True), (4, False, 0, False), (2, False, 0, True),
                                                             (4, True, 2, False), (3, False, 2, False)])
def test_every_form_of_the_stage_refuses(size, behind, ahead, level2, bad_offsets):
    refuse_and_go_on(model(11 + behind, synth.FP32, LOOKUPS[size]), behind, ahead, level2, good=3, bad_offsets=bad_offsets)


@pytest.mark.parametrize("refused,later", [("one_workgroup", "kernel_a_pass"), ("few_workgroups", "many_workgroups"), ("many_workgroups", "kernel_a_pass"),
                                           ("many_workgroups", "one_workgroup"), ("kernel_a_pass", "few_workgroups"), ("kernel_a_pass", "many_workgroups"),
                                           ("large", "few_workgroups"), ("many_workgroups", "large")])
@pytest.mark.parametrize("ahead", [True, False], ids=["ahead", "one_by_one"])
def test_one_form_hears_of_the_refusal_of_another(refused, later, ahead):
    """the good batches, in front of the refused one and behind it, go through another form of the stage"""
    a, b = LOOKUPS[refused], LOOKUPS[later]
    refuse_and_go_on(model(31, synth.FP32, max(a, b)), 3, ahead, 0, samples=[b, max(a, b), b, b, a], good=4)


def test_the_first_refusal_is_the_one_reported():
    """bad offsets behind an index out of range, then good batches: TBE_ERANGE, as if it had been asked for at once"""
    cfg = model(1, synth.FP32)
    g, o, host, dev, _ = start(cfg, 3)
    train(g, o, cfg, 0, host, dev)
    zero = torch.zeros(cfg.batch, cfg.sum_dim, device="cuda")
    off = dev[1][1].clone()
    off[0] = 1
    for b in (dev[2], (dev[1][0], off), dev[0], dev[1], dev[0], dev[1]):
        g.forward(*b)
        g.backward_update(zero, cfg.lr, cfg.eps)
    expect_refusal(g.stats, -2)
    g.close()
    o.close()


@pytest.mark.parametrize("seed", range(6))
@pytest.mark.parametrize("forwarded", [True, False])
@pytest.mark.parametrize("depth,level2", [(1, 0), (1, 1), (1, 2), (2, 0), (3, 0)])
def test_refused_batch_behind_batches_fetched_ahead(depth, level2, forwarded, seed):
    """The last batch in front of the refused one has not trained and holds rows whose value is in its copies alone.  In the
    pipeline several batches deep several such batches are in their cache lines already, some of their rows as copies that
    wait for the forward."""
    refuse_behind_fetched(model(20 + seed, synth.FP32), depth, level2, forwarded)


@pytest.mark.parametrize("size", ["many_workgroups", "kernel_a_pass"])
@pytest.mark.parametrize("forwarded", [True, False])
@pytest.mark.parametrize("depth,level2", [(1, 0), (1, 2), (2, 0), (3, 0)])
def test_every_form_refuses_behind_batches_fetched_ahead(depth, level2, forwarded, size):
    refuse_behind_fetched(model(27, synth.FP32, LOOKUPS[size]), depth, level2, forwarded, steps=4)


def refuse_behind_fetched(cfg, depth, level2, forwarded, steps=6):
    g, o, host, dev, (Wn, Mn, Wp, Mp) = start(cfg, steps + depth, second_level_factor=level2)
    g.set_prefetch_depth(depth)
    for b in dev[:depth]:
        g.prefetch(*b)
    for s in range(steps - 1):
        train(g, o, cfg, s, host, dev, dev[s + depth:s + depth + 1])
    g.prefetch(*dev[-1])
    if forwarded:
        g.forward(*dev[steps - 1])
    assert o.stats()[1]["bypasses"] > 0 and o.stats()[1]["evictions"] > 0
    expect_refusal(g.flush)
    o.flush()
    compare_backing(cfg, Wn, Mn, Wp, Mp, "after the refused batch")
    g.close()
    o.close()
