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


@pytest.mark.parametrize("seed", range(6))
@pytest.mark.parametrize("ready", [False, True], ids=["inputs_ordered", "inputs_ready"])
@pytest.mark.parametrize("depth,level2", [(1, 0), (1, 1), (2, 0), (3, 0)])
def test_sizes_and_orders_in_turn(seed, ready, depth, level2):
    from paper_2305_01515_amd.tbe import TBE
    rng = np.random.RandomState(1000 * depth + seed)
    tabs = [T(4001, 16, synth.FP32, None, "poisson", 1.0, cache_slots=4 * 100), T(900, 8, synth.FP32, None, "poisson", 1.0, cache_slots=0),
            T(50, 32, synth.FP32, None, "poisson", 1.0, cache_slots=52 * 4)]
    cfg = synth.WorkloadCfg("mixed", tabs, batch=9000, ways=4, steps=24, seed=seed, init_std=0.05, lr=0.05)
    Wn, Mn, Wp, Mp = make_backing(cfg)
    slots = [t.cache_slots for t in tabs]
    host = []
    for _ in range(24):  # a handful of lookups, around the line of one kernel, beyond it, and above 65536
        batch = int(rng.choice([1, 3, 40, 500, 1300, 1400, 2500, 9000], p=[.1, .1, .2, .2, .15, .1, .1, .05]))
        lens = rng.poisson(2.9 if batch == 9000 else 1.0, (3, batch))
        off = np.concatenate([[0], np.cumsum(lens.ravel())]).astype(np.int64)
        idx = np.concatenate([rng.randint(0, t.rows, int(n.sum())) for t, n in zip(tabs, lens)]).astype(np.int64)
        host.append((idx, off, rng.randn(batch, cfg.sum_dim).astype(np.float32)))
    g = TBE(Wp, Mp, slots, cfg.ways, cfg.batch, max(1, max(b[0].size for b in host)), second_level_factor=level2)
    if depth > 1:
        g.set_prefetch_depth(depth)
    dev = [tuple(torch.from_numpy(x).cuda() for x in b) for b in host]
    torch.cuda.synchronize()
    g.set_inputs_ready(ready)
    ahead, outs = 0, []
    for s in range(len(dev)):
        def prefetch(most):
            nonlocal ahead
            while ahead < min(len(dev), s + most) and rng.rand() < 0.6:
                g.prefetch(*dev[ahead][:2])
                ahead += 1
        ahead = max(ahead, s)
        prefetch(depth + 1)      # before the forward: the batch itself and those that the pipeline takes ahead of it
        outs.append(g.forward(*dev[s][:2]))
        ahead = max(ahead, s + 1)
        prefetch(depth + 1)      # between forward and update
        g.backward_update(dev[s][2], cfg.lr, cfg.eps)
    g.flush()
    outs = [o.cpu().numpy() for o in outs]
    o = Oracle(Wn, Mn, slots, cfg.ways)
    for (idx, off, grad), out in zip(host, outs):
        o.prefetch(idx, off)
        ref = o.forward()
        assert np.abs(out - ref).max() <= 1e-5 * np.abs(ref).max()  # fp32 sums of a few terms
        o.backward_update(grad, cfg.lr, cfg.eps)
    o.flush()
    compare_backing(cfg, Wn, Mn, Wp, Mp, "at the end")
    g.close()
    o.close()
