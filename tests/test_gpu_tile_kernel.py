"""Heavy rows of the largest batches, more than 2097152 lookups: the table's gradients in tiles in LDS and the kernel that adds up the
partial sums, at every width, with sum and mean pooling, over several steps (a row's parts count themselves in, and the count has
to be back at zero for the next).  Rows narrower than four lanes have a workgroup each there."""
import numpy as np
import pytest

from paper_2305_01515_amd import synth
from parity_util import run_parity

pytestmark = pytest.mark.gpu
T = synth.TableCfg
BATCH = 63600  # 33 lookups a bag of all tables: 2098800


def heavy(dim, dtype, pool=28):
    """a row with all lookups of its table, 63600 in 32 parts; rows with 65 to a quarter of a million; rows with some dozen and none"""
    return [T(1, dim, dtype, None, "fixed", 1, cache_slots=2), T(700, dim, dtype, 1.0, "fixed", pool, cache_slots=500),
            T(20000, dim, dtype, None, "fixed", 4, cache_slots=9000)]


@pytest.mark.parametrize("dim,dtype,pooling", [(4, synth.FP32, "mean"), (8, synth.FP32, "sum"), (16, synth.FP16, "mean")]
                         + [(d, synth.FP32, p) for d, p in ((16, "sum"), (20, "mean"), (64, "mean"), (128, "sum"), (256, "mean"))]
                         + [(d, synth.FP16, p) for d, p in ((32, "mean"), (40, "sum"), (128, "mean"), (256, "sum"), (512, "sum"))])
def test_rows_of_every_width(dim, dtype, pooling):
    steps = 2 if dtype == synth.FP16 and dim > 128 else 3  # (the oracle takes seconds a step)
    st = run_parity(synth.WorkloadCfg("tiles", heavy(dim, dtype), batch=BATCH, ways=2, steps=steps, seed=dim, init_std=0.05, lr=0.05), steps=steps,
                    order="early", pooling=pooling)
    assert st["last"]["lookups"] > 2097152 and st["last_long_rows"] > 300


@pytest.mark.parametrize("pooling", ["sum", "mean"])
def test_widths_side_by_side_and_sizes_in_turn(pooling):
    """rows of 2, 16 and 32 lanes in one model; batches of 63600 bags, 47448, one and 63600 a table: the tile kernel, the entries'
    kernel in between"""
    tabs = heavy(64, synth.FP32, 14) + heavy(256, synth.FP16, 8) + [T(90, 8, synth.FP32, 1.1, "fixed", 9, cache_slots=40)]
    st = run_parity(synth.WorkloadCfg("mixed", tabs, batch=BATCH, ways=2, steps=4, seed=3, init_std=0.05, lr=0.05), steps=4, order="ahead",
                    pooling=pooling, vary_batch=59)
    assert st["last_long_rows"] > 0


@pytest.mark.parametrize("bags", [2097153, 262145])
def test_few_heavy_rows_and_none(bags):
    """one lookup a bag, and eight: a single heavy row among rows with a lookup or two, then rows with 64 lookups at most"""
    pool = 1 if bags > 2000000 else 8
    for tabs in ([T(1, 16, synth.FP32, None, "fixed", 1, cache_slots=2)], [T(2000000, 16, synth.FP32, None, "fixed", pool, cache_slots=0)]):
        if pool > 1 and tabs[0].rows == 1:
            tabs = tabs + [T(900000, 16, synth.FP32, None, "fixed", pool - 1, cache_slots=0)]
        st = run_parity(synth.WorkloadCfg("few", tabs, batch=bags, ways=2, steps=2, seed=1, init_std=0.05, lr=0.05), steps=2, order="inline",
                        touched_only=True)
        assert (st["last_long_rows"] > 0) == (tabs[0].rows == 1)


@pytest.mark.parametrize("pooling", ["sum", "mean"])
def test_partial_sums_in_the_static_scratch(pooling):
    """tbe_backward_update_static: bit for bit what tbe_backward_update leaves, at each of three steps"""
    from paper_2305_01515_amd.tbe import TBE
    from parity_util import make_backing
    cfg = synth.WorkloadCfg("static", heavy(16, synth.FP32), batch=BATCH, ways=2, steps=3, seed=9, init_std=0.05, lr=0.05)
    stream = synth.BatchStream(cfg)
    batches = [tuple(x.cuda() for x in stream.next()) for _ in range(3)]
    grads = [synth.grad_out(cfg, s + 1).cuda() for s in range(3)]
    got = []
    for static in (False, True):
        _, _, W, M = make_backing(cfg)
        g = TBE(W, M, [t.cache_slots for t in cfg.tables], cfg.ways, cfg.batch, 2098800, pooling=pooling)
        outs = []
        for (idx, off), grad in zip(batches, grads):
            outs.append(g.forward(idx, off))
            (g.backward_update_static if static else g.backward_update)(grad, cfg.lr, cfg.eps)
        g.flush()
        got.append([o.cpu().numpy() for o in outs] + [x.numpy().copy() for x in W + M])
        g.close()
    assert all(np.array_equal(a, b) for a, b in zip(*got))
