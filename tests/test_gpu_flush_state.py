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
