"""Max pooling: the lookups' records of the maxima they supplied, and the kernel that gives a row's chains of lookups a
wavefront each: every number of lanes per row, rows with 65 to about a thousand lookups (one chunk a chain to many,
ragged ends)."""
import pytest
import torch

from paper_2305_01515_amd import synth
from parity_util import run_parity

pytestmark = pytest.mark.gpu
T = synth.TableCfg


@pytest.mark.parametrize("dim,dtype", [(4, synth.FP32), (8, synth.FP32), (16, synth.FP32), (20, synth.FP32), (32, synth.FP32),
                                       (64, synth.FP32), (100, synth.FP32), (256, synth.FP32), (8, synth.FP16), (64, synth.FP16),
                                       (128, synth.FP16), (200, synth.FP16), (512, synth.FP16)])
def test_rows_of_every_width_and_length(dim, dtype):
    tabs = [T(900, dim, dtype, 1.3, "poisson", 9, 0, 60, cache_slots=16 * 9), T(3, 16, dtype, None, "fixed", 2, cache_slots=16),
            T(1, dim, dtype, None, "fixed", 1)]
    st = run_parity(synth.WorkloadCfg("rec", tabs, batch=523, ways=16, steps=3, seed=dim, init_std=0.05, lr=0.05), steps=3,
                    order="early", pooling="max")
    assert st["last_long_rows"] > 0 and st["parted_at"] is None  # no near-tie taken differently: values compared to the end


def test_records_take_no_memory_of_their_own():
    """a byte per lane and lookup, in memory that the handle has anyway: setting the mode allocates the positions alone"""
    from paper_2305_01515_amd.tbe import TBE, lib, pinned_empty
    n, batch, dim = 1 << 20, 64, 256
    g = TBE([pinned_empty((1000, dim), torch.float32).zero_()], [pinned_empty((1000,), torch.float32).zero_()], [64], 8, batch, n)
    free = torch.cuda.mem_get_info()[0]
    assert lib().tbe_set_pooling(g._h, 2) == 0
    taken = free - torch.cuda.mem_get_info()[0]
    assert taken <= 3 * 4 * (n + batch * dim) + (16 << 20)  # three buffers; (one such record: 64 MB)
    g.close()
