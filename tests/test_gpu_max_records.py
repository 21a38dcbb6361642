"""Max pooling: who supplied the maxima, as the backward takes it (records of the lookups of binary16 rows, positions for
fp32 rows), and the kernel that gives the chains of lookups of a hot row a wavefront each: every number of lanes per row, rows with 65 to about a thousand lookups (one chunk a chain to many,
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
            T(1, dim, dtype, None, "fixed", 1), T(70, 24, synth.FP16 if dtype == synth.FP32 else synth.FP32, 1.1, "poisson", 4, 0, 20)]
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


@pytest.mark.parametrize("batch", [512, 513, 1024, 1025, 6000])
@pytest.mark.parametrize("dim", [64, 128, 200, 512])
def test_rows_around_the_line_of_the_hot_ones(dim, batch):
    """rows with exactly 512, 513, 1024 and 1025 lookups, binary16 rows of 8, 16, 32 and 64 lanes and fp32 rows of 16, 32 and 64
    beside each other, and several with many more"""
    half, full = synth.FP16, synth.FP32
    tabs = [T(1, dim, half, None, "fixed", 1, cache_slots=8), T(40, 20, full, 1.2, "fixed", 3, cache_slots=16),
            T(7, dim, half, 1.0, "poisson", 5, 0, 30, cache_slots=8), T(1, min(dim, 256), full, None, "fixed", 1),
            T(300, dim, half, 1.3, "poisson", 6, 0, 40, cache_slots=80), T(90, min(dim, 256), full, 1.3, "poisson", 5, 0, 40, cache_slots=40)]
    st = run_parity(synth.WorkloadCfg("hot", tabs, batch=batch, ways=8, steps=2, seed=dim + batch, init_std=0.05, lr=0.05), steps=2,
                    order="early", pooling="max")
    assert st["last_long_rows"] > 0 and st["parted_at"] is None


@pytest.mark.parametrize("dtype", [synth.FP32, synth.FP16])
def test_unpacked_payload_with_both_storage_types(dtype):
    """bags too long for the packed payload: positions come from the offsets, inside the bag for fp32 rows, in input order for
    binary16 rows"""
    other = synth.FP16 if dtype == synth.FP32 else synth.FP32
    tabs = [T(900, 64, dtype, 1.1, "poisson", 60, 0, 150, cache_slots=56), T(70, 24, other, 1.1, "poisson", 40, 0, 120)]
    st = run_parity(synth.WorkloadCfg("unpacked", tabs, batch=64, ways=8, steps=3, seed=94, init_std=0.05, lr=0.05), steps=3,
                    order="ahead", pooling="max", max_batch=1 << 26)
    assert st["last_long_rows"] > 0 and st["parted_at"] is None
