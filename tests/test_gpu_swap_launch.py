"""Transfer and commit of a batch with none in flight: one launch up to 8192 lookups, two beyond, in turn in one model."""
import pytest

from paper_2305_01515_amd import synth
from parity_util import run_parity

pytestmark = pytest.mark.gpu
T = synth.TableCfg


@pytest.mark.parametrize("order", ["inline", "serial"])
@pytest.mark.parametrize("level2,init,overlap", [(0, None, True), (2, None, True), (1, (3, 0.05), True), (0, (4, 0.05), False)])
@pytest.mark.parametrize("batch,dim,dtype", [(1, 16, synth.FP32), (127, 64, synth.FP16), (1023, 256, synth.FP32), (1024, 4, synth.FP32),
                                             (1025, 128, synth.FP16)])
def test_batches_on_both_sides_of_the_line(batch, dim, dtype, level2, init, overlap, order):
    """1024 bags of 8 lookups: 8192.  Rows that hit, that push others out, that bypass, that come back at once; batches of varying
    size, so that the list of parked victims is longer than the next batch's rows and shorter"""
    tabs = [T(4 * batch + 50, dim, dtype, 0.6, "fixed", 5, cache_slots=4 * (batch // 4 + 1)),
            T(batch + 9, 16, synth.FP32, None, "fixed", 3, cache_slots=4 * (batch // 16 + 1))]
    st = run_parity(synth.WorkloadCfg("swap", tabs, batch=batch, ways=4, steps=6, seed=batch, init_std=0.05, lr=0.05), steps=6, order=order,
                    overlap=overlap, second_level_factor=level2, deferred_init=init, vary_batch=7 if batch > 1 else 0)
    if batch > 1:
        assert st["total"]["bypasses"] > 0 and st["total"]["evictions"] > 0


@pytest.mark.parametrize("batch", [40, 1024, 1100])
def test_after_a_pipeline_and_a_flush(batch):
    """overlapped batches, whose commits park the copies of the batch before, end with a batch that nothing is prefetched behind"""
    tabs = [T(5 * batch, 64, synth.FP16, 0.5, "poisson", 8, 0, 30, cache_slots=4 * (batch // 4 + 1))]
    cfg = synth.WorkloadCfg("after", tabs, batch=batch, ways=4, steps=5, seed=batch, init_std=0.05, lr=0.05)
    run_parity(cfg, steps=5, order="ahead")
    run_parity(cfg, steps=5, order="inline", flush_every=2)
