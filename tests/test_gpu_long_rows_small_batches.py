"""Heavy rows (more than 64 lookups) of small batches: a workgroup each in the launch of the rest of the backward up to a number
of lookups that depends on the rows' lanes, the tile kernel (or a launch of their own, for narrow rows) beyond."""
import pytest

from paper_2305_01515_amd import synth
from parity_util import run_parity

pytestmark = pytest.mark.gpu
T = synth.TableCfg


@pytest.mark.parametrize("pooling", ["sum", "mean"])
@pytest.mark.parametrize("dim,dtype,bags", [(4, synth.FP32, 1024), (16, synth.FP32, 1024), (64, synth.FP32, 256), (256, synth.FP32, 64),
                                            (128, synth.FP16, 256), (512, synth.FP16, 64), (24, synth.FP16, 1024)])
def test_either_side_of_the_line(dim, dtype, bags, pooling):
    """bags x 16 lookups x lanes: 65536 lanes in all, and one bag less and more; a few rows with most of the lookups, a row with 65"""
    for batch in (bags - 1, bags, bags + 1):
        tabs = [T(5, dim, dtype, 1.2, "fixed", 15, cache_slots=4), T(batch // 65 + 1, dim, dtype, None, "fixed", 1, cache_slots=0)]
        st = run_parity(synth.WorkloadCfg("long", tabs, batch=batch, ways=2, steps=3, seed=batch, init_std=0.05, lr=0.05), steps=3,
                        order="early", pooling=pooling)
        assert st["last_long_rows"] > 0


def test_widths_on_both_sides_in_one_model():
    """2048 lookups: rows of 64 lanes take the tile kernel, the others share the rest's launch"""
    tabs = [T(4, 256, synth.FP32, 1.0, "fixed", 4, cache_slots=2), T(9, 8, synth.FP32, None, "fixed", 2, cache_slots=4),
            T(300, 32, synth.FP16, 1.2, "poisson", 2, 0, 9, cache_slots=64)]
    st = run_parity(synth.WorkloadCfg("widths", tabs, batch=256, ways=2, steps=4, seed=2, init_std=0.05, lr=0.05), steps=4, order="inline")
    assert st["last_long_rows"] > 0
