"""Heavy rows (more than 64 lookups): a workgroup for each of a row's entries in the launch of the rest of the backward, or in one
behind it, up to 2097152 lookups, the tile kernel (or a launch of their own, for narrow rows) beyond."""
import pytest

from paper_2305_01515_amd import synth
from parity_util import run_parity

pytestmark = pytest.mark.gpu
T = synth.TableCfg


@pytest.mark.parametrize("pooling", ["sum", "mean"])
@pytest.mark.parametrize("dim,dtype,bags", [(4, synth.FP32, 1024), (16, synth.FP32, 1024), (64, synth.FP32, 256), (256, synth.FP32, 64),
                                            (128, synth.FP16, 256), (512, synth.FP16, 64), (24, synth.FP16, 1024)])
def test_either_side_of_the_line(dim, dtype, bags, pooling):
    """a few rows with most of the lookups, a row with 65, where bags x 16 lookups x lanes are 65536 lanes, one bag less and one more"""
    for batch in (bags - 1, bags, bags + 1):
        tabs = [T(5, dim, dtype, 1.2, "fixed", 15, cache_slots=4), T(batch // 65 + 1, dim, dtype, None, "fixed", 1, cache_slots=0)]
        st = run_parity(synth.WorkloadCfg("long", tabs, batch=batch, ways=2, steps=3, seed=batch, init_std=0.05, lr=0.05), steps=3,
                        order="early", pooling=pooling)
        assert st["last_long_rows"] > 0


def test_widths_on_both_sides_in_one_model():
    """rows of 64, 2 and 4 lanes side by side"""
    tabs = [T(4, 256, synth.FP32, 1.0, "fixed", 4, cache_slots=2), T(9, 8, synth.FP32, None, "fixed", 2, cache_slots=4),
            T(300, 32, synth.FP16, 1.2, "poisson", 2, 0, 9, cache_slots=64)]
    st = run_parity(synth.WorkloadCfg("widths", tabs, batch=256, ways=2, steps=4, seed=2, init_std=0.05, lr=0.05), steps=4, order="inline")
    assert st["last_long_rows"] > 0


@pytest.mark.parametrize("pooling", ["sum", "mean"])
@pytest.mark.parametrize("dim,dtype", [(4, synth.FP32), (20, synth.FP32), (256, synth.FP32), (128, synth.FP16)])
@pytest.mark.parametrize("n", [255, 256, 257, 512, 2049, 32768, 32769, 60000, 262145])
def test_rows_of_one_and_of_many_entries(n, dim, dtype, pooling):
    """a row with all n lookups of its table (an entry for every 256, 512 or 1024 of them), beside rows with none or one entry"""
    tabs = [T(1, dim, dtype, None, "fixed", 1, cache_slots=2), T(60, dim, dtype, 1.3, "fixed", 1, cache_slots=16)]
    st = run_parity(synth.WorkloadCfg("entries", tabs, batch=n, ways=2, steps=2, seed=n, init_std=0.05, lr=0.05), steps=2, order="early",
                    pooling=pooling)
    assert st["last_long_rows"] >= min(64, (n + 2047) // 2048)


WIDTHS = [(d, synth.FP32) for d in (4, 8, 16, 28, 64, 128, 256)] + [(d, synth.FP16) for d in (8, 16, 32, 40, 128, 256, 512)]


@pytest.mark.parametrize("dim,dtype,n,pooling", [(d, t, n, p) for d, t in WIDTHS for n, p in ((300, "mean"), (5000, "sum"))]
                         + [(8, synth.FP32, 524300, "mean"), (16, synth.FP16, 524300, "sum"), (128, synth.FP32, 524300, "sum")])
def test_rows_of_every_width(dim, dtype, n, pooling):
    """1 to 64 lanes a row: the sums of the lane groups of a wavefront, of its wavefronts and of a row's entries; a row with all
    lookups of its table, some hundred rows with 65 and more, in one launch with the other rows and in one behind them"""
    tabs = [T(1, dim, dtype, None, "fixed", 1, cache_slots=2), T(n // 150 + 1, dim, dtype, 0.8, "fixed", 1, cache_slots=16)]
    st = run_parity(synth.WorkloadCfg("width", tabs, batch=n // 2, ways=2, steps=2, seed=dim, init_std=0.05, lr=0.05), steps=2, order="early",
                    pooling=pooling)
    assert st["last_long_rows"] > 0


@pytest.mark.parametrize("n", [524288, 524289, 2097152, 2097153])
def test_either_side_of_the_larger_lines(n):
    """the launch of their own, and the tile kernel: rows with a third of the lookups, some hundred and none"""
    tabs = [T(3001, 32, synth.FP32, 1.4, "fixed", 1, cache_slots=2048)]
    st = run_parity(synth.WorkloadCfg("lines", tabs, batch=n, ways=8, steps=1, seed=3, init_std=0.05, lr=0.05), steps=1, order="early")
    assert st["last_long_rows"] > 100
