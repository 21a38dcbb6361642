"""Rows are moved by 4, 8 or 16 lanes of 16 bytes, by the widest row of the model: parity at the widths on either side
of every change, with tables of unlike width in one model, in the pipelines that move rows by other kernels."""
import pytest

from paper_2305_01515_amd import synth
from parity_util import run_parity

pytestmark = pytest.mark.gpu


def model(dims, dtype):
    tabs = [synth.TableCfg(900 + 37 * i, d, dtype, 1.05, "poisson", 6, 0, 40, cache_slots=16 * (5 + i)) for i, d in enumerate(dims)]
    return synth.WorkloadCfg("rows", tabs, batch=61, ways=16, steps=5, seed=77, init_std=0.05, lr=0.05)


# bytes of a row: 16, 64, 80, 128, 144 (fp32) and 112, 128, 144, 1024 (fp16)
@pytest.mark.parametrize("dims,dtype", [((4,), synth.FP32), ((16, 8), synth.FP32), ((20, 4), synth.FP32), ((32, 12), synth.FP32),
                                        ((36, 4), synth.FP32), ((56, 64), synth.FP16), ((72, 8), synth.FP16), ((512, 8), synth.FP16)])
@pytest.mark.parametrize("kw", [dict(order="ahead"), dict(order="pipe2"), dict(order="early", second_level_factor=2),
                                dict(order="inline", deferred_init=(5, 0.05), flush_every=2)],
                         ids=["ahead", "deep", "two_level", "deferred_flush"])
def test_rows_of_every_width(dims, dtype, kw):
    run_parity(model(dims, dtype), steps=5, **kw)
