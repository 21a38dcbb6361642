"""What makes the waits of the prefetch stage safe: a workgroup that has looked for long at what another one has yet to say counts
that one's part itself.  In libtbe.so it looks 64 times first, which these sizes do not provoke; here are builds of it that look 0
times -- every workgroup of the distinct rows' pass and of the lists' counts all those before it, a tile of the sort those that have
not spoken at its first look -- and once, so that what was heard and what was counted meet in one sum.  Cache state and lists bit
for bit against the oracle, values on its bars."""
import os

import pytest

from paper_2305_01515_amd import synth
from parity_util import run_parity

pytestmark = pytest.mark.gpu
T = synth.TableCfg


@pytest.fixture(params=[0, 1], ids=["looks_0", "looks_1"])
def impatient(request, monkeypatch):
    from paper_2305_01515_amd import build, tbe
    path = build.IMPATIENT[request.param]
    if not os.path.exists(path):
        build.build()
    monkeypatch.setattr(tbe, "LIB_PATH", path)
    monkeypatch.setattr(tbe, "_lib", None)
    assert tbe.lib()._name == path
    return request.param


def parity(tabs, batch, seed, **kw):
    return run_parity(synth.WorkloadCfg("recount", tabs, batch=batch, ways=8, steps=kw.get("steps", 3), seed=seed, init_std=0.05, lr=0.05),
                      **{"steps": 3, "order": "early", **kw})


@pytest.mark.parametrize("bits", [9, 16, 20, 23])
@pytest.mark.parametrize("batch", [700, 5000, 17000])
def test_segments_of_unlike_size(impatient, batch, bits):
    """tiles of 1024, 2048 and 4096 keys; digits of 8 to 10 bits, keys of one to three passes; tables without a lookup and of one row"""
    tabs = [T((1 << bits) - 1, 4, synth.FP32, 0.9, "fixed", 20, cache_slots=8 * 300), T(50, 4, synth.FP32, None, "fixed", 0, cache_slots=8),
            T(3001, 4, synth.FP32, None, "fixed", 2), T(1, 4, synth.FP32, None, "fixed", 1, cache_slots=8),
            T(900, 4, synth.FP32, 1.1, "poisson", 9, 0, 60, cache_slots=160)]
    parity(tabs, batch, bits)


@pytest.mark.parametrize("tables,rows,pool,batch", [(1, 1000003, 32, 2048), (70, 900, 2, 936), (26, 30000, 9, 190)])
def test_one_segment_of_tiles_of_1024_keys(impatient, tables, rows, pool, batch):
    parity([T(rows, 4, synth.FP32, 0.7, "fixed", pool, cache_slots=8 * 100) for _ in range(tables)], batch, batch)


def test_tiles_of_8192_keys(impatient):
    parity([T(60013, 4, synth.FP32, 1.1, "fixed", 30, cache_slots=8 * 2000), T(3001, 4, synth.FP32, None, "fixed", 2)], 66000, 1, steps=1)


def test_more_lookups_than_the_distinct_rows_pass_has_workgroups_for(impatient):
    parity([T(900001, 4, synth.FP32, 0.8, "fixed", 128, cache_slots=8 * 20000)], 66000, 5, steps=1)


@pytest.mark.parametrize("second_level", [0, 2])
@pytest.mark.parametrize("order", ["ahead", "inline"])
def test_misses_and_two_levels(impatient, order, second_level):
    """rows that hit, push others out, bypass and come back; lists of every kind, rows entered once and several times"""
    tabs = [T(40000, 16, synth.FP16, 0.7, "poisson", 12, 0, 90, cache_slots=8 * 900), T(2500, 32, synth.FP32, 1.2, "poisson", 9, 0, 60, cache_slots=8 * 20),
            T(600, 8, synth.FP32, None, "fixed", 3)]
    st = parity(tabs, 1500, 11, steps=6, order=order, second_level_factor=second_level, flush_every=2 if order == "inline" else 0)
    assert st["total"]["evictions"] > 0 and st["total"]["bypasses"] > 0 and st["last_long_rows"] > 0


@pytest.mark.parametrize("order", ["pipe3", "early"])
def test_max_pooling_and_a_deep_pipeline(impatient, order):
    parity([T(9000, 16, synth.FP32, 0.9, "poisson", 6, 0, 40, cache_slots=8 * 500), T(70, 32, synth.FP32, 1.0, "fixed", 2, cache_slots=16)], 1500, 4,
           steps=5, order=order, pooling="max")


def test_more_tables_than_constants_fit_in_lds(impatient):
    parity([T(5 + t % 13, 4, synth.FP32, None, "fixed", t % 4, cache_slots=8 * (t % 3)) for t in range(523)], 40, 5)
