"""The sort of a kernel a pass at the sizes where it can go wrong: segments that begin and end anywhere in a tile or have no
lookup, digits of every width, tiles of every size, slots that the sort adds up itself or has added up, and more lookups than
the pass behind it has workgroups for.  Cache state and lists bit for bit against the oracle, values on its bars."""
import numpy as np
import pytest

from paper_2305_01515_amd import synth
from parity_util import run_parity

pytestmark = pytest.mark.gpu
T = synth.TableCfg


def parity(tabs, batch, seed, steps=2):
    run_parity(synth.WorkloadCfg("segments", tabs, batch=batch, ways=8, steps=steps, seed=seed, init_std=0.05, lr=0.05), steps=steps, order="early")


@pytest.mark.parametrize("bits", [3, 8, 9, 10, 11, 12, 16, 20, 21, 22, 23])
def test_digits_of_every_width(bits):
    """one table whose keys have so many bits, then three side by side (a segment each: more than 2048 lookups a table)"""
    one = [T((1 << bits) - 1, 4, synth.FP32, 0.9, "fixed", 3, cache_slots=8 * (1 << min(bits, 9)))]
    parity(one, 2100, bits)
    parity(one + [T(5, 4, synth.FP32, None, "fixed", 3, cache_slots=8), T(777, 4, synth.FP32, None, "fixed", 3)], 2100, bits)


@pytest.mark.parametrize("batch", [1023, 1024, 1025, 2047, 2048, 2049, 4097])
def test_segments_around_the_tiles(batch):
    """tables of one, of two and of no lookup a bag; on average 2048 lookups a table from a batch of 2048 on"""
    tabs = [T(3000, 4, synth.FP32, None, "fixed", 1, cache_slots=160), T(50, 4, synth.FP32, None, "fixed", 0, cache_slots=8),
            T(900, 4, synth.FP32, 1.2, "fixed", 2, cache_slots=80), T(40, 4, synth.FP32, 1.0, "poisson", 1.0, 0, 9),
            T(7, 4, synth.FP32, None, "fixed", 1, cache_slots=8)]
    parity(tabs, batch, batch)


@pytest.mark.parametrize("batch,pool", [(9000, 1), (9000, 3), (70000, 1)])
def test_more_slots_than_the_sort_adds_up_itself(batch, pool):
    parity([T(20011, 4, synth.FP32, 1.0, "fixed", pool, cache_slots=8 * 400)], batch, batch)


@pytest.mark.parametrize("tables,rows,pool,batch", [(1, 1000003, 32, b) for b in (2047, 2048, 2049, 4097)]
                         + [(70, 900, 2, b) for b in (936, 937)] + [(65, 900, 17, b) for b in (118, 119)])
def test_one_segment_of_tiles_that_hear_all_before_them(tables, rows, pool, batch):
    """one table by 10 bits: tiles of 1024 keys up to 65536 lookups, then of 2048; many tables with few lookups each by 8 bits: up to
    131072, the most tiles of 1024 keys that a segment can have"""
    parity([T(rows, 4, synth.FP32, 0.7, "fixed", pool, cache_slots=8 * 100) for _ in range(tables)], batch, batch, steps=2)


@pytest.mark.parametrize("batch", [16384, 16385, 65536, 65537])
def test_tiles_of_every_size(batch):
    """32 lookups a bag: either side of 524288 and of 2097152 lookups, in two segments of unlike size"""
    parity([T(60013, 4, synth.FP32, 1.1, "fixed", 30, cache_slots=8 * 2000), T(3001, 4, synth.FP32, None, "fixed", 2)], batch, batch, steps=1)


def test_more_lookups_than_the_distinct_rows_pass_has_workgroups_for():
    parity([T(900001, 4, synth.FP32, 0.8, "fixed", 128, cache_slots=8 * 20000)], 66000, 5, steps=1)


@pytest.mark.parametrize("tables", [511, 512, 513])
def test_as_many_tables_as_can_be_segments_and_one_more(tables):
    """one lookup a bag, 2049 of each table; beyond 512 tables they are one segment"""
    parity([T(3 + 7 * (t % 9), 4, synth.FP32, None, "fixed", 1, cache_slots=8 * (t % 3)) for t in range(tables)], 2049, tables, steps=1)


@pytest.mark.parametrize("within", [300, 1500])
@pytest.mark.parametrize("tables,batch", [(1, 3000), (3, 4100)])
def test_long_bags_among_short_ones(tables, batch, within):
    """two lookups a bag on average or fewer: a lane a bag, and all of a wavefront's lanes for what a bag has beyond 16; one segment and
    three; with room for 2^22 bags the payload takes bags of 1024 lookups, so that the longest fits or does not"""
    from test_gpu_mixed_calls import run
    rng = np.random.RandomState(within + tables)
    tabs = [T(40000 - 9000 * t, 4, synth.FP32, None, "fixed", 1, cache_slots=8 * 300) for t in range(tables)]
    host = []
    for step in range(3):
        lens = rng.poisson(0.6, (tables, batch))
        for at, n in zip(rng.choice(tables * batch, 12, False), (15, 16, 17, 18, 64, 79, 80, 81, 144, 200, within, 2)):
            lens.ravel()[at] = n
        lens[-1, -1] = 33 if step else 0  # the last bag, in a wavefront with few others
        off = np.concatenate([[0], np.cumsum(lens.ravel())]).astype(np.int64)
        host.append((np.concatenate([rng.randint(0, c.rows, l.sum()) for c, l in zip(tabs, lens)]).astype(np.int64), off,
                     rng.randn(batch, 4 * tables).astype(np.float32)))
    run(synth.WorkloadCfg("short", tabs, batch=(1 << 22) // tables, ways=8, steps=3, seed=1, init_std=0.05, lr=0.05), host, rng, False)
