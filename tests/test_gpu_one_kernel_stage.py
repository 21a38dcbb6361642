"""The prefetch stage of very small batches, which is one kernel: lookups and bags on either side of the lines up to which it is
taken, one workgroup and many, every replacement policy and level, and such batches in turn with larger ones."""
import pytest

from paper_2305_01515_amd import synth
from parity_util import run_parity

pytestmark = pytest.mark.gpu
T = synth.TableCfg


@pytest.mark.parametrize("policy,level2", [("lru", 0), ("lfu", 0), ("lru", 1), ("lfu", 2)])
@pytest.mark.parametrize("batch,pool", [(1, 7), (16, 4), (255, 16), (256, 16), (257, 16), (1023, 4), (1024, 4), (1025, 3)])
def test_lookups_and_bags_around_the_lines(batch, pool, policy, level2):
    """4080, 4096 and 4112 lookups; 2046, 2048 and 2050 bags; sets by the thousand (many workgroups) and a handful (few).  (With a
    second level the line is at 2048 lookups, see below.)"""
    for rows, slots in ((9001, 4 * 700), (90, 4 * 3)):
        tabs = [T(rows, 8, synth.FP32, 0.9, "fixed", pool - pool // 2, cache_slots=slots),
                T(rows // 2, 16, synth.FP32, None, "fixed", pool // 2, cache_slots=slots // 2)]
        run_parity(synth.WorkloadCfg("one", tabs, batch=batch, ways=4, steps=4, seed=batch, init_std=0.05, lr=0.05), steps=4,
                   order="early", policy=policy, second_level_factor=level2)


@pytest.mark.parametrize("batch,pool,order,level2,overlap", [(127, 16, "early", 2, True), (128, 16, "early", 2, True), (129, 16, "early", 2, True),
                                                             (63, 16, "early", 0, False), (64, 16, "inline", 1, False), (65, 16, "early", 0, False)])
def test_lookups_around_the_other_lines(batch, pool, order, level2, overlap):
    """2048 lookups with a second level of few sets, 1024 on one stream"""
    tabs = [T(9001, 8, synth.FP32, 0.9, "fixed", pool - 3, cache_slots=4 * 300), T(700, 16, synth.FP32, None, "fixed", 3, cache_slots=64)]
    run_parity(synth.WorkloadCfg("other", tabs, batch=batch, ways=4, steps=4, seed=batch, init_std=0.05, lr=0.05), steps=4,
               order=order, second_level_factor=level2, overlap=overlap)


@pytest.mark.parametrize("overlap,batch", [(True, 168), (False, 42)])
def test_in_turn_with_larger_batches(overlap, batch):
    """Poisson bags: batches of one model fall on both sides of the line, 4096 lookups beside training and 1024 on one stream"""
    tabs = [T(3000, 16, synth.FP16, 1.0, "poisson", 20.3, 0, 60, cache_slots=256), T(500, 8, synth.FP32, None, "poisson", 4, 0, 20)]
    run_parity(synth.WorkloadCfg("turn", tabs, batch=batch, ways=16, steps=12, seed=1, init_std=0.05, lr=0.05), steps=12,
               order="early", overlap=overlap)


@pytest.mark.parametrize("policy,level2", [("lru", 1), ("lfu", 2), ("lru", 0)])
def test_many_rows_of_few_sets(policy, level2):
    """400 sets and 2048 lookups: with a second level 26 workgroups, without one 16; a table without a cache beside them"""
    tabs = [T(20000, 8, synth.FP32, None, "fixed", 3, cache_slots=400 * 4), T(3000, 16, synth.FP32, 0.8, "fixed", 1, cache_slots=0)]
    run_parity(synth.WorkloadCfg("few", tabs, batch=512, ways=4, steps=5, seed=8, init_std=0.05, lr=0.05), steps=5,
               order="early", policy=policy, second_level_factor=level2)


@pytest.mark.parametrize("tables", [512, 513, 900])
def test_many_tables(tables):
    """up to 512 tables the constants are in LDS; more are looked up in memory"""
    tabs = [T(5 + t % 13, 4, synth.FP32, None, "fixed", t % 4 == 1, cache_slots=4 * (t % 3)) for t in range(tables)]
    run_parity(synth.WorkloadCfg("many", tabs, batch=2, ways=4, steps=3, seed=5, init_std=0.05, lr=0.05), steps=3, order="early")


@pytest.mark.parametrize("order,level2", [("early", 0), ("ahead", 0), ("pipe2", 0), ("early", 2)])
def test_rows_of_some_batches_on_the_stage_s_stream(order, level2):
    """batches of about 1024 rows of 1 KB, half of them bypassed: the rows of some are moved on the stage's stream, those of others
    on the link's, in turn"""
    tabs = [T(3000, 256, synth.FP32, None, "poisson", 5, 0, 40, cache_slots=(405 if level2 else 100) * 4), T(800, 256, synth.FP32, 0.9, "poisson", 3, 0, 20, cache_slots=0)]
    st = run_parity(synth.WorkloadCfg("wide", tabs, batch=128, ways=4, steps=12, seed=6, init_std=0.05, lr=0.05), steps=12,
                    order=order, second_level_factor=level2)
    assert st["total"]["bypasses"] > 0 and st["total"]["evictions"] > 0


@pytest.mark.parametrize("min_windows", [1, 100, 1 << 30])
def test_probe_grouping_that_the_caller_sets(min_windows):
    tabs = [T(20000, 8, synth.FP32, None, "fixed", 3, cache_slots=400 * 4), T(3000, 16, synth.FP32, 0.8, "fixed", 1, cache_slots=60)]
    run_parity(synth.WorkloadCfg("group", tabs, batch=500, ways=4, steps=4, seed=8, init_std=0.05, lr=0.05), steps=4, order="early",
               probe_min_windows=min_windows)
