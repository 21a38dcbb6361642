"""The rules by which small batches take their ways through the library -- how many workgroups the one-kernel stage has, which
batches it takes -- on either side of their lines.  They are host functions of the sizes: compiled here from the header that
holds them, no GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
MAIN = r"""
#include <cstdio>
#include <cstring>
#include "tbe_internal.h"
using namespace tbe;
int main() {
  char what[64];
  long long T, sets, stride, n, batch, l2;
  while (scanf("%63s %lld %lld %lld %lld %lld %lld", what, &T, &sets, &stride, &n, &batch, &l2) == 7) {
    Geometry g{};
    g.T = (int)T;
    g.total_sets = (uint32_t)sets;
    g.ovf_stride = (uint32_t)stride;
    long long r = -1;
    if (!strcmp(what, "workgroups")) r = one_stage_workgroups(g, l2 != 0, n);
    if (!strcmp(what, "one_kernel")) r = one_kernel_batch(g, l2 != 0, false, n, (int)batch);
    if (!strcmp(what, "one_kernel_one_stream")) r = one_kernel_batch(g, l2 != 0, true, n, (int)batch);
    if (!strcmp(what, "link_with_stage")) r = link_with_stage(g, l2 != 0, n, (int)batch);
    if (!strcmp(what, "compute_stream_ordered")) r = on_compute_stream(g, false, l2 != 0, n);  // (l2: never_bypasses)
    if (!strcmp(what, "compute_stream_ready")) r = on_compute_stream(g, true, l2 != 0, n);
    if (!strcmp(what, "write_back_beside")) r = write_back_beside(g, n);
    g.probe_min_windows = (int)sets;
    if (!strcmp(what, "probe_min_windows")) r = probe_min_windows(g, (int)n);
    printf("%lld\n", r);
  }
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    if not shutil.which(HIPCC):
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.hip").write_text(MAIN)
    subprocess.check_call([HIPCC, "--offload-host-only", "-std=c++17", "-O0", "-w", "-I", os.path.join(ROOT, "paper_2305_01515_amd", "csrc"),
                           "-I", os.path.join(ROOT, "include"), str(d / "rules.hip"), "-o", str(d / "rules")])

    def ask(what, T=1, sets=0, row_bytes=64, n=1, batch=1, level2=0):
        line = f"{what} {T} {sets} {row_bytes} {n} {batch} {level2}\n"
        return int(subprocess.run([str(d / "rules")], input=line, capture_output=True, text=True, check=True).stdout)
    return ask


def test_workgroups_for_sets_and_for_lists(rule):
    """a thread per lookup even where a batch touches a handful of sets; a wavefront per set; one for some dozen lookups"""
    for n, want in ((1, 1), (64, 1), (65, 1), (1024, 1), (1025, 2), (2049, 3), (4096, 4)):
        assert rule("workgroups", sets=0, n=n) == want
    for sets, n, want in ((31, 4096, 4), (79, 4096, 5), (313, 4096, 16), (9999, 96, 6), (9999, 128, 8), (9999, 4096, 16), (9999, 64, 1)):
        assert rule("workgroups", sets=sets, n=n) == want
    for sets, n, want in ((313, 2048, 20), (511, 2048, 32), (512, 2048, 16), (31, 2048, 2)):  # (the table itself counts as a set)
        assert rule("workgroups", sets=sets, n=n, level2=1) == want


def test_batches_that_one_kernel_takes(rule):
    """with a prefetch stream and without; with a second level fewer where there are more than two and a half rows a set"""
    for T, sets, level2, most, one_stream in ((1, 0, 0, 4096, 1024), (512, 0, 0, 4096, 1024), (513, 0, 0, 1536, 512), (1, 900, 1, 2252, 1024),
                                              (1, 9999, 1, 4096, 1024), (1, 500, 1, 2048, 1024), (1, 0, 1, 2048, 1024), (513, 0, 1, 1536, 512)):
        for what, m in (("one_kernel", most), ("one_kernel_one_stream", one_stream)):
            assert rule(what, T=T, sets=sets, n=m, level2=level2) and not rule(what, T=T, sets=sets, n=m + 1, level2=level2)
    assert not rule("one_kernel", n=0)
    for T, batch in ((1, 2048), (2, 1024), (512, 4)):
        assert rule("one_kernel", T=T, batch=batch, n=500) and not rule("one_kernel", T=T, batch=batch + 1, n=500)


def test_few_rows_are_moved_on_the_stage_s_stream(rule):
    """1024 rows, or half a megabyte of them, as far as the one kernel goes; with a second level two and a half a set"""
    for row_bytes, sets, level2, most in ((16, 0, 0, 4096), (128, 0, 0, 4096), (256, 0, 0, 2048), (512, 0, 0, 1024), (1024, 0, 0, 1024),
                                          (16, 199, 1, 500), (1024, 9999, 1, 1024), (16, 9999, 1, 4096)):
        assert rule("link_with_stage", row_bytes=row_bytes, sets=sets, n=most, level2=level2)
        assert not rule("link_with_stage", row_bytes=row_bytes, sets=sets, n=most + 1, level2=level2)
    assert not rule("link_with_stage", T=2, batch=1025, n=500)  # more bags than the one kernel takes


def test_batches_that_go_to_the_compute_stream(rule):
    """prefetched by the forward itself: 65536 lookups; with the inputs ready 4 MB of rows, unless every row has its place in the
    cache"""
    for what, never_bypasses, row_bytes, most in (("compute_stream_ordered", 0, 1024, 65536), ("compute_stream_ordered", 1, 16, 65536),
                                                  ("compute_stream_ready", 0, 1024, 4096), ("compute_stream_ready", 0, 256, 16384),
                                                  ("compute_stream_ready", 0, 16, 65536), ("compute_stream_ready", 1, 1024, 65536)):
        assert rule(what, row_bytes=row_bytes, n=most, level2=never_bypasses)
        assert not rule(what, row_bytes=row_bytes, n=most + 1, level2=never_bypasses)


def test_long_write_backs_leave_the_compute_stream(rule):
    """32 MB of rows that may have been bypassed"""
    for row_bytes, least in ((1024, 32768), (512, 65536)):
        assert rule("write_back_beside", row_bytes=row_bytes, n=least) and not rule("write_back_beside", row_bytes=row_bytes, n=least - 1)


def test_what_the_caller_sets_of_the_probe_s_grouping_holds_for_every_batch(rule):
    """sets: what tbe_set_probe_grouping was given (0: not called); n: wavefronts of the one-kernel stage (0: another batch)"""
    for given in (1, 300, 4096, 1 << 30):
        for waves in (0, 16, 256):
            assert rule("probe_min_windows", sets=given, n=waves) == given
    assert rule("probe_min_windows", n=0) == 4096 and rule("probe_min_windows", n=16) == 16
