"""The sort's rules: whatever the model and the batch, the scratch that a handle allocates is large enough, and the key
generation's workgroups, which write some thousand counters each, are 1024 or as many as have 256 lookups.  Host functions of the
sizes, compiled here from the header that holds them, no GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
MAIN = r"""
#include <cstdio>
#include <random>
#include "tbe_internal.h"
using namespace tbe;
int main() {
  std::mt19937_64 rng(7);
  auto upto = [&](double most) { return (long long)std::exp(std::uniform_real_distribution<>(0, std::log(most))(rng)); };
  for (int model = 0; model < 30000; model++) {
    Geometry g{};
    g.T = model % 3 ? (int)upto(600) : model % 2 ? 512 : 513;
    g.seg_bits = 1 + (int)(rng() % 32);
    g.key_bits = std::min(32, g.seg_bits + (int)(rng() % 10));
    const int max_batch = (int)upto(std::min(4e6, 2147483647.0 / g.T));
    const long long max_n = upto(5e7);
    const SortNeeds need = sort_needs(g, max_n, max_batch);
    for (int x = 0; x < 60; x++) {
      const long long line[] = {kTiles1k, kTiles1kSegment, kTiles2k, kTiles4k, kSegmentLookups * g.T, kTiles1k * g.T, 2ll * g.T * max_batch};
      long long n = x < 30 ? upto(max_n + 1.0) : line[x % 7] + x % 3 - 1;
      if (n > max_n || n < 0) n = max_n;
      const int batch = x % 4 ? (int)upto(max_batch + 1.0) : max_batch;
      const SortShape s = sort_shape(g, n, batch);
      const long long words = (long long)s.digits.passes << s.rb, bags = (long long)g.T * batch;
      const bool ok = (long long)(s.slots + 1) * s.segs * words <= need.slots && s.tiles <= need.tiles && (2ll * s.tiles << s.rb) <= need.said &&
                      s.slots >= 1 && (long long)s.slots * s.segs <= std::max(1024ll, n / 256) && (s.add_slots || s.slots <= kSlotsHeard) &&
                      s.digits.passes <= kMaxSortPasses && s.rb <= 10 && (long long)s.bags * s.segs == bags && s.segs <= kLutTables &&
                      s.lanes == (n <= 2 * bags ? 1 : 8);
      if (!ok) {
        printf("T %d seg_bits %d key_bits %d max_batch %d max_n %lld batch %d n %lld: slots %d segs %d lanes %d tiles %d\n", g.T, g.seg_bits,
               g.key_bits, max_batch, max_n, batch, n, s.slots, s.segs, s.lanes, s.tiles);
        return 1;
      }
    }
  }
  printf("ok\n");
}
"""


def test_scratch_and_workgroups_of_any_model(tmp_path):
    if not shutil.which(HIPCC):
        pytest.skip("no hipcc")
    (tmp_path / "shapes.hip").write_text(MAIN)
    subprocess.check_call([HIPCC, "--offload-host-only", "-std=c++17", "-O1", "-w", "-I", os.path.join(ROOT, "paper_2305_01515_amd", "csrc"),
                           "-I", os.path.join(ROOT, "include"), str(tmp_path / "shapes.hip"), "-o", str(tmp_path / "shapes")])
    r = subprocess.run([str(tmp_path / "shapes")], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout
