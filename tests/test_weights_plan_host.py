"""How the first weights pass cuts the key tiles into runs (csrc/weights_plan.h), against the cut itself: where the second pass is to
make the log-sum-exp, no item of any batch meets more runs than it reads; and runs of two tiles, which halve the first pass's
workgroups, are taken only where that spares the launch of the log-sum-exp.  Every length around the lines, alone and beside others,
with odd and even sums of tiles."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_08317_amd", "csrc")
PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "weights_plan.h"
static int first_tile(int w, int workgroups, int n_tiles) { return static_cast<int>(static_cast<int64_t>(w) * n_tiles / workgroups); }
int main() {
  long n = 0, bad = 0, halves = 0, paired66 = 0;
  std::vector<std::vector<int>> batches;
  for (int L = 1; L <= 140; ++L)
    for (int heads = 1; heads <= 8; heads *= 2)
      for (int other : {0, 1, 2, 33, 66, 67}) {
        std::vector<int> items;
        for (int h = 0; h < heads; ++h) items.push_back(L);
        for (int h = 0; other && h < heads; ++h) items.push_back(other);
        batches.push_back(items);
        batches.push_back({items.rbegin(), items.rend()});
        if (L % 7 == 0) batches.push_back(std::vector<int>(512 / L * 2 + 3, L));
      }
  for (const auto& items : batches)
    for (int rows : {64, 128, 132, 256}) {
      int tiles = 0, most = 0;
      for (int t : items) { tiles += t; most = std::max(most, t); }
      const rdkv::RunPlan p = rdkv::run_plan(tiles, most, rows, 2);
      bool ok = p.workgroups >= 1 && p.workgroups <= rdkv::workgroups_of(tiles, 2);
      const bool half = p.workgroups < rdkv::workgroups_of(tiles, 2);
      halves += half;
      ok = ok && (!half || (p.few && rows <= 128));
      std::vector<int> run(tiles);
      for (int w = 0; w < p.workgroups; ++w)
        for (int t = first_tile(w, p.workgroups, tiles); t < first_tile(w + 1, p.workgroups, tiles); ++t) run[t] = w;
      int t0 = 0;
      for (int t : items) {
        if (p.few && run[t0 + t - 1] - run[t0] + 1 > rdkv::kFewRuns) ok = false;
        t0 += t;
      }
      if (half && most == 66) ++paired66;
      ++n;
      if (!ok && bad++ < 5) std::printf("%zu items, %d tiles, the longest of %d, %d rows: %d workgroups, few %d\n", items.size(), tiles, most, rows, p.workgroups, p.few);
    }
  std::printf("%ld batches, %ld wrong, %ld in pairs\n", n, bad, halves);
  return bad != 0 || halves == 0 || paired66 == 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_runs_of_every_item_are_as_few_as_the_second_pass_reads(tmp_path):
    (tmp_path / "plan.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I" + CSRC, "-o", "plan", "plan.cpp"], cwd=tmp_path, check=True)
    p = subprocess.run([tmp_path / "plan"], capture_output=True, text=True)
    print(p.stdout)
    assert p.returncode == 0, p.stdout
