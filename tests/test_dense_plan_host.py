"""Where the uncompressed step may write its outputs inside the launch that reads its inputs (csrc/dense_plan.h): never when a byte of
either output is a byte of any input.  Spans at every distance around each other, against the bytes one by one."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_08317_amd", "csrc")
PROGRAM = r"""
#include <cstdio>
#include "dense_plan.h"
using rdkv::Span;
static bool share(const Span& a, const Span& b) {
  for (size_t i = 0; i < a.bytes; ++i)
    for (size_t j = 0; j < b.bytes; ++j)
      if (static_cast<const char*>(a.at) + i == static_cast<const char*>(b.at) + j) return true;
  return false;
}
int main() {
  static char memory[256];
  const size_t sizes[] = {0, 1, 4, 7};
  long n = 0, bad = 0;
  for (int in = 0; in < 3; ++in)
    for (int o = 0; o < 2; ++o)
      for (size_t a : sizes)
        for (size_t b : sizes)
          for (int at = -9; at <= 9; ++at) {
            // the others stand apart; one input and one output meet
            Span ins[3] = {{memory + 10, 5}, {memory + 30, 5}, {memory + 50, 5}}, outs[2] = {{memory + 100, 5}, {memory + 120, 5}};
            ins[in] = {memory + 200, a};
            outs[o] = {memory + 200 + at, b};
            ++n;
            bad += rdkv::dense_outputs_apart(ins[0], ins[1], ins[2], outs[0], outs[1]) == share(ins[in], outs[o]);
          }
  bad += !rdkv::dense_outputs_apart({memory, 5}, {memory + 5, 5}, {memory + 10, 5}, {memory + 15, 5}, {nullptr, 0});
  std::printf("%ld placements, %ld wrong\n", n, bad);
  return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_an_output_in_any_inputs_memory_is_seen(tmp_path):
    (tmp_path / "plan.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I" + CSRC, "-o", "plan", "plan.cpp"], cwd=tmp_path, check=True)
    p = subprocess.run([tmp_path / "plan"], capture_output=True, text=True)
    print(p.stdout)
    assert p.returncode == 0, p.stdout
