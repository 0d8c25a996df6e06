"""The stop flag of launches that record the launch before them: whenever the
waves of a launch look at it, before or after their own launch's recording
block has set it, they decide alike, and every launch after that one skips.
The header the kernels include, compiled for the CPU and driven through all
positions of the recording block among its launch's waves."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1610_06749_amd", "csrc")

HARNESS = r"""
#include <cstdio>
#include "stop_flag.h"
using namespace it;
// Launches 0, 1, ... of alternating parity; launch l records launch l - 1,
// whose step ends the run if it is `last`, and its recording block acts after
// `at` of its `waves` readers have looked.  A launch is of one-step kernels,
// whose waves each look at their parity's bit, or (bit l % 4 of `blocked`) of a
// pass of several steps, whose blocks each look once at the whole flag and whose
// first block passes a stop on.  With close >= 0 a launch without tile blocks
// records launch `close` before launch close + 1, which then has no recording
// block.
static int run(int last, int first_parity, int blocked, int at, int waves, int close) {
  int f = 0;
  long passes = first_parity;  // launches recorded (the parity is theirs)
  for (int l = 0; l < last + 8; ++l) {
    const int parity = (l + first_parity) & 1;
    const bool several = blocked >> (l % 4) & 1;
    int skipped = 0;
    for (int w = 0; w <= waves; ++w) {
      if (w == at && l > 0 && l - 1 != close) {
        if (f) {
          if (!several) f = kStopAll;
        } else {
          if (((passes + 1) & 1) != parity) return 3;  // the kernels take it from there
          if (l - 1 == last) f = stop_after(parity);
          ++passes;
        }
      }
      if (w == waves) break;
      const bool skips = several ? f != 0 : launch_skips(f, parity);
      if (several && skips && w == 0) f = kStopAll;
      skipped += skips;
    }
    // launch last + 1 steps past the stop, unless a closing launch came before
    // it; the blocks of a pass of several steps may find the stop or not
    const int until = close == last ? last : last + 1;
    if (several && l == last + 1 && close != last) {
    } else {
      if (skipped != 0 && skipped != waves) return 1;  // the waves disagree
      if ((skipped == waves) != (l > until)) return 2;
    }
    if (l == close) {
      if (!f) ++passes;
      if (f || l == last) f = kStopAll;
    }
  }
  return 0;
}
int main() {
  for (int last = 0; last < 5; ++last)
    for (int parity = 0; parity < 2; ++parity)
      for (int blocked = 0; blocked < 16; ++blocked)
        for (int at = 0; at <= 4; ++at)
          for (int close = -1; close < 9; ++close)
            if (int bad = run(last, parity, blocked, at, 4, close)) {
              std::printf("last %d parity %d blocked %d at %d close %d: %d\n", last, parity, blocked, at, close, bad);
              return 1;
            }
  return 0;
}
"""


def test_waves_of_a_launch_decide_alike(tmp_path):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no host compiler")
    src = tmp_path / "harness.cpp"
    src.write_text(HARNESS)
    exe = str(tmp_path / "harness")
    subprocess.check_call([cxx, "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
