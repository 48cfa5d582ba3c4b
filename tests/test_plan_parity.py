"""Launches of a captured call (csrc/lbm_plan.h, steps_ahead_parity), without a GPU: they add up to
the call's steps, none is longer than the plan's, and they are odd or even in number as asked."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_21242_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "lbm_plan.h"
int main() {
  for (int most : {2, 3, 4, 5, 7, 8, 64, 4096})
    for (int tile = most > 4; tile < 2; ++tile)
      for (long n = 1; n < 300; ++n)
        for (int odd = 0; odd < 2; ++odd) {
          if (n == 1 && !odd) continue;  // one step is one launch
          long left = n, count = 0, want = odd;
          while (left > 0) {
            const long s = lbm::steps_ahead_parity(left, tile ? 0 : most, tile ? most : 0, want);
            if (s < 1 || s > most || s > left) { std::printf("n %ld most %d: launch of %ld\n", n, most, s); return 1; }
            left -= s;
            want ^= 1;
            ++count;
          }
          if (count % 2 != odd) { std::printf("n %ld most %d tile %d: %ld launches\n", n, most, tile, count); return 1; }
          long plain = 0;
          for (long m = n; m > 0; m -= lbm::steps_ahead(m, tile ? 0 : most, tile ? most : 0)) ++plain;
          if (count > plain + 2) { std::printf("n %ld most %d: %ld launches, %ld\n", n, most, count, plain); return 1; }
        }
  std::puts("ok");
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_captured_calls_keep_the_parity_of_their_launches(tmp_path):
    src = tmp_path / "parity.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "parity"
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
