"""The stop of a minor cycle, on the CPU: one workgroup writes it while the launch's other waves may read it
before or after.  Waves of one workgroup that went different ways would leave a barrier without the others' maxima."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2206_15117_amd", "csrc")

MODEL = r"""
#include <cstdio>
#include "clean_state.hpp"
using namespace pg;
int main() {
  int bad = 0;
  for (int max_iter = 0; max_iter <= 6; ++max_iter)
    for (int stops = 0; stops <= max_iter; ++stops) {  // iteration `stops` finds nothing; stops = max_iter: none does
      CleanState st{kCleanRuns};
      int taken = 0;
      for (int step = 0; step < max_iter; ++step) {
        const CleanState before = st;
        const bool runs = !clean_over(before.stop, step);
        if (runs && step == stops) st.stop = step;
        bad += clean_over(before.stop, step) != clean_over(st.stop, step);  // a wave that read it late
        taken += runs && step < stops;
        bad += runs && step > stops;
      }
      bad += taken != stops || clean_components(st.stop, max_iter) != stops;
    }
  std::printf("%d\n", bad);
  return bad != 0;
}
"""


def test_every_wave_of_a_launch_goes_the_same_way(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ is not installed")
    src, exe = tmp_path / "model.cpp", str(tmp_path / "model")
    src.write_text(MODEL)
    res = subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(src), "-o", exe], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    res = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, res.stdout
