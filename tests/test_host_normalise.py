"""The vector arithmetic of the weight normalisation under UndefinedBehaviorSanitizer, on the CPU, with its float
arrays where a frame may put them: on 4 bytes, not on the vector's 16."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2206_15117_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

MAIN = r"""
#include <cmath>
#include <cstdio>
#include "weight_normalise.hpp"
struct alignas(16) Four { float v[4]; };
struct Frame { float pad; pg::Pixels<Four> img, weight; };
int main() {
  Frame f;
  const Four img = {{6.0f, NAN, 8.0f, -1.0f}}, weight = {{2.0f, 0.25f, 0.5f, NAN}}, low = {{0.0f, 0.1f, NAN, 0.4f}};
  f.img = pg::Pixels<Four>(img);
  f.weight = pg::Pixels<Four>(weight);
  const Four got = pg::over_weight(f.img, f.weight, 0.5f);
  const bool any = pg::any_reaches(f.weight, 0.5f), none = pg::any_reaches(pg::Pixels<Four>(low), 0.5f);
  const float one = pg::over_weight(pg::Pixels<float>(3.0f), pg::Pixels<float>(0.75f), 0.5f);
  return got.v[0] == 3.0f && got.v[1] == 0.0f && got.v[2] == 16.0f && got.v[3] == 0.0f && any && !none && one == 4.0f ? 0 : 1;
}
"""


def test_no_misaligned_vector_access(tmp_path):
    if shutil.which("g++") is None or not os.path.exists(os.path.join(ROCM, "include", "hip", "hip_runtime.h")):
        pytest.skip("g++ or the HIP headers are not installed")
    src, exe = tmp_path / "main.cpp", str(tmp_path / "main")
    src.write_text(MAIN)
    res = subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                          "-D__HIP_PLATFORM_AMD__", "-I", CSRC, "-I", os.path.join(ROCM, "include"), str(src), "-o", exe],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    res = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0 and "runtime error" not in res.stderr, res.stderr
