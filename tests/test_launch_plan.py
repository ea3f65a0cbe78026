"""The integer arithmetic that says which workgroup does what (csrc/launch_plan.h), compiled by the host compiler and enumerated."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2508_02317_amd", "csrc")


def _run(tmp_path, body):
    """Compiles a program around the header and returns what it prints; it must end with status 0."""
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    src, exe = str(tmp_path / "plan.cpp"), str(tmp_path / "plan")
    open(src, "w").write('#include <algorithm>\n#include <cstdio>\n#include <random>\n#include <vector>\n#include "launch_plan.h"\n'
                         "using namespace moe;\n" + body)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I", CSRC, src, "-o", exe], check=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    assert res.returncode == 0, res.stdout[-2000:]
    return res.stdout


def test_a_launch_has_fewer_than_2_to_the_32_threads(tmp_path):
    """The fp32 data and weight gradients share a launch: the workgroups of 480 million rows and of their combine weights, 32 and 256
    rows each, fit one by one but not together."""
    _run(tmp_path, """int main() {
      const size_t rows = 480000000, dx = rows / 32 + 1024, wgrad = 3 * 1024 + rows / 256;
      const bool ok = fits_one_launch(dx, 256) && fits_one_launch(wgrad, 256) && !fits_one_launch(dx + wgrad, 256) &&
                      fits_one_launch(16777215, 256) && !fits_one_launch(16777216, 256) && fits_one_launch(4194303, 1024) && !fits_one_launch(4194304, 1024);
      return ok ? 0 : 1;
    }""")
