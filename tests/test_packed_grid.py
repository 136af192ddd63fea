"""The packed kernel's grid rule, which the planner and the launcher share:
no schedule is planned that the launcher would refuse (host code, no GPU)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

PROGRAM = """
#include <cstdio>
#include "kernels.hpp"
int main() {
  long long threads, tiles, whole, shares;
  while (std::scanf("%lld %lld %lld %lld", &threads, &tiles, &whole, &shares) == 4)
    std::printf("%d\\n", int(comet::packed_grid_fits(threads, tiles, whole, shares)));
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="host compiler not found")
def test_grid_rule(tmp_path):
    src, exe = tmp_path / "grid.cpp", str(tmp_path / "grid")
    src.write_text(PROGRAM)
    p = subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(ROCM, "include"),
                        "-I" + os.path.join(ROOT, "include"),
                        "-I" + os.path.join(ROOT, "paper_2102_06827_amd", "csrc"), str(src), "-o", exe],
                       capture_output=True, text=True)
    assert p.returncode == 0, p.stderr[-2000:]
    lim = (2**32 - 1) // 256
    cases = {
        (256, 1, 1, 0): 1, (512, 8192, 7680, 512): 1,
        (256, lim, lim, 0): 1, (256, lim + 1, lim + 1, 0): 0,
        (512, lim, lim, 0): 0,
        (256, lim, lim - 5, 5): 1, (256, lim, lim - 5, 6): 0,
        # all tiles shared: the fix-up has a workgroup for each of them
        (256, lim, 0, 512): 1, (256, lim + 1, 0, 512): 0,
        # 129 x 2^28 outputs on 32 x 64 tiles, and on 128 x 128 of 256 threads
        (256, 5 * 2**22, 5 * 2**22, 0): 0, (256, 2**22, 2**22, 0): 1,
    }
    r = subprocess.run([exe], input="\n".join("%d %d %d %d" % c for c in cases), capture_output=True, text=True)
    assert [int(x) for x in r.stdout.split()] == list(cases.values())
