"""Every launch plan that hieravg_set_batch can select against the buffers
that create sizes, on the host (a plan that does not fit would write past
them on the GPU): builds tests/plan_host_check.cpp, which includes the plans'
source, against the library and runs it."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_batch_plan_fits_the_buffers(tmp_path):
    from paper_1903_05133_amd import build
    if not shutil.which(build.hipcc()):
        pytest.skip("hipcc not found")
    if not os.path.exists(build.LIB):
        build.build()
    exe = str(tmp_path / "plan_host_check")
    # the plans' translation unit; the launchers come from the built library
    cmd = [build.hipcc(), "--offload-arch=gfx950", "-O1", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"), "-I", build.CSRC, "-x", "hip",
           os.path.join(ROOT, "tests", "plan_host_check.cpp"), "-x", "none", build.LIB,
           "-Wl,-rpath," + os.path.dirname(build.LIB), "-o", exe]
    res = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert res.returncode == 0, res.stderr[-4000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    print(run.stdout)
    assert run.returncode == 0 and "plan checks ok" in run.stdout, run.stdout + run.stderr[-2000:]
