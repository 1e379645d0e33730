"""Device allocations that fail during the hierarchy setup (no GPU: the HIP runtime and the kernels are host
stand-ins, tests/setup_alloc_driver.cpp).  A failed setup gives back what it had allocated; without room for
the inverse of the coarsest factor the setup succeeds with the factor alone."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2501_17656_amd", "csrc")


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc (host compilation only)")
def test_failed_allocations_of_the_setup(tmp_path):
    objs = []
    for src in (os.path.join(ROOT, "tests", "setup_alloc_driver.cpp"), os.path.join(CSRC, "h2_build.cpp"),
                os.path.join(CSRC, "plan.cpp")):
        objs.append(str(tmp_path / (os.path.basename(src) + ".o")))
        res = subprocess.run(["hipcc", "-std=c++17", "-O1", "-fPIC", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-c",
                              src, "-o", objs[-1]], capture_output=True, text=True, timeout=300)
        assert res.returncode == 0, res.stderr[-4000:]
    exe = str(tmp_path / "setup_alloc_driver")
    res = subprocess.run(["g++", *objs, "-o", exe], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr[-4000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0 and "all checks passed" in run.stdout, (run.stdout + run.stderr)[-4000:]
