"""A step of two launches whose second one fails (CPU: the driver in
tests/c_abi/launch_failure.c stands in for the HIP runtime's launch calls)."""
import os
import shutil
import subprocess

import pytest

from paper_2508_01744_amd import _build

HERE = os.path.dirname(os.path.abspath(__file__))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.mark.skipif(shutil.which("gcc") is None, reason="gcc not found")
def test_failed_launch_folds_no_reward_twice(tmp_path):
    assert os.path.exists(_build.LIB), "run __graft_entry__.build()"
    exe = str(tmp_path / "launch_failure")
    subprocess.run(["gcc", "-std=c11", "-O1", "-Wall", "-rdynamic", "-D__HIP_PLATFORM_AMD__", "-I", _build.INCLUDE,
                    "-I", os.path.join(ROCM, "include"), os.path.join(HERE, "c_abi", "launch_failure.c"), _build.LIB,
                    "-L", os.path.join(ROCM, "lib"), "-lamdhip64", "-Wl,-rpath," + os.path.dirname(_build.LIB),
                    "-Wl,-rpath," + os.path.join(ROCM, "lib"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "0 failures" in r.stdout, r.stdout[-4000:] + r.stderr[-2000:]
