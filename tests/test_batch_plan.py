"""Block plans of batches of mixed sizes and of lattices beyond the last-level cache (lbm_plan.h):
the choice of steps and shape and its search, which the cover and capacity checks of test_block_launch.py
leave open."""
import os
import shutil
import subprocess

import pytest

from test_persistent_protocol import CSRC, PROTO, ROOT


@pytest.mark.parametrize("harness", ["batch_plan", "lattice_far", "plan_search"])
def test_plans(tmp_path, harness):
    exe, rocm = str(tmp_path / "plans"), "/opt/rocm/include"
    if not os.path.isdir(rocm) or shutil.which("g++") is None:
        pytest.skip("no HIP headers or g++")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", rocm, "-I",
                           os.path.join(ROOT, "include"), "-I", CSRC, "-o", exe, os.path.join(PROTO, f"{harness}.cpp")])
    res = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0 and "0 failures" in res.stdout, res.stdout + res.stderr
