"""What ends a call in block launches: one or two steps that large lattices and batches leave to
the marching tiles, where those are faster.

* CPU: the rules (lbm_plan.h) against measured times.
* GPU: bitwise the states of single steps, for every rest of a call, above and below the
  sizes where the route changes."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from test_block_launch import MEAN, MODELS, _same, lbm  # noqa: F401
from test_persistent_protocol import CSRC, PROTO, ROOT


def _harness(tmp_path, name):
    exe, rocm = str(tmp_path / "harness"), "/opt/rocm/include"
    if not os.path.isdir(rocm) or shutil.which("g++") is None:
        pytest.skip("no HIP headers or g++")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", rocm, "-I",
                           os.path.join(ROOT, "include"), "-I", CSRC, "-o", exe, os.path.join(PROTO, name)])
    res = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0 and "0 failures" in res.stdout, res.stdout + res.stderr


def test_lattice_rule_takes_the_faster_launch(tmp_path):
    _harness(tmp_path, "lattice_rest.cpp")


# blocks for every rest; one step by tiles (FP32); one (FP32) or both (FP64); both; idle lanes keep the blocks
@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("nx,ny", [(800, 700), (1000, 1000), (1500, 1400), (2000, 1900), (300, 5500)])
def test_lattice_calls_of_few_steps_equal_single_steps(lbm, precision, nx, ny):  # noqa: F811
    from paper_1412_7228_amd import inputs

    print(f"[gpu-case] calls of few steps {nx}x{ny} {precision}", flush=True)
    cfg = dict(MODELS["cs"], nx=nx, ny=ny, kappa=0.3, precision=precision)
    rho = inputs.spinodal(nx, ny, MEAN["cs"], noise=1e-2, seed=2)
    a, b = lbm.Lattice(cfg), lbm.Lattice(cfg)
    b.set_launch(0, 0, 1)
    for lat in (a, b):
        lat.init_field(rho)
    for n in (1, 1, 2, 3, 4, 5, 7, 8, 10, 1):
        a.step(n)
        b.step(n)
        assert _same(a, b), n
