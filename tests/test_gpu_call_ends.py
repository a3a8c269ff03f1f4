"""Where block launches end: the lattice sizes above which the marching tiles run, and the one or
two steps at the end of a call that large lattices and batches leave to them.

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


def test_batch_rule_takes_the_faster_launches(tmp_path):
    _harness(tmp_path, "batch_tail.cpp")


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


# the last and the first size on either side of block_max_cells: 12 * 2^20 cells in FP32, 7 * 2^20 in FP64
@pytest.mark.gpu
@pytest.mark.parametrize("precision,n", [("fp32", 3547), ("fp32", 3548), ("fp64", 2709), ("fp64", 2710)])
def test_default_launch_at_the_limit_of_blocks(lbm, precision, n):  # noqa: F811
    from paper_1412_7228_amd import inputs

    print(f"[gpu-case] default launch {n}^2 {precision}", flush=True)
    cfg = dict(MODELS["cs"], nx=n, ny=n, kappa=0.3, precision=precision)
    rho = inputs.spinodal(n, n, MEAN["cs"], noise=1e-2, seed=2)
    a, b = lbm.Lattice(cfg), lbm.Lattice(cfg)
    b.set_launch(0, 0, 1)
    for lat in (a, b):
        lat.init_field(rho)
    for steps in (3, 4, 200):  # 200: a replayed graph of three-step launches or of two-step tiles
        a.step(steps)
        b.step(steps)
        assert _same(a, b), steps


# wide domains, whose calls of few steps go to the tiles; uneven ones; narrow ones, which keep the blocks
@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("sizes", [[(1024, 1000)] * 8, [(2000, 1500), (300, 200), (64, 64)], [(70, 60)] * 900])
def test_batch_calls_of_few_steps_equal_single_steps(lbm, precision, sizes):  # noqa: F811
    from paper_1412_7228_amd import inputs

    print(f"[gpu-case] batch calls of few steps {sizes[0]} x {len(sizes)} {precision}", flush=True)
    cfgs = [dict(MODELS["cs"], nx=x, ny=y, kappa=0.1 * (i % 8), precision=precision) for i, (x, y) in enumerate(sizes)]
    b = lbm.Batch(cfgs)
    rhos = {}
    for i, s in enumerate(sizes):
        rhos.setdefault(s, inputs.spinodal(*s, MEAN["cs"], noise=1e-2, seed=3))
        b.init_field(i, rhos[s])
    calls = (1, 1, 2, 3, 4, 5, 7, 8, 10, 1)
    for n in calls:
        b.step(n)
    b.sync()
    for i in sorted({0, len(sizes) // 2, len(sizes) - 1}):
        lat = lbm.Lattice(cfgs[i])
        lat.set_launch(0, 0, 1)
        lat.init_field(rhos[sizes[i]])
        lat.step(sum(calls))
        assert np.array_equal(b.f_soa(i), lat.f_soa(), equal_nan=True), i
