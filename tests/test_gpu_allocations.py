"""When the library allocates and makes graphs: its calls of hipMalloc, hipHostMalloc and
hipGraphInstantiate counted (in a process of their own, through a shim in the global scope)."""
import json
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))

PRELUDE = """
import ctypes, json, os, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
sys.path.insert(0, sys.argv[2])
import numpy as np
from paper_1412_7228_amd import inputs, lbm
lbm.load_library()
out = {}
cfg = dict(eos="cs", T_over_Tc=0.8, A=-0.5, kappa=0.3)
def counted(name, f):
    before = shim.shim_mallocs(), shim.shim_pinned()
    f()
    out[name] = [shim.shim_mallocs() - before[0], shim.shim_pinned() - before[1]]
"""


def _run(tmp_path, body):
    shim = str(tmp_path / "shim.so")
    subprocess.check_call(["g++", "-O1", "-shared", "-fPIC", "-std=c++17", "-o", shim,
                           os.path.join(HERE, "protocol", "hip_alloc_shim.cpp"), "-ldl"])
    script = tmp_path / "script.py"
    script.write_text(PRELUDE + body + "\nprint('RESULT ' + json.dumps(out))\n")
    res = subprocess.run([sys.executable, "-u", str(script), shim, os.path.dirname(HERE)], capture_output=True, text=True,
                         timeout=100)
    assert res.returncode == 0, res.stdout + res.stderr
    return json.loads(next(l for l in res.stdout.splitlines() if l.startswith("RESULT "))[7:])


def test_nothing_is_allocated_after_the_state_is_set(tmp_path):
    """Steps and every read-out of an initialised lattice or batch allocate nothing (a caller may
    have taken all memory since, or forbid allocations); setting the state does."""
    print("[gpu-case] allocations after init: 100^2, 600^2, a batch", flush=True)
    r = _run(tmp_path, """
for n in (100, 600):
    lat = lbm.Lattice(dict(cfg, nx=n, ny=n))
    counted(f"init {n}", lambda: lat.init_field(inputs.spinodal(n, n, 0.16, seed=1)))
    counted(f"step {n}", lambda: (lat.step(7), lat.sync()))
    counted(f"observables {n}", lambda: lat.observables(check=False))
    counted(f"fields {n}", lambda: (lat.fields(), lat.field("f3")))
b = lbm.Batch([dict(cfg, nx=n, ny=n) for n in (64, 100)])
counted("init batch", lambda: [b.init_field(i, inputs.spinodal(n, n, 0.16, seed=1)) for i, n in enumerate((64, 100))])
counted("step batch", lambda: (b.step(7), b.sync()))
counted("observables batch", lambda: b.observables())
counted("fields batch", lambda: (b.field(0, "rho"), b.field(1, "ux")))
""")
    assert all(v == [1, 1] for k, v in r.items() if k.startswith("init")), r
    assert all(v == [0, 0] for k, v in r.items() if not k.startswith("init")), r


def test_refused_pinned_memory_falls_back_to_copies(tmp_path):
    """Where the system gives no pinned memory, every call that uses it works through device arrays and
    copies, with the same results bit for bit."""
    print("[gpu-case] refused pinned memory: a lattice, a batch, the network", flush=True)
    r = _run(tmp_path, """
def results():
    q = []
    lat = lbm.Lattice(dict(cfg, nx=60, ny=50))
    g = np.random.default_rng(0)
    lat.init_field(inputs.spinodal(60, 50, 0.16, seed=1), 1e-3 * g.random((50, 60)), 1e-3 * g.random((50, 60)))
    lat.step(9)
    q += [lat.f_soa(), lat.fields()["rho"], lat.fields()["ux"], np.array(list(lat.observables(check=False).values()))]
    b = lbm.Batch([dict(cfg, nx=n, ny=n) for n in (20, 60)])
    for i, n in enumerate((20, 60)):
        b.init_field(i, inputs.spinodal(n, n, 0.16, seed=1))
    b.step(5)
    q += [b.f_soa(1), b.field(0, "uy")] + [np.array(list(o.values())) for o in b.observables()]
    net = lbm.MLP(max_batch=64)
    net.set_params(g.normal(0, 0.1, net.nparams))
    x, t = g.normal(size=(50, 3)), g.normal(size=(50, 3))
    q += [net.forward(x), *net.backward(x, t)]
    net.set_data(x, t)
    q += [net.train(5, 1e-3), net.train(9, 1e-3), net.params()]
    return q
a = results()
shim.shim_refuse_pinned(1)
before = shim.shim_pinned()
b = results()
out["asked"] = shim.shim_pinned() - before
out["same"] = [bool(np.array_equal(x, y, equal_nan=True)) for x, y in zip(a, b)]
""")
    assert r["asked"] >= 3 and all(r["same"]) and len(r["same"]) == 14, r


def test_repeated_batch_calls_replay_their_graphs(tmp_path):
    """Equal calls make at most one graph for each buffer they start from, also where a call is an odd
    number of launches and so ends on the other buffer: blocks (several steps a launch), whole
    domains (one launch), tiles of one and two steps; and the states are those of one call."""
    print("[gpu-case] graphs of repeated batch calls", flush=True)
    r = _run(tmp_path, """
for name, sizes, launch in (("blocks", [200] * 4, None), ("whole", [20, 40], None), ("tiles", [200] * 4, (128, 16, 2)),
                            ("single", [200] * 4, (64, 16, 1))):
    for n in (1, 3, 5, 8):
        b, once = (lbm.Batch([dict(cfg, nx=s, ny=s) for s in sizes]) for _ in range(2))
        for q in (b, once):
            if launch:
                q.set_launch("per_step", launch[0], launch[1], steps_per_pass=launch[2])
            for i, s in enumerate(sizes):
                q.init_field(i, inputs.spinodal(s, s, 0.16, seed=1))
        before = shim.shim_graphs()
        for _ in range(6):
            b.step(n)
        b.sync()
        out[f"{name} {n}"] = shim.shim_graphs() - before
        once.step(6 * n)
        out[f"{name} {n} same"] = int(np.array_equal(b.f_soa(0), once.f_soa(0)))
""")
    assert all(v == 1 for k, v in r.items() if k.endswith("same")), r
    assert all(v <= 2 for k, v in r.items() if not k.endswith("same")), r
