"""Batched paths held to a kernel they do not share: graphs of the default launch (blocks, whole
domains) against single-step tiles, and the batch's own two-step tiles, asked for by shape, over
many domains of uneven size."""
import numpy as np
import pytest

from test_block_launch import MEAN, MODELS, lbm  # noqa: F401

pytestmark = pytest.mark.gpu


def _uneven(precision, n):
    g = np.random.default_rng(4)
    return [dict(MODELS["cs"], nx=int(a), ny=int(b), kappa=float(k), precision=precision)
            for a, b, k in zip(g.integers(40, 330, n), g.integers(40, 330, n), g.uniform(0, 0.8, n))]


def _fill(lbm, cfgs, shape=None):  # noqa: F811
    from paper_1412_7228_amd import inputs

    b = lbm.Batch(cfgs)
    if shape:
        b.set_launch("per_step", *shape[:2], steps_per_pass=shape[2])
    for i, c in enumerate(cfgs):
        b.init_field(i, inputs.spinodal(c["nx"], c["ny"], MEAN["cs"], noise=1e-2, seed=i))
    return b


# the default launch and the two-step tiles by name, against single-step tiles of every domain
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("shape", [None, (256, 16, 2), (128, 16, 2)])
def test_uneven_batch_replayed_graphs_equal_single_step_tiles(lbm, precision, shape):  # noqa: F811
    print(f"[gpu-case] uneven batch {shape} {precision}", flush=True)
    cfgs = _uneven(precision, 90)
    a, b = _fill(lbm, cfgs, shape), _fill(lbm, cfgs, (64, 32, 1))
    for n in (31, 31, 31, 2, 2, 2):  # replays from both buffers
        a.step(n)
        b.step(n)
    a.sync()
    b.sync()
    for i in range(0, 90, 7):
        assert np.array_equal(a.f_soa(i), b.f_soa(i), equal_nan=True), i


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_whole_domains_equal_single_step_tiles(lbm, precision):  # noqa: F811
    print(f"[gpu-case] whole domains {precision}", flush=True)
    cfgs = [dict(MODELS["cs"], nx=8 + i % 37, ny=5 + i % 41, kappa=0.01 * (i % 70), precision=precision) for i in range(300)]
    a, b = _fill(lbm, cfgs), _fill(lbm, cfgs, (64, 32, 1))
    for n in (31, 31, 31, 2, 2, 2):
        a.step(n)
        b.step(n)
    a.sync()
    b.sync()
    for i in range(0, 300, 23):
        assert np.array_equal(a.f_soa(i), b.f_soa(i), equal_nan=True), i
