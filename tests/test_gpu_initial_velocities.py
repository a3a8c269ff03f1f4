"""Initial states with velocities, at the sizes where the fields' way to the device changes: all three
through pinned memory, the density alone, none; and domains of a batch that share one stage."""
import numpy as np
import pytest

from test_gpu_observables import lbm  # noqa: F401
from test_oracle_units import EX, EY, W

pytestmark = pytest.mark.gpu


def _initial(nx, ny, seed):
    g = np.random.default_rng(seed)
    return 0.1 + 0.2 * g.random((ny, nx)), 0.1 * g.random((ny, nx)) - 0.05, 0.1 * g.random((ny, nx)) - 0.05


def _check(f, rho, ux, uy):
    """The equilibrium of second order; about 20 roundings in FP64 of terms up to 2.5 rho w, times ten."""
    eu = EX[:, None, None] * ux + EY[:, None, None] * uy
    want = W[:, None, None] * rho * (1 + 3 * eu + 4.5 * eu**2 - 1.5 * (ux**2 + uy**2))
    assert np.abs(f - want).max() <= 200 * 2.0**-53 * 2.5 * 0.3 * W.max()


@pytest.mark.parametrize("nx,ny", [(3, 5), (128, 128), (129, 128), (222, 221), (222, 222), (512, 512), (513, 512)])
def test_lattice(lbm, nx, ny):  # noqa: F811
    print(f"[gpu-case] initial velocities {nx}x{ny}", flush=True)
    lat = lbm.Lattice(dict(nx=nx, ny=ny, eos="cs", T_over_Tc=0.8, A=-0.5, precision="fp64"))
    for seed in (1, 2):  # a fresh stage, a used one
        s = _initial(nx, ny, seed)
        lat.init_field(*s)
        _check(lat.f_soa().reshape(9, ny, nx), *s)
        lat.init_field(s[0], None, s[2])
        _check(lat.f_soa().reshape(9, ny, nx), s[0], 0 * s[1], s[2])


@pytest.mark.parametrize("largest", [(100, 150), (100, 170), (250, 200), (512, 513)])
def test_batch(lbm, largest):  # noqa: F811
    print(f"[gpu-case] initial velocities of a batch, largest domain {largest}", flush=True)
    sizes = [(10, 10), (100, 149), (60, 90), largest]
    b = lbm.Batch([dict(nx=x, ny=y, eos="cs", T_over_Tc=0.8, A=-0.5, precision="fp64") for x, y in sizes])
    states = [_initial(x, y, i) for i, (x, y) in enumerate(sizes)]
    for i, s in enumerate(states):
        b.init_field(i, *s)
    for i, (x, y) in enumerate(sizes):
        _check(b.f_soa(i).reshape(9, y, x), *states[i])
