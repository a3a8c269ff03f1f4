"""The one-pass observables against the fields they reduce, at the edges of their tiles: widths
around the 254 columns of a tile, rows that its height does not divide, more tiles than blocks."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lbm():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no HIP device visible")
    from paper_1412_7228_amd import lbm as m

    m.load_library()
    return m


def _check(o, rho, ux, uy):
    """Sums of n FP64 values in any order differ by at most n ulp of the sum of their magnitudes (n < 2^20
    here: 2.4e-10 at the very worst, about sqrt(n) ulp in practice); extremes and samples are exact."""
    ny, nx = rho.shape
    tol = rho.size * 2.0 ** -52
    assert abs(o["mass"] - rho.sum()) <= tol * np.abs(rho).sum()
    for k, v in (("mom_x", ux), ("mom_y", uy)):
        assert abs(o[k] - (rho * v).sum()) <= tol * np.abs(rho * v).sum() + 1e-300
    assert o["rho_min"] == rho.min() and o["rho_max"] == rho.max()
    assert o["rho_in"] == rho[ny // 2, nx // 2] and o["rho_out"] == rho[0, 0]
    u = np.sqrt(ux * ux + uy * uy).max()
    assert abs(o["max_u"] - u) <= 8 * 2.0 ** -52 * u
    assert o["n_nonfinite"] == 0


SIZES = [(3, 3), (64, 4), (253, 5), (254, 9), (255, 31), (508, 33), (509, 40), (1000, 300), (3, 140001), (140001, 3)]


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("nx,ny", SIZES)
def test_lattice_observables_reduce_the_fields(lbm, nx, ny, precision):
    from paper_1412_7228_amd import inputs

    print(f"[gpu-case] observables {nx}x{ny} {precision}", flush=True)
    lat = lbm.Lattice(dict(nx=nx, ny=ny, eos="cs", T_over_Tc=0.8, A=-0.5, kappa=0.3, precision=precision))
    lat.init_field(inputs.spinodal(nx, ny, 0.16, noise=1e-2, seed=3))
    lat.step(5)
    f = lat.fields()
    _check(lat.observables(check=False), f["rho"], f["ux"], f["uy"])
    _check(lat.observables(check=False, noalloc=True), f["rho"], f["ux"], f["uy"])


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("copies", [1, 40])  # 40: rows enough for the taller tiles
def test_batch_observables_reduce_each_domain(lbm, precision, copies):
    from paper_1412_7228_amd import inputs

    print(f"[gpu-case] batch observables x{copies} {precision}", flush=True)
    sizes = [s for s in SIZES if s[0] * s[1] < 10 ** 5] * copies + [(600, 900)]
    b = lbm.Batch([dict(nx=x, ny=y, eos="vdw", T_over_Tc=0.9, K=0.3, A=-0.5, kappa=0.2, precision=precision)
                   for x, y in sizes])
    for i, (x, y) in enumerate(sizes):
        b.init_field(i, inputs.spinodal(x, y, 3.6, noise=1e-2, seed=i))
    for n in (3, 4):  # either buffer
        b.step(n)
        obs = b.observables()
        for i in sorted({0, 1, 2, 3, 4, 5, 6, len(sizes) - 1}):
            _check(obs[i], *(b.field(i, k) for k in ("rho", "ux", "uy")))


@pytest.mark.parametrize("scale,u", [(1e160, 1e-2), (1e-160, 1e-2), (1.0, 1e-80), (1e-120, 1e-60)])
def test_largest_velocity_where_squares_leave_the_range(lbm, scale, u):
    """max_u of states whose squared momenta or densities overflow or underflow (the velocities do
    not), the larger velocities in the later rows of a tile; the bound of _check (8 ulp)."""
    print(f"[gpu-case] observables at densities of {scale} and velocities of {u}", flush=True)
    nx, ny = 70, 60
    g = np.random.default_rng(7)
    rho = scale * (1.0 + 0.1 * g.random((ny, nx)))
    ramp = u * np.arange(1, ny + 1)[:, None] / ny
    lat = lbm.Lattice(dict(nx=nx, ny=ny, eos="ideal", precision="fp64"))
    lat.init_field(rho, ramp * (1.0 + 0.1 * g.random((ny, nx))), -ramp * g.random((ny, nx)))
    f = lat.fields()
    want = np.hypot(f["ux"], f["uy"]).max()
    assert abs(lat.observables(check=False)["max_u"] - want) <= 8 * 2.0 ** -52 * want
