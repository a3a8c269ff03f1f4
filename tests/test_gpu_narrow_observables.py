"""The observables of narrow lattices (up to 126 columns: several tiles side by side in a workgroup)
against the fields they reduce, alone and among wide domains of a batch."""
import numpy as np
import pytest

from test_gpu_observables import _check, lbm  # noqa: F401

pytestmark = pytest.mark.gpu

# 3 columns: 51 tiles a workgroup; 126 and 127: the last narrow and the first wide width; 62 and 63: four
# tiles and three; rows that leave tiles and workgroups part empty, fewer rows than a workgroup's
SIZES = [(3, 3), (3, 203), (3, 204), (3, 9000), (4, 100003), (7, 1000), (16, 40000), (31, 29), (62, 28), (63, 4011),
         (126, 9), (126, 5003), (127, 997)]


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("nx,ny", SIZES)
def test_narrow_lattices(lbm, nx, ny, precision):  # noqa: F811
    from paper_1412_7228_amd import inputs

    print(f"[gpu-case] narrow observables {nx}x{ny} {precision}", flush=True)
    lat = lbm.Lattice(dict(nx=nx, ny=ny, eos="cs", T_over_Tc=0.8, A=-0.5, kappa=0.3, precision=precision))
    lat.init_field(inputs.spinodal(nx, ny, 0.16, noise=1e-2, seed=3))
    lat.step(5)
    f = lat.fields()
    _check(lat.observables(check=False), f["rho"], f["ux"], f["uy"])
    _check(lat.observables(check=False, noalloc=True), f["rho"], f["ux"], f["uy"])


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_narrow_and_wide_domains_of_a_batch(lbm, precision):  # noqa: F811
    from paper_1412_7228_amd import inputs

    print(f"[gpu-case] narrow and wide domains {precision}", flush=True)
    sizes = [(3, 204), (300, 70), (32, 2011), (127, 50), (126, 50), (5, 5)]
    cfgs = [dict(nx=x, ny=y, eos="vdw", T_over_Tc=0.9, K=0.3, A=-0.5, kappa=0.2, precision=precision) for x, y in sizes]
    rhos = [inputs.spinodal(x, y, 3.6, noise=1e-2, seed=i) for i, (x, y) in enumerate(sizes)]
    b = lbm.Batch(cfgs)
    for i, r in enumerate(rhos):
        b.init_field(i, r)
    b.step(3)
    for i, o in enumerate(b.observables()):
        lat = lbm.Lattice(cfgs[i])
        lat.init_field(rhos[i])
        lat.step(3)
        w = lat.observables(check=False)
        assert all(o[k] == w[k] or (np.isnan(o[k]) and np.isnan(w[k])) for k in o), (i, o, w)
        _check(o, *(b.field(i, k) for k in ("rho", "ux", "uy")))


def test_narrow_buffer_above_4gib(lbm):  # noqa: F811
    """32 x 1,900,000 FP32 (4.4 GB of state) as 19,000 copies of 32 x 100; the bound of the sums: a
    lane adds at most 40 rows, a workgroup's tree, a workgroup of the second kernel 2 partials a lane
    and its tree: under 150 roundings, with a factor of ten."""
    from paper_1412_7228_amd import inputs

    print("[gpu-case] narrow observables 32x1900000 fp32", flush=True)
    cfg = dict(eos="cs", T_over_Tc=0.8, A=-0.5, kappa=0.3, precision="fp32")
    rho = inputs.spinodal(32, 100, 0.16, noise=1e-2, seed=5)
    small = lbm.Lattice(dict(cfg, nx=32, ny=100))
    big = lbm.Lattice(dict(cfg, nx=32, ny=1900000))
    small.init_field(rho)
    big.init_field(np.tile(rho, (19000, 1)))
    for lat in (small, big):
        lat.step(3)
    f, want, got = small.fields(), small.observables(check=False), big.observables(check=False)
    big.close()
    for k in ("rho_min", "rho_max", "max_u", "rho_out"):
        assert got[k] == want[k], k
    assert abs(got["mass"] - 19000 * f["rho"].sum()) <= 3.3e-13 * 19000 * f["rho"].sum()
