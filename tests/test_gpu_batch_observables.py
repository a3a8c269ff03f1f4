"""The observables of a batch's domains: those of the same lattice alone, bit for bit, whatever
else is in the batch, from a workspace that grows with the domains and not with their product."""
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


def _cfg(nx, ny, precision):
    return dict(nx=nx, ny=ny, eos="cs", T_over_Tc=0.8, A=-0.5, kappa=0.3, precision=precision)


# sides around a tile's 254 columns and its rows; 60 copies: rows enough to fill the GPU with tall tiles
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("copies", [1, 60])
def test_a_domains_observables_are_the_lattices(lbm, precision, copies):
    from paper_1412_7228_amd import inputs

    print(f"[gpu-case] batch observables against lattices, x{copies} {precision}", flush=True)
    sizes = [(3, 3), (64, 4), (254, 41), (255, 130), (600, 500)]
    rhos = [inputs.spinodal(x, y, 0.16, noise=1e-2, seed=i) for i, (x, y) in enumerate(sizes)]
    want = []
    for (x, y), r in zip(sizes, rhos):
        lat = lbm.Lattice(_cfg(x, y, precision))
        lat.init_field(r)
        lat.step(5)
        want.append({k: v for k, v in lat.observables(check=False).items() if k != "status"})
    b = lbm.Batch([_cfg(x, y, precision) for x, y in sizes * copies])
    for i in range(b.n):
        b.init_field(i, rhos[i % len(sizes)])
    b.step(5)
    for i, o in enumerate(b.observables()):
        w = want[i % len(sizes)]
        assert all(o[k] == w[k] or (np.isnan(o[k]) and np.isnan(w[k])) for k in w), (i, o, w)


def test_workspace_of_one_large_domain_among_many_small(lbm):
    """One 2048^2 among 3,000 of 16^2: 2 MB of records, list and partials (n times the large domain's
    partials would take 220 MB), within 64 MB with what the runtime rounds up; and the right values."""
    import torch

    print("[gpu-case] batch observables workspace, 3000 x 16^2 + 2048^2", flush=True)
    sizes = [(16, 16)] * 3000 + [(2048, 2048)]
    b = lbm.Batch([dict(nx=x, ny=y, eos="ideal", precision="fp32") for x, y in sizes])
    g = np.random.default_rng(1)
    small, large = 1.0 + 0.1 * g.random((16, 16)), 1.0 + 0.1 * g.random((2048, 2048))
    for i in range(3000):
        b.init_field(i, small)
    b.init_field(3000, large)
    b.sync()
    free = torch.cuda.mem_get_info()[0]
    obs = b.observables()
    assert free - torch.cuda.mem_get_info()[0] < 64 << 20
    for o, rho in ((obs[0], small), (obs[2999], small), (obs[3000], large)):
        assert abs(o["mass"] - rho.sum()) <= rho.size * 2.0 ** -23 * 1.1  # nine FP32 populations a cell
        assert abs(o["rho_max"] - rho.max()) <= 9 * 2.0 ** -24 * rho.max()


@pytest.mark.parametrize("precision,tx,ty", [("fp32", 120, 102), ("fp64", 78, 78)])
def test_observables_of_a_buffer_above_4gib(lbm, precision, tx, ty):
    """The reduction's variant with one buffer resource per lattice row, more tiles than
    workgroups: a lattice of 100 x 100 copies of a small one (4.4 GB) has its extremes exactly,
    and 10^4 times its sums, which a lane adds over at most 3 tiles of 40 rows and two trees of 8
    levels: 150 roundings, 3.3e-14 of the sum of magnitudes, with a factor of ten."""
    from paper_1412_7228_amd import inputs

    print(f"[gpu-case] observables of {100 * tx} x {100 * ty} {precision}", flush=True)
    rho = inputs.spinodal(tx, ty, 0.183713, noise=1e-2, seed=12)
    small = lbm.Lattice(_cfg(tx, ty, precision))
    small.init_field(rho)
    small.step(4)
    f, want = small.fields(), small.observables(check=False)
    big = lbm.Lattice(_cfg(100 * tx, 100 * ty, precision))
    big.init_field(np.tile(rho, (100, 100)))
    big.step(4)
    for got in (big.observables(check=False), big.observables(check=False, noalloc=True)):
        for k in ("rho_min", "rho_max", "max_u", "rho_out", "p_out"):
            assert got[k] == want[k], k
        assert got["n_nonfinite"] == got["n_domain"] == 0
        assert abs(got["mass"] - 1e4 * f["rho"].sum()) <= 3.3e-13 * 1e4 * f["rho"].sum()
        for k, u in (("mom_x", "ux"), ("mom_y", "uy")):
            m = f["rho"] * f[u]
            assert abs(got[k] - 1e4 * m.sum()) <= 3.3e-13 * 1e4 * np.abs(m).sum()
    big.close()
