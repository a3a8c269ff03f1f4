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
