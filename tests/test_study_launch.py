"""The launch shape that the studies ask the batch for (no device: the batch is a stand-in)."""
import numpy as np
import pytest

from paper_1412_7228_amd import laplace, lbm, studies


class StandIn:
    def __init__(self, cfgs):
        self.n, self.asked = len(cfgs), None
        StandIn.last = self

    def set_launch(self, mode="per_step", tile_x=0, tile_y=0, steps_per_pass=0):
        self.asked = (mode, tile_x, tile_y, steps_per_pass)

    def init_field(self, i, rho):
        pass

    def step(self, n):
        pass

    def observables(self):
        o = {k: 0.0 for k, _ in lbm.Obs._fields_}
        return [dict(o, n_nonfinite=0, n_domain=0, sigma=np.nan) for _ in range(self.n)]

    def close(self):
        pass


@pytest.mark.parametrize("spp,tile,want", [(2, None, (0, 0)), (1, None, (128, 16)), (1, (0, 0), (0, 0)), (2, (256, 8), (256, 8))])
def test_shape_of_the_studies(monkeypatch, spp, tile, want):
    monkeypatch.setattr(lbm, "Batch", StandIn)
    kw = {} if tile is None else dict(tile=tile)
    laplace.run_cases([dict(n=8, R=2, kappa=0.0, T_over_Tc=0.8, A=-0.5)], 4, steps_per_pass=spp, rhos=[None], **kw)
    assert StandIn.last.asked == ("per_step", *want, spp)
    studies._run_batch([{}], [None], 4, steps_per_pass=spp, **kw)
    assert StandIn.last.asked == ("per_step", *want, spp)
