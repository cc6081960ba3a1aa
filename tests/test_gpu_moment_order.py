"""The moment sums of a row take the order that the lanes asked for give, whatever
the number of particles or the length of the rows: the corrections of a particle
with a near-singular m2 amplify the last bit of its moments, so another order
would show in them."""
import pytest
import torch

import crk_inputs as ci
from paper_2202_02840_amd import CRK_FP64, CRK_MIXED, CRK_MIXED_ADAPT, Context
from paper_2202_02840_amd import pipeline as pl

pytestmark = pytest.mark.gpu

KEYS = ("m0", "m1", "m2", "gm0", "gm1", "gm2")


def _moments(ps, prec, lanes):
    ctx = Context(0)
    ctx.set_lanes(mom=lanes)
    dev, prm = pl.upload(ps), pl.params_for(ps, 64.0, prec)
    ctx.build_cells(dev["x"], dev["y"], dev["z"], dev["H"], prm)
    return ctx.moments(prm)


# few particles, many, and rows of some 200 entries
@pytest.mark.parametrize("n_side, n, nngb", [(10, 65, 40.0), (10, 997, 60.0), (40, 64000, 64.0), (24, 13824, 200.0)])
@pytest.mark.parametrize("prec", [CRK_FP64, CRK_MIXED, CRK_MIXED_ADAPT])
def test_moments_take_the_lanes_asked_for(prec, n_side, n, nngb):
    ps = ci.lognormal_box(n_side, sigma=1.0, seed=71, n_particles=n, nngb=nngb, hcap=0.45)
    by_default, one = _moments(ps, prec, 0), _moments(ps, prec, 1)
    assert all(torch.equal(by_default[k], one[k]) for k in KEYS)   # one lane is the default
    split = {g: _moments(ps, prec, g) for g in (4, 16)}
    for a, b in ((one, split[4]), (one, split[16]), (split[4], split[16])):
        assert not all(torch.equal(a[k], b[k]) for k in KEYS)
