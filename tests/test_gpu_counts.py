"""The singular count of the corrections after every order of calls: the moment
pass clears it by the way, so a second call after one moment pass, or one after
another build or a mapping without that pass, has to clear it itself."""
import numpy as np
import pytest

import crk_inputs as ci
from paper_2202_02840_amd import CRK_FP64, CRK_MIXED_ADAPT, Context
from paper_2202_02840_amd import pipeline as pl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [CRK_FP64, CRK_MIXED_ADAPT])
@pytest.mark.parametrize("balanced", [0, 8])   # the other moment kernel does not clear
def test_singular_count(prec, balanced):
    # 60 particles with neighbours, 40 whose support holds nobody
    rng = np.random.default_rng(5)
    pos = np.concatenate([0.2 + 0.1 * rng.random((3, 60)), rng.random((3, 40))], axis=1)
    H = np.concatenate([np.full(60, 0.2), np.full(40, 1e-4)])
    ps = ci.ParticleSet(*pos, H, np.full(100, 0.01), np.ones(100), np.zeros((3, 100)), None, L=1.0)
    ctx = Context(0)
    ctx.set_wave_mapping(mom=balanced)
    dev, prm = pl.upload(ps), pl.params_for(ps, 64.0, prec)

    def build():
        ctx.build_cells(dev["x"], dev["y"], dev["z"], dev["H"], prm)

    build()
    mom = ctx.moments(prm)
    first = ctx.corrections(mom)["n_singular"]
    assert first >= 40
    assert ctx.corrections(mom)["n_singular"] == first
    ctx.moments(prm)
    ctx.moments(prm)
    assert ctx.corrections(mom)["n_singular"] == first
    ctx.moments(prm)
    build()
    assert ctx.corrections(mom)["n_singular"] == first
