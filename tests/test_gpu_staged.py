"""Derivative and compatible passes with partner records staged through LDS:
every lane mapping, on particle counts that leave a wavefront and a lane group
partly empty, against the default mapping (which the parity tests hold to the
oracle)."""
import numpy as np
import pytest
import torch

import crk_inputs as ci
from paper_2202_02840_amd import CRK_FP64, CRK_MIXED_ADAPT, Context
from paper_2202_02840_amd import pipeline as pl

pytestmark = pytest.mark.gpu


def _box(n):
    return ci.lognormal_box(10, sigma=1.0, seed=61, n_particles=n, nngb=24.0, hcap=0.3)


def _run(ps, prec, wave, lanes):
    ctx = Context(0)
    ctx.set_lanes(der=lanes)
    ctx.set_wave_mapping(deriv=wave)
    out = pl.step(ctx, pl.upload(ps), pl.params_for(ps, 64.0, prec), timestep=True, compat_dt=1e-3)
    torch.cuda.synchronize()
    return {k: out[k].cpu().numpy() for k in ("dpdt", "dudt", "vsig", "csq", "du_compat")}


# the pair terms are the same bits for every mapping: only FP64 sums of a few
# hundred terms change their order (terms up to ~1e3 times the sum)
@pytest.mark.parametrize("n", [1, 7, 65, 997])
@pytest.mark.parametrize("prec", [CRK_FP64, CRK_MIXED_ADAPT])
@pytest.mark.parametrize("wave, lanes", [(0, 1), (0, 8), (0, 64), (4, 8), (16, 8), (32, 8)])
def test_mappings_agree(prec, wave, lanes, n):
    ps = _box(n)
    ref, res = _run(ps, prec, 8, 8), _run(ps, prec, wave, lanes)
    for k in ref:
        assert np.abs(res[k] - ref[k]).max() <= 1e-10 * np.abs(ref[k]).max(), k
