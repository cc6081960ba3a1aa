"""Moment pass and velocity gradient with their index rows tiled through LDS:
every number of lanes a row, on particle counts that leave the last wavefront
partly empty, with rows of about 60 neighbours (more than one tile with one
and two lanes, less than one with more)."""
import pytest

import crk_inputs as ci
from gpu_helpers import compare, gpu_run, normwise, oracle_run
from paper_2202_02840_amd import CRK_FP64, CRK_MIXED, Context

pytestmark = pytest.mark.gpu

MOMENTS = ("m0", "m1", "m2", "gm0", "gm1", "gm2")


def _box(n):
    return ci.lognormal_box(10, sigma=1.0, seed=67, n_particles=n, nngb=60.0, hcap=0.45)


def _run(ps, prec, mom, grad):
    ctx = Context(0)
    ctx.set_lanes(mom=mom, grad=grad)
    return gpu_run(ps, prec, ctx=ctx)


# sums of a few hundred terms: the bars of the FP64 and the FP32 path
@pytest.mark.parametrize("n", [1, 65, 997])
@pytest.mark.parametrize("lanes", [1, 2, 4, 8, 16, 32, 64])
@pytest.mark.parametrize("prec, bar", [(CRK_FP64, 1e-12), (CRK_MIXED, 1e-5)])
def test_moments_of_every_row_split(prec, bar, lanes, n):
    ps = _box(n)
    errs = compare(_run(ps, prec, lanes, 8), oracle_run(ps), MOMENTS)
    assert max(errs.values()) <= bar, errs


# the pair terms are the same bits for every split: only FP64 sums of a few
# hundred terms change their order (terms up to ~1e3 times the sum)
@pytest.mark.parametrize("n", [1, 65, 997])
@pytest.mark.parametrize("lanes", [1, 2, 4, 16, 32, 64])
@pytest.mark.parametrize("prec", [CRK_FP64, CRK_MIXED])
def test_velocity_gradient_of_every_row_split(prec, lanes, n):
    ps = _box(n)
    assert normwise(_run(ps, prec, 4, lanes)["gradv"], _run(ps, prec, 4, 8)["gradv"]) <= 1e-10
