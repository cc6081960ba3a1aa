"""Rows of more than one and two tiles of indices, at every number of lanes whose
tiles they outgrow (28 entries with one lane, 60, 120, 224 and 480 with sixteen),
row starts of any alignment, against the oracle."""
import numpy as np
import pytest

import crk_inputs as ci
from gpu_helpers import compare, gpu_run, oracle_run
from paper_2202_02840_amd import CRK_FP64, CRK_MIXED, Context

pytestmark = pytest.mark.gpu

N = 2003


@pytest.fixture(scope="module")
def dense():
    g = np.random.default_rng(101)
    ps = ci.ParticleSet(*g.random((3, N)), g.uniform(0.3, 0.45, N), np.full(N, 1.0 / N), np.ones(N),
                        0.01 * g.standard_normal((3, N)), None, L=1.0)
    ref = oracle_run(ps)
    rows = ref["n_pairs"] / N
    assert rows > 480
    return ps, ref


# the bars of the FP64 and the FP32 path: sums of under a thousand terms
@pytest.mark.parametrize("lanes", [1, 2, 4, 8, 16])
@pytest.mark.parametrize("prec, bar", [(CRK_FP64, 1e-12), (CRK_MIXED, 1e-5)])
def test_moments_and_gradient(dense, prec, bar, lanes):
    ps, ref = dense
    ctx = Context(0)
    ctx.set_lanes(mom=lanes, grad=lanes)
    errs = compare(gpu_run(ps, prec, ctx=ctx), ref, ("V", "m0", "m1", "m2", "gm0", "gm1", "gm2", "gradv"))
    assert max(errs.values()) <= bar, errs
