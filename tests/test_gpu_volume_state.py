"""Whose volumes a moment call uses: those of the current lists in the precision
asked for, after a call in another precision and after a replay that follows a
build of another box."""
import pytest
import torch

import crk_inputs as ci
from paper_2202_02840_amd import CRK_FP64, CRK_MIXED, CRK_MIXED_ADAPT, Context
from paper_2202_02840_amd import pipeline as pl

pytestmark = pytest.mark.gpu

KEYS = ("nsum", "V", "m0", "m1", "m2", "gm0", "gm1", "gm2")


def _built(ps, prec, balanced=0):
    ctx = Context(0)
    ctx.set_wave_mapping(mom=balanced)
    dev = pl.upload(ps)
    ctx.build_cells(dev["x"], dev["y"], dev["z"], dev["H"], pl.params_for(ps, 64.0, prec))
    return ctx, dev


def _same(a, b, keys=KEYS):
    for k in keys:
        assert torch.equal(a[k], b[k]), k


@pytest.mark.parametrize("prec", [CRK_FP64, CRK_MIXED_ADAPT])
@pytest.mark.parametrize("balanced", [0, 8])
def test_moments_after_another_precision(prec, balanced):
    ps = ci.lognormal_box(10, sigma=1.0, seed=81)
    prm, other = pl.params_for(ps, 64.0, prec), pl.params_for(ps, 64.0, CRK_MIXED)
    ref = _built(ps, prec, balanced)[0].moments(prm)
    ctx, _ = _built(ps, prec, balanced)
    mixed = ctx.moments(other)
    _same(ctx.moments(prm), ref)
    _same(ctx.moments(prm), ref)
    _same(ctx.moments(other), mixed)
    _same(ctx.moments(prm, want_moments=False), ref, ("nsum", "V"))


@pytest.mark.parametrize("recorded, between", [(CRK_MIXED, CRK_FP64), (CRK_FP64, CRK_MIXED), (CRK_FP64, CRK_FP64)])
def test_moments_after_a_replay(recorded, between):
    ps, small = ci.lognormal_box(12, sigma=1.0, seed=82), ci.lattice_box(6, seed=83)
    ctx = Context(0)
    dev = pl.upload(ps)
    io = ctx.step_buffers(dev)
    ctx.graph_capture(io, pl.params_for(ps, 64.0, recorded))
    d = pl.upload(small)
    ctx.build_cells(d["x"], d["y"], d["z"], d["H"], pl.params_for(small, 64.0, between))
    ctx.graph_replay()
    assert ctx.n == ps.n
    prm = pl.params_for(ps, 64.0, CRK_FP64)
    _same(ctx.moments(prm), _built(ps, recorded)[0].moments(prm))
