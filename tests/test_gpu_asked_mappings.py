"""Lane mappings: what is asked for is what runs, also on few particles, and what
is not asked for does not follow the lists, so that a recorded step sums like an
eager one whatever its supports have grown to."""
import itertools

import pytest
import torch

import crk_inputs as ci
from paper_2202_02840_amd import CRK_FP64, CRK_MIXED_ADAPT, Context
from paper_2202_02840_amd import pipeline as pl

pytestmark = pytest.mark.gpu


def _run(setup, prec=CRK_FP64, **over):
    ps = ci.lognormal_box(10, sigma=1.0, seed=91, n_particles=997, nngb=60.0, hcap=0.45)
    ctx = Context(0)
    setup(ctx)
    return pl.step(ctx, pl.upload(ps), pl.params_for(ps, 64.0, prec, **over), compat_dt=1e-3)


# FP64 sums of some 60 terms in another order differ in some last bit of some particle
def _all_differ(outs, keys):
    for a, b in itertools.combinations(outs, 2):
        for k in keys:
            assert not torch.equal(a[k], b[k]), k


def test_gradient_lanes():
    _all_differ([_run(lambda c: c.set_lanes(grad=g)) for g in (1, 2, 4, 8, 16, 32)], ("gradv",))


def test_derivative_mappings():
    outs = [_run(lambda c: c.set_wave_mapping(deriv=w)) for w in (4, 8, 16, 32)]
    _all_differ(outs, ("dpdt", "dudt", "du_compat"))

    def lanes(g):
        def setup(c):
            c.set_wave_mapping(deriv=0)
            c.set_lanes(der=g)
        return setup
    _all_differ(outs + [_run(lanes(g)) for g in (1, 4, 64)], ("dpdt", "dudt"))


def test_lanes_of_the_fp64_rows():
    rows = [_run(lambda c: c.set_lanes(grad=g, der=g), CRK_MIXED_ADAPT, kappa_max=0.0) for g in (1, 4, 8, 64)]
    _all_differ(rows, ("gradv", "dpdt", "dudt", "du_compat"))


def test_recorded_step_sums_like_an_eager_one():
    # supports 1.4 times larger: 64 neighbours become 176
    ps = ci.lattice_box(41, seed=92)
    prm, dev = pl.params_for(ps, 64.0, CRK_FP64), pl.upload(ps)
    cell = 0.5 * float(ps.H[0])
    ctx, eager = Context(0), Context(0)
    io, ref = ctx.step_buffers(dev), eager.step_buffers(dev)
    ctx.graph_capture(io, prm, cell_size=cell, headroom=3.0)
    dev["H"].mul_(1.4)
    eager.step(ref, prm, cell_size=cell)
    ctx.graph_replay()
    for k in ("perm", "V", "m2", "B", "gB", "gradv", "dpdt", "dudt"):
        assert torch.equal(io[k], ref[k]), k


# particles a wavefront of the derivative pass: 8 from 2^14 particles on, 4 if their
# rows are long
@pytest.mark.parametrize("nres, wave", [(64.0, 8), (128.0, 8), (160.0, 8), (268.0, 4)])
def test_own_choice_of_the_derivative_pass(nres, wave):
    ps = ci.lognormal_box(26, sigma=1.0, seed=93, nngb=nres, hcap=0.45)
    prm, dev = pl.params_for(ps, nres, CRK_FP64), pl.upload(ps)
    own, asked = Context(0), Context(0)
    asked.set_wave_mapping(deriv=wave)
    a, b = pl.step(own, dev, prm, compat_dt=1e-3), pl.step(asked, dev, prm, compat_dt=1e-3)
    for k in ("dpdt", "dudt", "du_compat"):
        assert torch.equal(a[k], b[k]), k


# lanes of the FP64 rows: by n and the neighbours
@pytest.mark.parametrize("side, nres, lanes", [(10, 64.0, 32), (10, 24.0, 16), (41, 24.0, 8), (64, 64.0, 16)])
def test_own_choice_of_the_fp64_rows(side, nres, lanes):
    ps = ci.lognormal_box(side, sigma=1.0, seed=94, nngb=nres, hcap=0.45)
    prm, dev = pl.params_for(ps, nres, CRK_MIXED_ADAPT, kappa_max=0.0), pl.upload(ps)
    own, asked = Context(0), Context(0)
    asked.set_lanes(der=lanes)
    a, b = pl.step(own, dev, prm, compat_dt=1e-3), pl.step(asked, dev, prm, compat_dt=1e-3)
    for k in ("dpdt", "dudt", "du_compat"):
        assert torch.equal(a[k], b[k]), k
