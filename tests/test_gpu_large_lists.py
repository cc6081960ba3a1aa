"""Lists of more than 2048 blocks of 1024 rows (the support iteration's running
particles, the rows with an FP64 partner), whose counts are scanned: nine copies of
a box as a batch give each copy what the box gives alone."""
import numpy as np
import pytest
import torch

import crk_inputs as ci
from paper_2202_02840_amd import CRK_FP64, CRK_MIXED_ADAPT, Context
from paper_2202_02840_amd import pipeline as pl

pytestmark = pytest.mark.gpu

COPIES, SIDE = 9, 64
CELL = 1.0 / 32.0   # for both, so that they are sorted and walked alike


@pytest.fixture(scope="module")
def boxes():
    ps = ci.lognormal_box(SIDE, sigma=1.5, seed=97)
    both, off = pl.concat([ps] * COPIES)
    assert both.n > 2048 * 1024 and ps.n % 64 == 0
    return ps, both, off


def _same(one, many, n):
    for b in range(COPIES):
        assert torch.equal(many[..., b * n:(b + 1) * n], one)


def test_rows_with_fp64_partners(boxes):
    ps, both, off = boxes
    outs = []
    for box, offsets in ((ps, None), (both, off)):
        ctx = Context(0)
        ctx.set_lanes(vol=4, mom=1, grad=8, der=16)
        ctx.set_wave_mapping(deriv=8)
        prm = pl.params_for(box, 64.0, CRK_MIXED_ADAPT)
        outs.append(pl.step(ctx, pl.upload(box), prm, CELL, box_offsets=offsets))
        rows = ctx.adaptive_rows()
        assert 0 < rows[0] <= rows[1] < box.n
        outs[-1]["rows"] = rows
        ctx.close()
    one, many = outs
    assert many["rows"] == tuple(COPIES * r for r in one["rows"])
    for k in ("gradv", "dpdt", "dudt"):
        _same(one[k], many[k], ps.n)


def test_support_iteration(boxes):
    ps, both, off = boxes
    outs = []
    for box, offsets in ((ps, [0, ps.n]), (both, off)):
        ctx = Context(0)
        dev = pl.upload(box)
        ctx.build_cells_batch(offsets, dev["x"], dev["y"], dev["z"], dev["H"], pl.params_for(box, 64.0, CRK_FP64),
                              CELL)
        H, iters, unconverged = ctx.hsolve(64.0, ctx.permute(dev["H"], True), 1e-7, 200)
        outs.append((H, iters, unconverged))
        ctx.close()
    (H1, it1, un1), (H, it, un) = outs
    assert un == COPIES * un1
    _same(H1, H, ps.n)
    _same(it1, it, ps.n)
