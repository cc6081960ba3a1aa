"""Smoothing-length iteration at the edges of its lists and rows: particle
counts about the 1024 that a block of the compaction takes, with most rows over
the narrow cap, and supports with more candidates than a wavefront's registers
hold (1280), against the oracle."""
import numpy as np
import pytest

import crk_inputs as ci
import oracle
from paper_2202_02840_amd import CRK_FP64, Context
from paper_2202_02840_amd import pipeline as pl

pytestmark = pytest.mark.gpu


# both stop at |dH| <= 1e-7 H: they agree to about 1.5 times that
@pytest.mark.parametrize("n, nres, tune", [
    (1023, 64.0, (16, 8, 72, 1.2)), (1025, 64.0, (8, 8, 72, 1.2)), (2049, 64.0, None),
    (4096, 1200.0, None)])
def test_counts_and_rows(n, nres, tune):
    ps = ci.lognormal_box(10, sigma=0.5, seed=311, n_particles=n, nngb=min(nres, 0.4 * n), hcap=0.45)
    Href, itref, nf = oracle.hsolve(ps.x, ps.y, ps.z, ps.H, nres, tol=1e-7, max_iter=1000)
    assert nf == 0
    ctx = Context(0)
    if tune:
        ctx.set_hsolve(*tune)
    dev = pl.upload(ps)
    ctx.build_cells(dev["x"], dev["y"], dev["z"], dev["H"], pl.params_for(ps, nres, CRK_FP64))
    Hn, it, nun = ctx.hsolve(nres, ctx.permute(dev["H"], True), 1e-7, 1000)
    perm = ctx.perm.long().cpu().numpy()
    H, iters = np.empty(n), np.empty(n, dtype=np.int32)
    H[perm], iters[perm] = Hn.cpu().numpy(), it.cpu().numpy()
    assert nun == 0
    assert np.abs(H / Href - 1).max() < 1e-6
    assert np.abs(iters - itref).max() <= 1
