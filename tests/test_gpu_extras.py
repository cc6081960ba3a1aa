"""Pairs a particle gets from larger supports (its extras) ascend in the other
particle: rows about as long as their lane group's LDS row (128 entries, or 256
where a particle has over 32 extras in the mean), as a wavefront's LDS (1056
and 1040), and longer than two of those, and gather rows past 1024 walked
again or not."""
import numpy as np
import pytest

import crk_inputs as ci
from paper_2202_02840_amd import CRK_FP64, Context
from paper_2202_02840_amd import pipeline as pl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n, every", [(337, 8), (2770, 69), (6100, 152), (1010, 3), (4110, 3)])
def test_extras_ascend(n, every):
    rng = np.random.default_rng(n)
    pos = rng.random((3, n))
    H = np.full(n, 0.45)
    H[::every] = 0.02   # small supports inside everybody's
    ps = ci.ParticleSet(*pos, H, np.full(n, 1.0 / n), np.ones(n), np.zeros((3, n)), None, L=1.0)
    ctx = Context(0)
    dev, prm = pl.upload(ps), pl.params_for(ps, 64.0, CRK_FP64)
    for _ in range(2):   # the second build has scratch rows for the longest row
        perm, _ = ctx.build_cells(dev["x"], dev["y"], dev["z"], dev["H"], prm)
        goff, poff, pidx = (t.cpu().numpy() for t in (ctx.export_neighbors(0)[0], *ctx.export_neighbors(1)))
        p = perm.long().cpu().numpy()
        small = np.flatnonzero(H[p] < 0.1)
        for i in small[:200]:
            w = np.abs(pos[:, p] - pos[:, p[i], None])
            w = np.minimum(w, 1.0 - w)
            r2 = (w * w).sum(0)
            extras = np.flatnonzero((r2 < H[p] ** 2) & (r2 >= H[p[i]] ** 2))
            ng = goff[i + 1] - goff[i] - 1   # (exported with the particle itself)
            assert np.array_equal(pidx[poff[i] + ng:poff[i + 1]], extras), (n, i)
