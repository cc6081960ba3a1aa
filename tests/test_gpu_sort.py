"""Order of a build's particles at the sizes where the sort changes: one
particle, a block of it, the blocks up to which digit counts are added up in
place (128 of 1024 or 2048 keys) and past them, an even and an odd number of
digit passes."""
import numpy as np
import pytest

import crk_inputs as ci
from paper_2202_02840_amd import CRK_FP64, Context
from paper_2202_02840_amd import pipeline as pl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 1023, 1025, 131072, 131073, 262144, 262145])
@pytest.mark.parametrize("side", [0.3, 0.02])   # two bits an axis and six: one pass and three
def test_order(side, n):
    rng = np.random.default_rng(n)
    pos = rng.random((3, n))
    H = np.full(n, min(0.4, 0.5 * n ** (-1.0 / 3.0)))
    ps = ci.ParticleSet(*pos, H, np.full(n, 1.0 / n), np.ones(n), np.zeros((3, n)), None, L=1.0)
    ctx = Context(0)
    dev = pl.upload(ps)
    perm, pairs = ctx.build_cells(dev["x"], dev["y"], dev["z"], dev["H"], pl.params_for(ps, 64.0, CRK_FP64),
                                  cell_size=side)
    nc = ctx.n_cells
    key = np.zeros(n, dtype=np.int64)
    for axis in range(3):
        k = np.minimum(np.floor(pos[axis] * float(nc)).astype(np.int64), nc - 1)
        for b in range(8):
            key |= ((k >> b) & 1) << (3 * b + axis)
    assert np.array_equal(perm.cpu().numpy(), np.argsort(key, kind="stable"))
    off = ctx.export_neighbors(1)[0]
    assert int(off[-1]) == pairs and bool((off[1:] >= off[:-1]).all())
