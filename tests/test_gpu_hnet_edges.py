"""Network kernels at their edges: features of wavefronts some of whose
particles have another H than the build's, gradients and losses of batches that
end inside a tile and of more tiles than a step of their sums takes (1024 of
the loss, 256 of the gradient)."""
import numpy as np
import pytest
import torch

import crk_inputs as ci
import oracle
from oracle import hnet
from paper_2202_02840_amd import CRK_FP64, Context
from paper_2202_02840_amd import pipeline as pl

pytestmark = pytest.mark.gpu


def _dev(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float32), device="cuda")


@pytest.mark.parametrize("n", [3, 61, 997])
@pytest.mark.parametrize("every", [1, 2, 31])
def test_features_of_mixed_supports(n, every):
    ps = ci.lognormal_box(10, sigma=1.0, seed=407, n_particles=n, nngb=40.0, hcap=0.4)
    ctx = Context(0)
    dev = pl.upload(ps)
    ctx.build_cells(dev["x"], dev["y"], dev["z"], dev["H"], pl.params_for(ps, 64.0, CRK_FP64))
    perm = ctx.perm.long().cpu().numpy()
    H = ps.H.copy()
    H[perm[::every]] *= 1.04
    got = np.empty((8, n))
    got[:, perm] = ctx.hnet_features(64.0, ctx.permute(torch.as_tensor(H, device="cuda"), True)).double().cpu().numpy()
    ref = oracle.hnet_features(ps.x, ps.y, ps.z, H, 64.0)
    # features are FP64 sums rounded to FP32
    assert np.abs(got - ref).max() <= 1e-6 * max(1.0, np.abs(ref).max())


# bars of the existing gradient test: FP32 sums of products of FP32 factors
@pytest.mark.parametrize("nb", [1, 16, 17, 16 * 257, 16 * 1025 + 3])
def test_gradient_and_loss(nb):
    g = np.random.default_rng(nb)
    f, t = g.normal(0, 1, (nb, 8)), g.normal(0, 0.3, nb)
    th = ci.hnet_init(19)
    ctx = Context(0)
    tht = _dev(th)
    m, v = torch.zeros_like(tht), torch.zeros_like(tht)
    grad, loss = ctx.hnet_train_step(tht, m, v, 1, 0.0, _dev(f.T), _dev(t), want_grad=True, want_loss=True)
    L, ref = hnet.backward(th.astype(np.float32).astype(np.float64), f.astype(np.float32).astype(np.float64),
                           t.astype(np.float32))
    assert abs(loss - L) <= 1e-5 * L
    assert np.abs(grad.double().cpu().numpy() - ref).max() <= 1e-4 * np.abs(ref).max()
