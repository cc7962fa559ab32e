"""The grid-transformation network's training step where the step kernel takes
it (from 576 blocks of 128 outputs on, from 704 with more than 16 rotations):
output counts that are no multiple of a unit's 16 or a block's 128 (m odd), batch
sizes around the tiles of 16 rotations, parameters, moments and gradient that
are not 16-byte aligned, and more blocks than waves (m = 23: 2,282 blocks on
2,048 waves, so that some waves take a second one).  Loss, gradient and Adam
update against the oracle's double precision.

Output biases of +-8 beside products below 7 keep every error away from zero, so
that every sign agrees.  What is left is rounding, at most one unit of 2^-24 per
operation of a chain times the sum of the magnitudes.  W1 and b1: 128 sums in a
block, a 64th of the blocks in a slice, 64 slices, 64 rotations and 20 in the
hidden layer.  W2: 64 + 20; b2: 64.  The loss, a sum of positive terms: 4 of each
of 4 tiles in 8 units of at most 2 blocks, 6 in a wave, 4 in a workgroup, 8 and
6 over the 512 workgroups, and 33 in an output.
"""
import numpy as np
import pytest
import torch

from frnn_util import random_rotations
from test_gpu_frnn_step import shifted

pytestmark = pytest.mark.gpu
H = 32


@pytest.mark.parametrize("m, nb, offset", [(15, 1, 1), (15, 15, 2), (15, 16, 3), (17, 1, 3), (17, 16, 0), (17, 17, 1),
                                           (17, 33, 2), (17, 63, 3), (17, 64, 1), (23, 2, 0), (23, 16, 3), (23, 33, 2)])
def test_step_kernel(orc, m, nb, offset):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2309_12543_amd import lsdf as B
    n, no = orc.frnn_nparam(m), 24 * m ** 3
    rng = np.random.default_rng(m * 100 + nb)
    p = rng.normal(scale=0.05, size=n)
    p[:10 * H] *= 6
    p[-no:] = rng.choice([-8.0, 8.0], size=no)
    p = p.astype(np.float32).astype(np.float64)
    R = random_rotations(nb, m).astype(np.float32).astype(np.float64)
    assert np.abs(orc.frnn_forward(p, m, R) - orc.frnn_target(m, R)).min() > 0.1
    m0, v0 = rng.normal(scale=1e-3, size=n), rng.uniform(0.5e-6, 1.5e-6, size=n)
    loss64, g64 = orc.frnn_loss_grad(p, m, R)
    print("[gpu] frnn_train_step", m, nb, offset, flush=True)
    P, M, V, G = shifted(p, offset), shifted(m0, offset), shifted(v0, offset), shifted(np.zeros(n), offset)
    Rd = torch.as_tensor(R.astype(np.float32), device="cuda")
    loss, _ = B.frnn_train_step(P, m, Rd, adam=(M, V), t=7, lr=1e-3, grad=G)
    g = G.cpu().numpy().astype(np.float64)
    eps, blocks = 2.0 ** -24, -(-no // 128)
    hidden = np.abs(p[:9 * H]).reshape(H, 9).sum(1).max() + np.abs(p[9 * H:10 * H]).max()
    w2 = np.abs(p[10 * H:-no]).reshape(no, H).mean(0).max()
    assert float(loss.item()) == pytest.approx(loss64, rel=(256 + 6 + 4 + 8 + 6 + 33) * eps)
    assert np.abs(g[:10 * H] - g64[:10 * H]).max() <= (128 + -(-blocks // 64) + 64 + 64 + 20) * eps * w2
    assert np.abs(g[10 * H:-no] - g64[10 * H:-no]).max() <= 84 * eps * hidden / no
    assert np.abs(g[-no:] - g64[-no:]).max() <= 64 * eps / no
    # Adam from the gradient the call returned, on the FP32 moments and decay rates it takes
    want, m1, v1 = p.copy(), m0.astype(np.float32).astype(np.float64), v0.astype(np.float32).astype(np.float64)
    orc.adam_step(want, m1, v1, g, 7, 1e-3, float(np.float32(0.9)), float(np.float32(0.999)))
    assert np.abs(P.cpu().numpy() - want).max() <= 2 ** -22 * np.abs(want).max()
    assert np.abs(M.cpu().numpy() - m1).max() <= 2 ** -22 * np.abs(m1).max()
    assert np.abs(V.cpu().numpy() - v1).max() <= 2 ** -22 * np.abs(v1).max()
    # the gradient alone: the same bits, nothing updated
    G2, before = shifted(np.zeros(n), offset), shifted(p, offset)
    B.frnn_train_step(before, m, Rd, grad=G2)
    assert torch.equal(G2, G) and np.array_equal(before.cpu().numpy(), p.astype(np.float32))
