"""The grid-transformation network's training step on both sides of the output
count from which another kernel takes it (65,536): 52,728 and 65,856 outputs
(m = 13, 14), and the edges of the larger one's tiles of 16 rotations.  Loss,
gradient and Adam update against the oracle's double precision.

Output biases of +-8 beside products below 7 keep every error away from zero, so
that every sign agrees.  What is left is rounding, at most one unit of 2^-24 per
operation of a chain times the sum of the magnitudes: 128 + 9 + 64 sums over the
outputs and 64 + 20 over the rotations and in the hidden layer for W1 and b1;
64 + 20 for W2; 64 for b2.
"""
import numpy as np
import pytest
import torch

from frnn_util import random_rotations

pytestmark = pytest.mark.gpu
H = 32


@pytest.mark.parametrize("m, nb", [(13, 1), (13, 33), (13, 64), (14, 1), (14, 15), (14, 16), (14, 17), (14, 33),
                                   (14, 64), (15, 63)])
def test_step_sizes(orc, m, nb):
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
    print("[gpu] frnn_train_step", m, nb, flush=True)
    dev = lambda a: torch.as_tensor(a.astype(np.float32), device="cuda")
    P, M, V, G = dev(p), dev(m0), dev(v0), dev(np.zeros(n))
    loss, _ = B.frnn_train_step(P, m, dev(R), adam=(M, V), t=7, lr=1e-3, grad=G)
    g = G.cpu().numpy().astype(np.float64)
    eps = 2.0 ** -24
    hidden = np.abs(p[:9 * H]).reshape(H, 9).sum(1).max() + np.abs(p[9 * H:10 * H]).max()
    w2 = np.abs(p[10 * H:-no]).reshape(no, H).mean(0).max()
    assert float(loss.item()) == pytest.approx(loss64, rel=1e-5)
    assert np.abs(g[:10 * H] - g64[:10 * H]).max() <= 285 * eps * w2
    assert np.abs(g[10 * H:-no] - g64[10 * H:-no]).max() <= 84 * eps * hidden / no
    assert np.abs(g[-no:] - g64[-no:]).max() <= 64 * eps / no
    # Adam from the gradient the call returned, on the FP32 moments and decay rates it takes
    want, m1, v1 = p.copy(), m0.astype(np.float32).astype(np.float64), v0.astype(np.float32).astype(np.float64)
    orc.adam_step(want, m1, v1, g, 7, 1e-3, float(np.float32(0.9)), float(np.float32(0.999)))
    assert np.abs(P.cpu().numpy() - want).max() <= 2 ** -22 * np.abs(want).max()
    assert np.abs(M.cpu().numpy() - m1).max() <= 2 ** -22 * np.abs(m1).max()
    assert np.abs(V.cpu().numpy() - v1).max() <= 2 ** -22 * np.abs(v1).max()
    # the gradient alone: the same bits, nothing updated
    G2, before = dev(np.zeros(n)), dev(p)
    B.frnn_train_step(before, m, dev(R), grad=G2)
    assert torch.equal(G2, G) and np.array_equal(before.cpu().numpy(), p.astype(np.float32))
