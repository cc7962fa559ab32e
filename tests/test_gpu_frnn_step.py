"""The grid-transformation network's training step where its tiles end: batch
sizes around the 16 rotations of a tile, output counts that are no multiple of
the 16 outputs of a wave (m odd), and parameters, moments and gradient that are
not 16-byte aligned.  Loss, gradient and Adam update against the oracle's
double precision.

No error of these inputs lies within 1e-5 of zero (they are chosen so), beyond an
FP32 output's rounding, so every sign agrees and what is left is rounding: at
most 2 * 64 + 64 products and sums of values below 4, 192 * 2^-24 * 4 = 5e-5 of
the largest gradient; for dW1 and db1, sums over up to 648 outputs, 7e-4.
"""
import numpy as np
import pytest
import torch

from frnn_util import random_rotations

pytestmark = pytest.mark.gpu
H = 32


def shifted(a, offset):
    """The array on the device, `offset` floats past a 256-byte boundary."""
    buf = torch.zeros(a.size + 4, device="cuda")
    out = buf[offset:offset + a.size]
    out.copy_(torch.as_tensor(a.astype(np.float32)))
    return out


@pytest.mark.parametrize("m, nb, offset", [(1, 1, 0), (1, 16, 3), (2, 15, 1), (3, 17, 2), (3, 33, 0), (3, 63, 1),
                                           (3, 64, 0)])
def test_step_edges(orc, m, nb, offset):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2309_12543_amd import lsdf as B
    n = orc.frnn_nparam(m)
    for seed in range(900, 920):          # the first inputs with no error near zero
        rng = np.random.default_rng(seed)
        p = rng.normal(scale=0.3, size=n).astype(np.float32).astype(np.float64)
        R = random_rotations(nb, seed).astype(np.float32).astype(np.float64)
        if np.abs(orc.frnn_forward(p, m, R) - orc.frnn_target(m, R)).min() > 1e-5:
            break
    else:
        pytest.fail("no such inputs")
    m0, v0 = rng.normal(scale=1e-3, size=n), rng.uniform(0.5e-6, 1.5e-6, size=n)
    loss64, g64 = orc.frnn_loss_grad(p, m, R)
    print("[gpu] frnn_train_step", m, nb, offset, flush=True)
    P, M, V, G = shifted(p, offset), shifted(m0, offset), shifted(v0, offset), shifted(np.zeros(n), offset)
    loss, _ = B.frnn_train_step(P, m, torch.as_tensor(R.astype(np.float32), device="cuda"), adam=(M, V), t=7, lr=1e-3,
                                grad=G)
    g = G.cpu().numpy().astype(np.float64)
    assert float(loss.item()) == pytest.approx(loss64, rel=1e-5)
    first = 10 * H                       # W1 and b1
    assert np.abs(g[:first] - g64[:first]).max() <= 7e-4 * np.abs(g64[:first]).max()
    assert np.abs(g[first:] - g64[first:]).max() <= 5e-5 * np.abs(g64[first:]).max()
    # Adam from the gradient the call returned, on the FP32 moments and decay rates it takes
    want, m1, v1 = p.copy(), m0.astype(np.float32).astype(np.float64), v0.astype(np.float32).astype(np.float64)
    orc.adam_step(want, m1, v1, g, 7, 1e-3, float(np.float32(0.9)), float(np.float32(0.999)))
    assert np.abs(P.cpu().numpy() - want).max() <= 2 ** -22 * np.abs(want).max()
    assert np.abs(M.cpu().numpy() - m1).max() <= 2 ** -22 * np.abs(m1).max()
    assert np.abs(V.cpu().numpy() - v1).max() <= 2 ** -22 * np.abs(v1).max()
    # the gradient alone: the same bits, nothing updated
    G2 = shifted(np.zeros(n), offset)
    before = shifted(p, offset)
    B.frnn_train_step(before, m, torch.as_tensor(R.astype(np.float32), device="cuda"), grad=G2)
    assert torch.equal(G2, G) and np.array_equal(before.cpu().numpy(), p.astype(np.float32))
