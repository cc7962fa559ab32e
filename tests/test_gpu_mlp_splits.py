"""A batch's gradient is the sum, in order and in single precision, of its
512-sample splits' gradients: rounds of tiles that do and do not divide evenly
among the workgroups, against calls of one split (which the oracle is held to
elsewhere).  The split counts are powers of two, so that 1 / B scales exactly
and the bits have to be equal."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bound", [0.06, np.inf])
@pytest.mark.parametrize("L, Bt", [(2, 1024), (5, 16384), (16, 4096)])
def test_batch_gradient_is_the_sum_of_its_splits(L, Bt, bound):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2309_12543_amd import lsdf as B
    rng = np.random.default_rng(L)
    P = torch.as_tensor(synth.mlp_init(L, 5).astype(np.float32), device="cuda")
    cen = rng.uniform(-0.1, 0.1, size=(L, 3))
    dom = B.make_domains(cen, np.full((L, 3), 1.2), np.full((L, 3), 0.1), bound)
    x = torch.as_tensor((cen[:, None] + rng.uniform(-1.1, 1.1, size=(L, Bt, 3))).astype(np.float32), device="cuda")
    y = torch.as_tensor(rng.normal(size=(L, Bt)).astype(np.float32), device="cuda")
    print("[gpu] splits", L, Bt, bound, flush=True)
    order = torch.arange(Bt, dtype=torch.int32, device="cuda").repeat(L, 1)
    loss, grad = (t.cpu() for t in B.mlp_loss_grad(P, dom, x, y, Bt, order))
    want, total = torch.zeros_like(grad), torch.zeros(L, dtype=torch.float64)
    n = Bt // 512
    for s in range(n):
        l, g = B.mlp_loss_grad(P, dom, x, y, 512, order[:, 512 * s:512 * (s + 1)].contiguous())
        want += g.cpu() / n
        total += l.cpu().double() / n
    assert torch.equal(grad, want)
    assert torch.allclose(loss.double(), total, rtol=1e-6, atol=0)
