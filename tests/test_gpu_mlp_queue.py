"""The learned query takes the network's pairs from a queue that mixes chunks
and configurations: a call of many configurations gives each one's own bits
(the calls of one configuration are held to the oracle elsewhere), at point
counts around the chunk of 256, with and without a remainder bound, and with
margins below which every or no pair may take the grid's value."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bound", [0.06, np.inf])
@pytest.mark.parametrize("M, C", [(40, 40), (255, 3), (256, 17), (257, 40), (1000, 5)])
@pytest.mark.parametrize("margin", [0.05, -np.inf, np.inf])
def test_many_configurations_equal_single_ones(tiny, M, C, bound, margin):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2309_12543_amd import lsdf as B
    gs = B.build_robot_grids(tiny.robot.links, tiny.grid_lo, tiny.grid_hi, tiny.grid_n, device="cuda")
    q = torch.as_tensor(tiny.q[:C], dtype=torch.float32, device="cuda")
    T = B.fk_batch(tiny.robot.dh, q, base_T=tiny.robot.base_T)
    pts = torch.as_tensor(tiny.points[::2][:M], dtype=torch.float32, device="cuda")
    P = torch.as_tensor(synth.mlp_init(tiny.L, 21).astype(np.float32), device="cuda")
    cen, half = synth.mlp_domain(tiny.grid_lo.astype(np.float64), tiny.grid_hi.astype(np.float64))
    doms = B.make_domains(cen, half, synth.mlp_core(tiny.grid_lo, tiny.grid_hi), bound)
    print("[gpu] query_mlp queue", M, C, bound, margin, flush=True)
    d, link, ld = B.query_min_distance_mlp(T, gs, P, doms, pts, margin=margin, link_dist=True)
    for c in range(C):
        d1, l1, ld1 = B.query_min_distance_mlp(T[c:c + 1].contiguous(), gs, P, doms, pts, margin=margin, link_dist=True)
        assert torch.equal(ld[c], ld1[0]) and torch.equal(d[c], d1[0]) and torch.equal(link[c], l1[0])
