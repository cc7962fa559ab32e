"""The largest link grid the library takes, 2^31 nodes, in the shape that 4 x 4 x
4 bricks of nodes pad the most: every node is written, and holds the distance.

Tolerance: 2e-6 m for points within 1 m, as in tests/test_gpu_link_sdf.py, and
the rounding into binary16 storage, 2^-11 of the value.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_thin_grid_of_2_31_nodes(orc):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2309_12543_amd import lsdf as B
    n = np.array([2, 1024, 1 << 20])
    lo, hi = np.full(3, -0.5, dtype=np.float32), np.full(3, 0.5, dtype=np.float32)
    verts = np.array([[-0.2, -0.1, -0.3], [0.3, 0.1, 0.0], [-0.1, 0.2, 0.25]], dtype=np.float32)
    tris = np.array([[0, 1, 2]], dtype=np.int32)
    gs = B.GridSet(lo[None], hi[None], n[None], device="cuda", dtype=torch.float16)
    gs.buf.fill_(float("nan"))
    print("[gpu] build_link_sdf", n, flush=True)
    B.build_link_sdf(torch.as_tensor(verts, device="cuda"), torch.as_tensor(tris, device="cuda"), None, gs, 0)
    # (NaN fails the comparison; in pieces, 2^31 flags at once are not wanted)
    assert all(bool((part == part).all()) for part in gs.buf.split(1 << 28))
    rng = np.random.default_rng(1)
    k = np.stack([rng.integers(0, m, 4000) for m in n], 1)
    k[:8] = [[x, y, z] for x in (0, 1) for y in (0, n[1] - 1) for z in (0, n[2] - 1)]
    flat = torch.as_tensor((k[:, 2] * n[1] + k[:, 1]) * n[0] + k[:, 0], device="cuda")
    got = gs.buf[flat].double().cpu().numpy()
    ref = orc.mesh_sdf(lo + k / (n - 1.0), verts.astype(np.float64), tris, np.array([0, 1], dtype=np.int32))
    assert (np.abs(np.abs(got) - np.abs(ref)) <= 2e-6 + 2.0 ** -11 * np.abs(ref)).all()
