"""The mesh distance where a mesh stops fitting one staging round, 1,024 slots of
LDS: a part of exactly as many triangles, one of 8 more (a second round of them),
parts whose triangles fit but whose slots, padded to 16 a part, do not, and one
slot run that fits to the last.  Judged against the oracle's double-precision
distance; tolerance 2e-6 m as derived in tests/test_gpu_link_sdf.py.
"""
import numpy as np
import pytest
import torch

import synth
from test_gpu_link_sdf import dev, signed_agree

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2309_12543_amd import lsdf
    lsdf.load_library()
    return lsdf


def capsule(triangles):
    nring = next(r for r in range(8, 1, -1) if triangles % (4 * r) == 0)
    v, t = synth.capsule_mesh((0.0, 0.02, -0.12), (0.03, 0.0, 0.14), 0.09, nseg=triangles // (4 * nring), nring=nring)
    assert len(t) == triangles
    return v, t


def boxes(n):
    rng = np.random.default_rng(n)
    return [synth.box_mesh(rng.uniform(-0.25, 0.25, 3), rng.uniform(0.02, 0.08, 3)) for _ in range(n)]


# triangles and slots: 1024, 1024 | 1032, 1040 | 1020, 1088 | 1008, 1024 | 2060, 2064
MESHES = {"full": [capsule(1024)], "over": [capsule(1032)], "padded": [capsule(840), *boxes(15)],
          "padded_full": [capsule(1008 - 16 * 3), *boxes(4)], "rounds": [capsule(2048), *boxes(1)]}


@pytest.mark.parametrize("name", MESHES)
def test_staging_rounds(B, orc, name):
    m = synth.union_mesh(MESHES[name])
    m.verts = m.verts.astype(np.float32).astype(np.float64)
    slots = sum(-(-n // 16) * 16 for n in np.diff(m.comp_first))
    assert (slots <= 1024) == (name in ("full", "padded_full"))
    lo, hi, n = (m.verts.min(0) - 0.05).astype(np.float32), (m.verts.max(0) + 0.05).astype(np.float32), (13, 18, 11)
    print("[gpu] build_link_sdf", name, len(m.tris), slots, flush=True)
    gs = B.GridSet(lo[None], hi[None], np.array([n]), device="cuda")
    v, t = dev(m.verts), dev(m.tris, torch.int32)
    B.build_link_sdf(v, t, m.comp_first, gs, 0)
    ax = [lo[a].astype(np.float64) + np.arange(n[a]) * ((hi[a].astype(np.float64) - lo[a]) / (n[a] - 1)) for a in range(3)]
    z, y, x = np.meshgrid(ax[2], ax[1], ax[0], indexing="ij")
    ref = orc.mesh_sdf(np.stack([x, y, z], -1).reshape(-1, 3), m.verts, m.tris, m.comp_first)
    signed_agree(gs.grid(0).cpu().numpy().astype(np.float64).ravel(), ref)
    rng = np.random.default_rng(3)
    pts = rng.uniform(m.verts.min(0) - 0.3, m.verts.max(0) + 0.3, size=(777, 3)).astype(np.float32)
    out = B.GridSet(np.full((1, 3), 9.0), np.full((1, 3), 9.5), np.array([[4, 4, 4]]), device="cuda")
    out.buf.zero_()
    got = B.sdf_labels(v, t, m.comp_first, out, 0, dev(pts)).cpu().numpy().astype(np.float64)
    signed_agree(got, orc.mesh_sdf(pts.astype(np.float64), m.verts, m.tris, m.comp_first))
