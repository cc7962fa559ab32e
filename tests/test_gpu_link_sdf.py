"""The mesh distance (lsdf_build_link_sdf, lsdf_sdf_labels) where its work
splits: meshes around one staging round (512 triangles) and several, group
remainders (8 triangles), brick remainders of the grid and grids too thin for
bricks, parts inside one another, and parts that are not closed (the solid
angle's branch).  Judged against the oracle's double-precision distance.

Tolerance: points and vertices lie within 1 m, where an FP32 coordinate
rounds by at most 2^-25 m = 3e-8 m; a closest point is a few such roundings
from the exact one and the distance one more: 2e-6 m, the bound the plain
build is held to.
"""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu
TOL = 2e-6


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2309_12543_amd import lsdf
    lsdf.load_library()
    return lsdf


def dev(a, dtype=torch.float32):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=dtype, device="cuda")


def part(kind):
    if kind == "box":
        return synth.box_mesh((0.05, -0.02, 0.03), (0.11, 0.07, 0.05))
    if kind == "tilted":            # capsule, 256 triangles: half a round
        return synth.capsule_mesh((-0.1, 0.02, 0.0), (0.13, -0.04, 0.2), 0.06)
    if kind == "round":             # 512 triangles: exactly one round
        return synth.capsule_mesh((0.0, 0.0, -0.1), (0.0, 0.0, 0.15), 0.08, nseg=32, nring=4)
    if kind == "rounds":            # 1,344 triangles: three rounds, a remainder in the last
        return synth.capsule_mesh((0.02, 0.0, -0.1), (0.0, 0.03, 0.15), 0.09, nseg=42, nring=8)
    v, t = part("tilted")
    if kind == "open":              # a triangle missing: 255, no longer closed
        return v, t[1:]
    if kind == "flipped":           # one triangle turned over: edges no longer cancel
        t = t.copy()
        t[7] = t[7][::-1]
        return v, t
    if kind == "inverted":          # closed, inside out: nothing is inside it
        return v, t[:, [0, 2, 1]]
    if kind == "unwelded":          # closed with its vertices repeated per triangle
        return v[t].reshape(-1, 3), np.arange(3 * len(t), dtype=np.int32).reshape(-1, 3)
    raise ValueError(kind)


MESHES = [("box",), ("tilted",), ("round",), ("rounds",), ("open",), ("flipped",), ("inverted",), ("unwelded",),
          ("box", "tilted"), ("rounds", "box", "open"), ("tilted", "inverted", "round")]


def mesh_of(kinds):
    m = synth.union_mesh([part(k) for k in kinds])
    m.verts = m.verts.astype(np.float32).astype(np.float64)
    return m


def signed_agree(got, ref):
    """Same distance; same sign wherever the distance exceeds the tolerance."""
    assert np.abs(np.abs(got) - np.abs(ref)).max() <= TOL, np.abs(np.abs(got) - np.abs(ref)).max()
    sure = np.abs(ref) > TOL
    assert np.array_equal(np.sign(got[sure]), np.sign(ref[sure]))


@pytest.mark.parametrize("kinds", MESHES, ids="+".join)
@pytest.mark.parametrize("n", [(17, 16, 9), (2, 3, 40)], ids=str)
def test_grid_matches_oracle(B, orc, kinds, n):
    m = mesh_of(kinds)
    lo, hi = (m.verts.min(0) - 0.05).astype(np.float32), (m.verts.max(0) + 0.05).astype(np.float32)
    print("[gpu] build_link_sdf", kinds, n, flush=True)
    gs = B.GridSet(lo[None], hi[None], np.array([n]), device="cuda")
    gs.buf.fill_(float("nan"))
    B.build_link_sdf(dev(m.verts), dev(m.tris, torch.int32), m.comp_first, gs, 0)
    got = gs.grid(0).cpu().numpy().astype(np.float64).ravel()
    ax = [lo[a].astype(np.float64) + np.arange(n[a]) * ((hi[a].astype(np.float64) - lo[a]) / (n[a] - 1)) for a in range(3)]
    z, y, x = np.meshgrid(ax[2], ax[1], ax[0], indexing="ij")
    signed_agree(got, orc.mesh_sdf(np.stack([x, y, z], -1).reshape(-1, 3), m.verts, m.tris, m.comp_first))


@pytest.mark.parametrize("kinds", MESHES, ids="+".join)
def test_labels_match_oracle(B, orc, kinds):
    """Every point outside a grid box too small to hold the mesh takes the
    exact distance, inside the parts too; N leaves a part-filled last wave."""
    m = mesh_of(kinds)
    rng = np.random.default_rng(5)
    lo, hi = m.verts.min(0) - 0.3, m.verts.max(0) + 0.3
    pts = rng.uniform(lo, hi, size=(1003, 3))
    # points level with vertices and straight above edges: the ray's ties
    pts[:300] = m.verts[rng.integers(0, len(m.verts), 300)] + rng.choice([-0.11, 0.0, 0.07], size=(300, 3))
    pts = pts.astype(np.float32)
    glo, ghi = np.full((1, 3), 9.0, np.float32), np.full((1, 3), 9.5, np.float32)
    gs = B.GridSet(glo, ghi, np.array([[4, 4, 4]]), device="cuda")
    gs.buf.zero_()
    print("[gpu] sdf_labels", kinds, flush=True)
    got = B.sdf_labels(dev(m.verts), dev(m.tris, torch.int32), m.comp_first, gs, 0, dev(pts)).cpu().numpy()
    signed_agree(got.astype(np.float64), orc.mesh_sdf(pts.astype(np.float64), m.verts, m.tris, m.comp_first))


def test_several_links_equal_one_at_a_time(B):
    """The one-launch calls of several links give each link's own bits, with
    grids of different sizes and a link without a part table."""
    from paper_2309_12543_amd import learned
    meshes = [mesh_of(k) for k in (("box",), ("rounds", "box", "open"), ("unwelded",))]
    meshes[0].comp_first = None
    lo = np.array([m.verts.min(0) - 0.05 for m in meshes], dtype=np.float32)
    hi = np.array([m.verts.max(0) + 0.05 for m in meshes], dtype=np.float32)
    n = np.array([[9, 20, 13], [16, 16, 16], [2, 3, 40]])
    gs, one = B.build_robot_grids(meshes, lo, hi, n), B.GridSet(lo, hi, n, device="cuda")
    rng = np.random.default_rng(6)
    samples = dev(rng.uniform(-0.4, 0.4, size=(3, 700, 3)))
    print("[gpu] several links", flush=True)
    labels = learned.labels_for_samples(meshes, gs, samples)
    for i, m in enumerate(meshes):
        v, t = dev(m.verts), dev(m.tris, torch.int32)
        B.build_link_sdf(v, t, m.comp_first, one, i)
        assert torch.equal(labels[i], B.sdf_labels(v, t, m.comp_first, gs, i, samples[i]))
    assert torch.equal(gs.buf, one.buf)
