"""Signs of the mesh distance (lsdf_sdf_labels, lsdf_build_link_sdf) at points
in the plane of a vertical face that is not axis-aligned, beside the face: the
ray that decides the sign runs in that plane, and the face's shadow is a
sliver as wide as the vertices' rounding.  Closed prisms lying on their sides,
with the oracle's solid angles in double precision as the judge.

Tolerance: that of tests/test_gpu_link_sdf.py, 2e-6 m for points within 1 m.
"""
import numpy as np
import pytest
import torch

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


def outline(kind):
    if kind == "wedge":
        return np.array([[-0.2, -0.1], [0.2, -0.1], [0.05, 0.15]])
    a = 2 * np.pi * np.arange(24) / 24
    return 0.1 * np.stack([np.cos(a), np.sin(a)], 1)


def prism(kind, direction, length=0.3):
    """An outline (across, up) swept along a horizontal direction: closed, its
    two ends vertical.  Vertices as the GPU holds them."""
    poly = outline(kind)
    d = np.array([*direction, 0.0]) / np.hypot(*direction)
    ring = poly[:, :1] * np.array([-d[1], d[0], 0.0]) + poly[:, 1:] * np.array([0.0, 0.0, 1.0])
    verts = np.concatenate([ring - 0.5 * length * d, ring + 0.5 * length * d]).astype(np.float32)
    n = len(poly)
    i, k = np.arange(1, n - 1), np.arange(n)
    j = (k + 1) % n
    tris = [np.stack([0 * i, i + 1, i], 1), np.stack([n + 0 * i, n + i, n + i + 1], 1),
            np.stack([k, j, n + j], 1), np.stack([k, n + j, n + k], 1)]
    return verts, np.concatenate(tris).astype(np.int32), np.array([0, 4 * n - 4], dtype=np.int32)


def signed_agree(got, ref):
    assert np.abs(np.abs(got) - np.abs(ref)).max() <= TOL, np.abs(np.abs(got) - np.abs(ref)).max()
    sure = np.abs(ref) > TOL
    wrong = sure & (np.sign(got) != np.sign(ref))
    assert not wrong.any(), (int(wrong.sum()), float(np.abs(ref[wrong]).max()))


@pytest.mark.parametrize("direction", [(0.6, 0.8), (0.8, 0.6), (1.0, 1.0), (5.0, 12.0), (12.0, -5.0)], ids=str)
@pytest.mark.parametrize("kind", ["wedge", "cylinder"])
def test_labels_in_the_plane_of_a_vertical_face(B, orc, kind, direction):
    verts, tris, first = prism(kind, direction)
    n, v = len(verts) // 2, verts.astype(np.float64)
    rng = np.random.default_rng(5)
    s, t = rng.uniform(-1.0, 2.0, size=(2, 20000, 1))
    pts = (v[n] + s * (v[n + n // 3] - v[n]) + t * (v[n + 2 * n // 3] - v[n])).astype(np.float32)
    gs = B.GridSet(np.full((1, 3), 9.0), np.full((1, 3), 9.5), np.array([[4, 4, 4]]), device="cuda")
    gs.buf.zero_()
    print("[gpu] sdf_labels", kind, direction, flush=True)
    got = B.sdf_labels(dev(verts), dev(tris, torch.int32), first, gs, 0, dev(pts)).cpu().numpy()
    signed_agree(got.astype(np.float64), orc.mesh_sdf(pts.astype(np.float64), v, tris, first))


def test_grid_with_nodes_in_the_plane_of_a_vertical_face(B, orc):
    """A plain grid over a wedge that meets the planes of its ends."""
    verts, tris, first = prism("wedge", (0.6, 0.8))
    lo, hi, n = verts.min(0) - np.float32(0.03), verts.max(0) + np.float32(0.03), 73
    print("[gpu] build_link_sdf wedge", flush=True)
    gs = B.GridSet(lo[None], hi[None], np.array([[n, n, n]]), device="cuda")
    B.build_link_sdf(dev(verts), dev(tris, torch.int32), first, gs, 0)
    got = gs.grid(0).cpu().numpy().astype(np.float64).ravel()
    h = ((hi.astype(np.float64) - lo) / (n - 1)).astype(np.float32)
    # the nodes as the GPU places them: one fused multiply-add per axis
    ax = [(lo[a].astype(np.float64) + np.arange(n) * h[a].astype(np.float64)).astype(np.float32) for a in range(3)]
    z, y, x = np.meshgrid(ax[2], ax[1], ax[0], indexing="ij")
    nodes = np.stack([x, y, z], -1).reshape(-1, 3).astype(np.float64)
    signed_agree(got, orc.mesh_sdf(nodes, verts.astype(np.float64), tris, first))
