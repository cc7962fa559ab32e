"""The rounding of the mesh distance (lsdf_build_link_sdf): over grids of a whole
arm's links, in root mean square no further from the oracle's double precision
than a plain single-precision evaluation in numpy, which takes each Voronoi
region's closest point with a division, a product and a sum, rounded each.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def plain_distance(p, tri):
    """Distances float32 [N] of points p [N][3] to the triangles [T][3][3], each
    operation rounded to float32."""
    one = np.float32(1.0)
    best = np.full(len(p), np.inf, dtype=np.float32)
    dot = lambda u, v: (u[..., 0] * v[..., 0] + u[..., 1] * v[..., 1]) + u[..., 2] * v[..., 2]
    for a, b, c in tri:
        ab, ac, ap, bp, cp = b - a, c - a, p - a, p - b, p - c
        d1, d2, d3, d4, d5, d6 = (dot(e, x) for x in (ap, bp, cp) for e in (ab, ac))
        va, vb, vc = d3 * d6 - d5 * d4, d5 * d2 - d1 * d6, d1 * d4 - d3 * d2
        with np.errstate(all="ignore"):
            inv = one / (va + vb + vc)
            along = lambda o, t, e: o + t[:, None] * e
            cases = [((d1 <= 0) & (d2 <= 0), np.broadcast_to(a, p.shape)),
                     ((d3 >= 0) & (d4 <= d3), np.broadcast_to(b, p.shape)),
                     ((vc <= 0) & (d1 >= 0) & (d3 <= 0), along(a, d1 / (d1 - d3), ab)),
                     ((d6 >= 0) & (d5 <= d6), np.broadcast_to(c, p.shape)),
                     ((vb <= 0) & (d2 >= 0) & (d6 <= 0), along(a, d2 / (d2 - d6), ac)),
                     ((va <= 0) & (d4 >= d3) & (d5 >= d6), along(b, (d4 - d3) / ((d4 - d3) + (d5 - d6)), c - b))]
            q = along(along(a, vb * inv, ab), vc * inv, ac)
        for on, point in reversed(cases):
            q = np.where(on[:, None], point, q)
        assert q.dtype == np.float32
        r = p - q
        best = np.fmin(best, dot(r, r))
    return np.sqrt(best)


def test_rounding_is_no_worse_than_a_plain_evaluations(orc, tiny):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2309_12543_amd import lsdf as B
    n, got_err, plain_err = 20, [], []
    for m in tiny.robot.links:
        verts, tris = m.verts.astype(np.float32), np.asarray(m.tris, dtype=np.int32)
        lo, hi = verts.min(0) - np.float32(0.05), verts.max(0) + np.float32(0.05)
        gs = B.GridSet(lo[None], hi[None], np.array([[n, n, n]]), device="cuda")
        print("[gpu] build_link_sdf", len(tris), flush=True)
        B.build_link_sdf(torch.as_tensor(verts, device="cuda"), torch.as_tensor(tris, device="cuda"), m.comp_first, gs, 0)
        h = ((hi.astype(np.float64) - lo) / (n - 1)).astype(np.float32)
        # the nodes as the GPU places them: one fused multiply-add per axis
        ax = [(lo[a].astype(np.float64) + np.arange(n) * h[a].astype(np.float64)).astype(np.float32) for a in range(3)]
        z, y, x = np.meshgrid(ax[2], ax[1], ax[0], indexing="ij")
        nodes = np.stack([x, y, z], -1).reshape(-1, 3)
        ref = orc.mesh_sdf(nodes.astype(np.float64), verts.astype(np.float64), tris, m.comp_first)
        # (inside a part both sides take other triangles than the nearest of all)
        out = ref > 0
        got_err.append(gs.grid(0).cpu().numpy().ravel().astype(np.float64)[out] - ref[out])
        plain_err.append(plain_distance(nodes[out], verts[tris]).astype(np.float64) - ref[out])
    got, plain = (np.sqrt(np.mean(np.concatenate(e) ** 2)) for e in (got_err, plain_err))
    print("[gpu] rms", got, "plain", plain, flush=True)
    assert got <= plain, (got, plain)
