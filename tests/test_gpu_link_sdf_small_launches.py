"""Mesh distances from launches of few workgroups, which are smaller ones, and of
many: the same nodes and points in either give the same bits, at the number of
workgroups and of triangles where the choice turns and beside them.  (Against the
oracle either is judged by the other tests of the mesh distance.)
"""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu
SMALL, MOST = 256, 256   # threads of a small workgroup, and the most of them in a launch


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2309_12543_amd import lsdf
    lsdf.load_library()
    return lsdf


class Mesh:
    def __init__(self, parts):
        at = np.cumsum([0] + [len(v) for v, _ in parts])
        self.verts = np.concatenate([v for v, _ in parts])
        self.tris = np.concatenate([t + k for (_, t), k in zip(parts, at)]).astype(np.int32)
        self.comp_first = np.cumsum([0] + [len(t) for _, t in parts]).astype(np.int32)


def mesh(kind):
    box = synth.box_mesh((0.05, -0.02, 0.03), (0.11, 0.07, 0.05))
    v, t = synth.capsule_mesh((-0.1, 0.02, 0.0), (0.13, -0.04, 0.2), 0.06)   # 256 triangles
    return {"box": Mesh([box]), "most": Mesh([(v, t)]), "open": Mesh([(v, t[1:])]),
            "more": Mesh([(v, t), box])}[kind]   # 268: large workgroups in any launch


def grids(B, meshes, n):
    lo = np.array([m.verts.min(0) - 0.05 for m in meshes], dtype=np.float32)
    hi = np.array([m.verts.max(0) + 0.05 for m in meshes], dtype=np.float32)
    return B.build_robot_grids(meshes, lo, hi, np.array(n))


@pytest.mark.parametrize("kind", ["box", "most", "open", "more"])
@pytest.mark.parametrize("n", [(5, 7, 9), (16, 16, 16), (2, 3, 40)])
def test_grids_of_small_and_large_launches(B, kind, n):
    m = mesh(kind)
    alone = grids(B, [m], [n])
    beside = grids(B, [m, mesh("box")], [n, (64, 64, 64)])   # 1,024 small workgroups more
    assert torch.equal(alone.grid(0), beside.grid(0))


@pytest.mark.parametrize("side", [39, 40, 41])   # 250, 250 and 275 small workgroups of bricks
def test_grid_at_the_turn(B, side):
    m = mesh("box")
    alone = grids(B, [m], [(side, 40, 40)])
    beside = grids(B, [m, m], [(side, 40, 40), (64, 64, 64)])
    assert torch.equal(alone.grid(0), beside.grid(0))


@pytest.mark.parametrize("kind", ["box", "most", "open", "more"])
@pytest.mark.parametrize("N", [1, 255, 257, SMALL * MOST, SMALL * MOST + 1])
def test_labels_of_small_and_large_launches(B, kind, N):
    m = mesh(kind)
    gs = grids(B, [m], [(16, 16, 16)])
    v = torch.as_tensor(np.asarray(m.verts, dtype=np.float32), device="cuda")
    t = torch.as_tensor(m.tris, device="cuda")
    gen = np.random.default_rng(11)
    p = torch.as_tensor(gen.uniform(m.verts.min(0) - 0.3, m.verts.max(0) + 0.3, size=(SMALL * MOST + 600, 3))
                        .astype(np.float32), device="cuda")
    many = B.sdf_labels(v, t, m.comp_first, gs, 0, p)
    few = B.sdf_labels(v, t, m.comp_first, gs, 0, p[:N].contiguous())
    assert torch.isfinite(many).all()
    assert torch.equal(few, many[:N])
