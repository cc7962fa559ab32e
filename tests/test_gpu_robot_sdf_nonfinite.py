"""Robot SDFs from link grids that hold NaN and infinite nodes: a pair whose
cell touches one has no value, in the exact build and in the build through the
grid-transformation network alike, and every other pair keeps its own.

The exact build is held to the single-precision twin's bits.  The network build
is judged in double precision with the tolerances that tests/
test_gpu_robot_sdf_edges.py derives (1.5e-4 for a value, 1e-5 grid steps for the
side of a box or cell face).
"""
import numpy as np
import pytest
import torch

from frnn_util import centres, exact_params
from test_gpu_robot_sdf_edges import TOL, half_width, poses, small_arm, to_dev

pytestmark = pytest.mark.gpu
R, ELO, N = 0.0625, (-0.5, -0.25, -0.5), (19, 12, 17)


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2309_12543_amd import lsdf
    lsdf.load_library()
    return lsdf


def poisoned_arm(B, rng):
    """small_arm with a NaN in one link's grid and a NaN and infinities in the other's."""
    gs, lo, hi, n, clean = small_arm(rng, torch.float32, B)
    bad = [g.copy() for g in clean]
    bad[0][2, 2, 2] = np.nan
    bad[1][1, 2, 3], bad[1][3, 3, 1], bad[1][0, 0, 0] = np.inf, -np.nan, np.inf
    for i in range(2):
        gs.set_grid(i, bad[i])
    return gs, lo, hi, n, clean, bad


def test_exact_build_drops_pairs_without_a_value(B, orc):
    rng = np.random.default_rng(17)
    gs, lo, hi, gn, _, bad = poisoned_arm(B, rng)
    T = poses(rng, 6, "rigid")
    print("[gpu] robot_sdf_build, non-finite nodes", flush=True)
    got = B.robot_sdf_build(to_dev(T), gs, B.make_env(ELO, R, N)).cpu().numpy().reshape(6, -1)
    each = orc.query_f32_each(T, lo, hi, gn, bad, orc.voxel_centres(ELO, R, N, np.arange(int(np.prod(N)))))
    assert np.isnan(each).any()
    want = np.fmin(np.fmin(each[:, 0], each[:, 1]), np.float32(np.inf)).astype(np.float32)
    assert np.array_equal(got.view(np.uint32), want.view(np.uint32))


def test_network_build_drops_pairs_without_a_value(B, orc):
    rng = np.random.default_rng(18)
    C = 21
    gs, lo, hi, gn, clean, bad = poisoned_arm(B, rng)
    T = poses(rng, C, "rigid")
    m = int(half_width(lo, hi, R).max())
    params = exact_params(m).astype(np.float32)
    print("[gpu] robot_sdf_build_frnn, non-finite nodes", flush=True)
    got = B.robot_sdf_build_frnn(to_dev(T), gs, B.make_env(ELO, R, N), to_dev(params), m).cpu().numpy().astype(np.float64)
    assert not np.isnan(got).any()
    j = np.rint((centres(m) + 1) * m - 0.5).astype(int)
    f = orc.frnn_forward(params.astype(np.float64), m, T[:, :, :, :3].reshape(-1, 3, 3).astype(np.float64))
    f = f.reshape(C, 2, -1, 3)

    def has_value(i, u):
        a = np.clip(np.floor(u).astype(int), 0, gn[i] - 2)[::-1]
        return np.isfinite(bad[i][a[0]:a[0] + 2, a[1]:a[1] + 2, a[2]:a[2] + 2]).all()

    sure, maybe = np.full(got.shape, np.inf), np.full(got.shape, np.inf)
    dropped, sides = 0, np.array(list(np.ndindex(3, 3, 3))) - 1
    for c in range(C):
        for i in range(2):
            rot, t = T[c, i, :, :3].astype(np.float64), T[c, i, :, 3].astype(np.float64)
            k, dt = orc.align(t, ELO, R, m)
            u = (m * R * f[c, i] - rot.T @ dt - lo[i]) / ((hi[i].astype(np.float64) - lo[i]) / (gn[i] - 1))
            vox = j + k
            near = ((vox >= 0) & (vox < N)).all(1) & ((u >= -1e-5) & (u <= gn[i] - 1 + 1e-5)).all(1)
            for q in np.flatnonzero(near):
                at = (c, vox[q, 2], vox[q, 1], vox[q, 0])
                # the cells the point may lie in, within the tolerance of their faces
                cells = [has_value(i, np.clip(u[q] + 1e-5 * s, 0, gn[i] - 1)) for s in sides]
                val = orc.trilinear_f64(clean[i].astype(np.float64), np.clip(u[q], 0, gn[i] - 1))
                dropped += not any(cells)
                if any(cells):
                    maybe[at] = min(maybe[at], val)
                if all(cells) and ((u[q] >= 1e-5) & (u[q] <= gn[i] - 1 - 1e-5)).all():
                    sure[at] = min(sure[at], val)
    assert dropped > 100
    assert np.isinf(got[np.isinf(maybe)]).all() and np.isfinite(got[np.isfinite(sure)]).all()
    fin = np.isfinite(got)
    assert (got[fin] >= maybe[fin] - TOL).all()
    assert (got[np.isfinite(sure)] <= sure[np.isfinite(sure)] + TOL).all()
