"""Robot SDFs over environments that the links' blocks stick out of: a window of
a larger environment on the same voxels holds the larger one's bits, whichever
part of the blocks it cuts off (waves of the network build whose voxels lie
outside it in every configuration take no part), and an environment out of
reach holds nothing but +inf.

The voxel edge is a power of two and every corner a multiple of it, so that the
alignment (in double) and the voxel centres are the same numbers in both.
"""
import numpy as np
import pytest
import torch

from frnn_util import exact_params
from test_gpu_robot_sdf_edges import half_width, poses, small_arm, to_dev

pytestmark = pytest.mark.gpu
R, LO, N = 0.0625, np.array([-16, -16, -16]), (32, 32, 32)   # corner in voxels


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2309_12543_amd import lsdf
    lsdf.load_library()
    return lsdf


# first voxel and size of each window
WINDOWS = [((0, 0, 0), (5, 7, 3)), ((20, 18, 27), (12, 14, 5)), ((11, 0, 0), (1, 32, 32)), ((0, 13, 0), (32, 1, 32)),
           ((0, 0, 17), (32, 32, 1)), ((15, 16, 14), (1, 1, 1)), ((9, 10, 8), (13, 11, 12))]


@pytest.mark.parametrize("network", [False, True], ids=["exact", "network"])
@pytest.mark.parametrize("C", [1, 19])
def test_windows_hold_the_larger_environments_bits(B, network, C):
    rng = np.random.default_rng(31)
    gs, lo, hi, _, _ = small_arm(rng, torch.float32, B)
    T = to_dev(poses(rng, C, "rigid"))
    m = int(half_width(lo, hi, R).max())
    params = to_dev(exact_params(m))

    def build(first, n):
        env = B.make_env((LO + np.array(first)) * R, R, n)
        print("[gpu] robot_sdf", "network" if network else "exact", C, first, n, flush=True)
        out = torch.full((C, n[2], n[1], n[0]), float("nan"), device="cuda")
        return B.robot_sdf_build_frnn(T, gs, env, params, m, out=out) if network else B.robot_sdf_build(T, gs, env, out=out)

    whole = build((0, 0, 0), N)
    assert torch.isfinite(whole).any() and not torch.isnan(whole).any()
    for f, n in WINDOWS:
        part = whole[:, f[2]:f[2] + n[2], f[1]:f[1] + n[1], f[0]:f[0] + n[0]]
        assert torch.equal(build(f, n), part), (f, n)
    for far in ((800, 0, 0), (0, -800, 0), (0, 0, 800)):
        assert torch.isinf(build(far, (9, 6, 5))).all(), far
