"""The query's block lists, tiles, shares of a group and dealt chunks: calls
whose sizes reach each of them give the twin's bits, or the bits of the same
work cut into calls that do not."""
import numpy as np
import pytest
import torch

from test_gpu_query import B, assert_bit_exact, run_query, to_dev, twin, upload_grids  # noqa: F401

pytestmark = pytest.mark.gpu


def packed_cloud(w, T32, M, rng):
    """Points uniform in random links' boxes at random waypoints."""
    c, i = rng.integers(0, len(T32), M), rng.integers(0, w.L, M)
    l = rng.uniform(w.grid_lo[i], w.grid_hi[i])
    x = np.einsum("mab,mb->ma", T32[c, i, :, :3].astype(np.float64), l) + T32[c, i, :, 3]
    return x.astype(np.float32)


@pytest.fixture(scope="module")
def tiny_grids(orc, tiny):
    return orc.workload_grids(tiny)


# points: the last block of one to seven, a group and its neighbours, a cloud
# below one block; chunks: a quarter, a half, a whole and two groups; one
# workgroup per CU and the largest chunk fill the lists and the tiles
@pytest.mark.parametrize("chunk,bpc", [(8, 16), (32, 1), (64, 2), (128, 0), (8192, 1)])
@pytest.mark.parametrize("C,M", [(1, 7), (64, 8), (65, 63), (3, 64), (40, 65), (129, 513), (40, 30001)])
def test_shares_lists_and_tiles(B, orc, tiny, tiny_grids, C, M, chunk, bpc):
    rng = np.random.default_rng(1000 * C + M)
    q = np.resize(tiny.q, (C, tiny.q.shape[1])) + 1e-3 * np.arange(C)[:, None]
    T32 = orc.fk(tiny.robot.dh, q, tiny.robot.base_T).astype(np.float32)
    pts = packed_cloud(tiny, T32, M, rng)
    gs = upload_grids(B, tiny, tiny_grids)
    print("[gpu] lists", C, M, chunk, bpc, flush=True)
    out = B.query_min_distance_batched(to_dev(T32), gs, to_dev(pts), to_dev([0, C], torch.int32),
                                       to_dev([0, M], torch.int64), link_dist=True, tuning=B.make_tuning(chunk, bpc, 2))
    assert_bit_exact(tuple(o.cpu().numpy() for o in out), twin(orc, tiny, T32, tiny_grids, pts))


@pytest.mark.parametrize("schedule", [1, 2])
@pytest.mark.parametrize("K", [1, 5])
def test_dealt_chunks(B, orc, tiny, tiny_grids, K, schedule):
    """Enough chunks per wave that they are dealt on demand (chunks of one
    group on one workgroup per CU), against one call per trajectory and slice
    of points at the default tiling."""
    rng = np.random.default_rng(K)
    C, M = 320 * K, 60000 * K
    q = rng.uniform(-2.5, 2.5, size=(C, tiny.q.shape[1]))
    T32 = orc.fk(tiny.robot.dh, q, tiny.robot.base_T).astype(np.float32)
    pts = packed_cloud(tiny, T32, M, rng)
    c_off = np.concatenate([[0], np.sort(rng.integers(1, C, K - 1)), [C]])
    m_off = np.concatenate([[0], np.sort(rng.integers(1, M, K - 1)), [M]])
    gs, Td, pd = upload_grids(B, tiny, tiny_grids), to_dev(T32), to_dev(pts)
    print("[gpu] dealt", K, schedule, flush=True)
    d, link, ld = B.query_min_distance_batched(Td, gs, pd, to_dev(c_off, torch.int32), to_dev(m_off, torch.int64),
                                               link_dist=True, tuning=B.make_tuning(64, 1, schedule))
    want = torch.full_like(ld, float("inf"))
    for k in range(K):
        for s in range(m_off[k], m_off[k + 1], 17001):
            part = B.query_min_distance(Td[c_off[k]:c_off[k + 1]].contiguous(), gs,
                                        pd[s:min(s + 17001, m_off[k + 1])].contiguous(), link_dist=True)[2]
            want[c_off[k]:c_off[k + 1]] = torch.minimum(want[c_off[k]:c_off[k + 1]], part)
    assert torch.equal(ld, want)
    assert torch.equal(d, want.min(1).values)
    assert torch.equal(link.long(), torch.where(torch.isfinite(d), want.argmin(1), -1))


def test_points_without_a_finite_box(B, orc, tiny, tiny_grids):
    """Huge, infinite and NaN coordinates leave the rest of their block found."""
    rng = np.random.default_rng(5)
    T32 = orc.fk(tiny.robot.dh, tiny.q[:40], tiny.robot.base_T).astype(np.float32)
    pts = packed_cloud(tiny, T32, 2000, rng)
    clean = np.delete(pts, np.arange(0, 2000, 8), axis=0)
    pts[::8] = rng.choice([np.inf, -np.inf, np.nan, 3e38, -3e38, 1e20], size=(250, 3))
    gs = upload_grids(B, tiny, tiny_grids)
    assert_bit_exact(run_query(B, T32, gs, pts), twin(orc, tiny, T32, tiny_grids, clean))
