"""Chunks of one to nine groups of 64 points: full batches of four group boxes,
and last ones of one to three, give the twin's bits."""
import numpy as np
import pytest
import torch

from test_gpu_query import B, assert_bit_exact, to_dev, twin, upload_grids  # noqa: F401
from test_gpu_query_lists import packed_cloud

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("groups", range(1, 10))
def test_groups_of_a_chunk(B, orc, tiny, tiny_grids, groups):
    rng = np.random.default_rng(groups)
    M = 64 * groups - groups % 3     # the last group whole, or a point or two short
    T32 = orc.fk(tiny.robot.dh, tiny.q[:45], tiny.robot.base_T).astype(np.float32)
    pts = packed_cloud(tiny, T32, M, rng)
    gs = upload_grids(B, tiny, tiny_grids)
    print("[gpu] groups", groups, M, flush=True)
    out = B.query_min_distance_batched(to_dev(T32), gs, to_dev(pts), to_dev([0, 45], torch.int32),
                                       to_dev([0, M], torch.int64), link_dist=True, tuning=B.make_tuning(1024, 1, 2))
    assert_bit_exact(tuple(o.cpu().numpy() for o in out), twin(orc, tiny, T32, tiny_grids, pts))
