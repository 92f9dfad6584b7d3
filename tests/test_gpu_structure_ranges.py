"""The structure build where the sort changes its block size and its digit
scan: few and many views (below and above 128 blocks of 4096 items), ragged
item counts, one tile to many.  Reference: the oracle's per-tile lists,
uplifted features and weight sums."""
import numpy as np
import pytest
import torch

import oracle
import paper_2410_14462_amd as lv
from helpers import beta_error, feature_error
from synth import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m,W,H", [(1, 1, 16, 16), (1023, 2, 40, 24), (1025, 1, 200, 130), (4097, 3, 64, 64),
                                     (9000, 45, 48, 33)])
def test_uplift_over_sort_block_sizes(n, m, W, H):
    sc = scenes.make_scene(90 + n, n, -3.5, 0.5, 0.0, 1.0)
    cams = [scenes.look_at(e, W, H, 55.0) for e in scenes.fibonacci_eyes(m, 4.0)]
    maps = [scenes.map_uniform(91, v, H, W, 5) for v in range(m)]
    f, b = lv.Scene.from_arrays(sc).uplift(cams, [torch.as_tensor(x, device="cuda") for x in maps])
    ref = oracle.uplift(sc, cams, maps)
    assert feature_error(f.cpu().numpy(), ref).max(initial=0.0) < 1e-4
    assert beta_error(b.cpu().numpy(), ref).max(initial=0.0) < 1e-4
