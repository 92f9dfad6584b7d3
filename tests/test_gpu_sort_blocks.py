"""The radix sort on both sides of its rules: blocks of 1024 or 4096 items (below
128 blocks of 4096, from 128 on) and the digit scan in one piece or split (from
64 blocks on with 10- and 11-bit digits, 256 with the 8-bit digits of the depth
sort).  References: the oracle's filtering and anchors, its per-tile lists."""
import numpy as np
import pytest
import torch

import oracle
import paper_2410_14462_amd as lv
from synth import scenes
from test_gpu_uplift import check_structure

pytestmark = pytest.mark.gpu


# 63 and 64 small blocks (the scan in one piece, split), 508 small blocks and 128
# large ones
@pytest.mark.parametrize("n", [63 * 1024, 63 * 1024 + 1, 64 * 1024 + 1, 127 * 4096, 127 * 4096 + 1, 128 * 4096 + 1])
def test_filtering_and_anchors(n):
    rng = np.random.default_rng(n)
    v = np.where(rng.uniform(size=n) < 0.5, rng.integers(-50, 50, n) / 8.0, rng.normal(size=n)).astype(np.float32)
    d = torch.as_tensor(v, device="cuda")
    for k in (1, n // 3, n - 1):
        assert np.array_equal(lv.prune_by_weight(d, k).cpu().numpy(), oracle.prune.keep_top_k(v, k))
    assert np.array_equal(lv.anchor_init(d, 0.1).cpu().numpy(), oracle.prune.anchor_init(v, 0.1))


@pytest.mark.parametrize("n", [255 * 1024, 255 * 1024 + 1, 300_000])
def test_depth_sort_of_one_view(n):
    sc = scenes.make_scene(n % 97, n, -5.5, 0.5, 0.0, 1.0)
    gs = lv.Scene.from_arrays(sc)
    cam = scenes.look_at(scenes.fibonacci_eyes(1, 4.0)[0], 333, 251, 55.0)
    assert check_structure(gs, sc, cam) > 10000
