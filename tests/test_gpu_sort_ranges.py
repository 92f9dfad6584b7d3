"""The radix sort and the positive count at the sizes where their kernels
change: block counts on both sides of the split digit scan (64 blocks of
4096 items, 11-bit digits), ragged last blocks.  Reference: the oracle's
filtering and anchors."""
import numpy as np
import pytest
import torch

import oracle
import paper_2410_14462_amd as lv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [63 * 4096, 63 * 4096 + 1, 64 * 4096 + 1, 79 * 4096 + 5, 1_000_003])
def test_filtering_and_anchors_around_the_split_scan(n):
    rng = np.random.default_rng(n)
    # half of the values tie with many others; signs of both kinds, zeros
    v = np.where(rng.uniform(size=n) < 0.5, rng.integers(-50, 50, n) / 8.0, rng.normal(size=n)).astype(np.float32)
    d = torch.as_tensor(v, device="cuda")
    for k in (1, n // 3, n - 1):
        assert np.array_equal(lv.prune_by_weight(d, k).cpu().numpy(), oracle.prune.keep_top_k(v, k))
    assert np.array_equal(lv.anchor_init(d, 0.1).cpu().numpy(), oracle.prune.anchor_init(v, 0.1))
