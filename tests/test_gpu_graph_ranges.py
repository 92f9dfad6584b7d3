"""The device graph where its kernels change: neighbour counts around the
list sizes (8, 16, 32), channel counts around the lanes per edge and the
16-byte loads (also rows that are not 16-byte aligned), rows of more than 32
and of more than 64 entries (many centres at one place choose the same
neighbours), grids of one cell and flat scenes.  Reference: the FP64 oracle
graph, structure bit-exact, values within FP32 rounding."""
import numpy as np
import pytest
import torch

import oracle
import paper_2410_14462_amd as lv

pytestmark = pytest.mark.gpu


def centres(n, seed):
    """Uniform centres; 130 at one place and 40 at another."""
    x = np.random.default_rng(seed).uniform(-1, 1, (n, 3)).astype(np.float32)
    x[50:180] = x[50]
    x[200:240] = x[200]
    return x


def check(x, f, k, aligned=True):
    n, D = f.shape
    d = lambda a: torch.as_tensor(np.ascontiguousarray(a, np.float32), device="cuda")
    scene = lv.Scene(d(x), d(np.full((n, 3), 0.01)), d(np.tile([1.0, 0, 0, 0], (n, 1))), d(np.full(n, 0.5)))
    ft = torch.empty(n * D + 1, device="cuda")[0 if aligned else 1:][:n * D].view(n, D)
    ft.copy_(d(f))
    rp, col, val = (t.cpu().numpy() for t in lv.Graph.knn(scene, ft, k).csr())
    rrp, rcol, rval = oracle.graph.knn_graph(x, f, k)
    assert np.array_equal(rp, rrp) and np.array_equal(col, rcol)
    assert np.all(np.abs(val.astype(np.float64) - rval) <= 2e-7 * np.abs(rval) + 1e-9)
    return int(np.diff(rp).max())


@pytest.mark.parametrize("k", [1, 8, 9, 16, 17, 32])
def test_list_sizes_and_long_rows(k):
    x = centres(1500, k)
    f = np.random.default_rng(k + 1).normal(size=(1500, 5)).astype(np.float32) + 1.0
    longest = check(x, f, k)
    assert longest > 64  # a row for the longest path too


@pytest.mark.parametrize("aligned", [True, False])
@pytest.mark.parametrize("D", [1, 4, 8, 9, 12, 64, 128, 129, 132])
def test_channel_counts(D, aligned):
    check(centres(600, D), np.random.default_rng(D).normal(size=(600, D)).astype(np.float32) + 0.5, 8, aligned)


@pytest.mark.parametrize("n", [3, 17, 65])
def test_small_and_flat_scenes(n):
    rng = np.random.default_rng(n)
    x = rng.uniform(-1, 1, (n, 3)).astype(np.float32)
    x[:, 1] = 0.25  # flat along y
    check(x, rng.normal(size=(n, 6)).astype(np.float32) + 1.0, min(16, n - 1))
