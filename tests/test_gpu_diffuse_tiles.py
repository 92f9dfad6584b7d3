"""A diffusion step on both sides of the rules that choose its form by the number
of rows (16, 32 or 64 rows per wave for few channels; a small and a large form for
rows of pieces), and on graphs of which every block takes several tiles of rows
one after the other, with hubs whose edges are loaded over several rounds.
Reference: the FP64 oracle on the same CSR."""
import numpy as np
import pytest
import torch

import paper_2410_14462_amd as lv
from oracle import diffuse as od
from test_gpu_diffuse_ranges import ragged_graph

pytestmark = pytest.mark.gpu

EDGES = [(1, 32768), (1, 32769), (2, 65536), (3, 65537), (4, 32769), (4, 65537),
         (8, 131072), (8, 131073), (16, 65537), (32, 32768), (64, 16384), (64, 16385)]
TILES = [(8, 700_001), (16, 350_003), (32, 170_003), (64, 90_001)]  # at least two tiles per block


@pytest.mark.parametrize("sdt", ["f32", "bf16"])
@pytest.mark.parametrize("D,n", EDGES + TILES)
def test_forms_and_tiles(D, n, sdt):
    # positive terms: a row's sum, the scale and the norm are each off by at most
    # (terms in a chain) 2^-24 relatively; the hub's chain is the longest, a norm's
    # is below 100.  BF16: the signal is rounded once (2^-9) more
    hub = 2500
    rp, col, val = ragged_graph(n, 3 * n + D, hub)
    g0 = torch.as_tensor(np.random.default_rng(n + D).uniform(0.1, 1.0, (n, D)).astype(np.float32))
    if sdt == "bf16":
        g0 = g0.to(torch.bfloat16)
    G = lv.Graph(*(torch.as_tensor(x, device="cuda") for x in (rp, col, val)))
    print(f"diffuse n={n} D={D} {sdt}", flush=True)
    out = G.diffuse(g0.cuda(), 1).float().cpu().numpy().astype(np.float64)
    ref = od.diffuse(od.csr_matrix(n, rp, col, val), g0.float().numpy().astype(np.float64), 1)
    tol = (hub + 100) * 2.0 ** -24 + (2.0 ** -8 if sdt == "bf16" else 0.0)
    assert np.all(np.abs(out - ref) <= tol * np.abs(ref))


@pytest.mark.parametrize("D", [1, 16, 37])
@pytest.mark.parametrize("steps", [63, 64, 95, 96, 97, 130])
def test_more_steps_than_norm_rows(steps, D):
    # 64 rows of norms are used in turn; positive terms, so a step is off by at
    # most (terms in a chain) 2^-24 relatively (rows that feed on themselves alone
    # may die out: below 1e-37 FP32 is no longer normal)
    n, hub = 300, 40
    rp, col, val = ragged_graph(n, 5, hub)
    rp, col, val = with_self_loops(n, rp, col, val)
    g0 = np.random.default_rng(D).uniform(0.1, 1.0, (n, D)).astype(np.float32)
    G = lv.Graph(*(torch.as_tensor(x, device="cuda") for x in (rp, col, val)))
    out = G.diffuse(torch.as_tensor(g0, device="cuda"), steps).cpu().numpy().astype(np.float64)
    ref = od.diffuse(od.csr_matrix(n, rp, col, val), g0.astype(np.float64), steps)
    assert np.all(np.abs(out - ref) <= steps * (hub + 100) * 2.0 ** -24 * np.abs(ref) + 1e-37)


def with_self_loops(n, rp, col, val):
    """One more edge of weight 1 per row, to itself: no signal dies out."""
    deg = np.diff(rp)
    rp2 = np.concatenate([[0], np.cumsum(deg + 1)]).astype(np.int32)
    col2 = np.insert(col, rp[1:], np.arange(n)).astype(np.int32)
    val2 = np.insert(val, rp[1:], 1.0).astype(np.float32)
    return rp2, col2, val2
