"""Diffusion over a graph of 2^31 - 1 edges, the most that is accepted: the
last rows' rounds reach past the last edge's 32-bit index.  Every edge of row i
leads to i with weight 1, so a step is out_i = degree_i g_i / |g| exactly up to
the scale, in the caller's order and in the scene's."""
import pytest
import torch

import paper_2410_14462_amd as lv

pytestmark = pytest.mark.gpu


def test_most_edges():
    if torch.cuda.mem_get_info()[0] < 80 << 30:
        pytest.skip("needs 80 GB of device memory")
    n, deg = 1 << 25, 64
    rp = (torch.arange(n + 1, device="cuda", dtype=torch.int64) * deg).clamp_(max=2 ** 31 - 1).to(torch.int32)
    col = torch.arange(n, device="cuda", dtype=torch.int32).repeat_interleave(deg)[:-1]
    assert col.numel() == 2 ** 31 - 1
    val = torch.ones(col.numel(), device="cuda", dtype=torch.bfloat16)
    print("graph of 2^31 - 1 edges", flush=True)
    graph = lv.Graph(rp, col, val)
    del rp, col, val
    degree = torch.full((n,), float(deg), device="cuda")
    degree[-1] = deg - 1
    gen = torch.Generator(device="cuda").manual_seed(1)
    x = torch.rand((n, 3), device="cuda", generator=gen)
    one = lambda *s: torch.ones(s, device="cuda")
    scene = lv.Scene(x, one(n, 3), one(n, 4), one(n))
    for D in (1, 5, 16):
        # small whole numbers: the sums of a row are exact
        g = torch.randint(1, 4, (n, D), device="cuda", generator=gen).float()
        for sc in (None, scene):
            print(f"most edges D={D} {'scene order' if sc else 'caller order'}", flush=True)
            out = graph.diffuse(g, 1, scene=sc)
            ratio = out / (degree[:, None] * g)
            lo, hi = ratio.amin(0), ratio.amax(0)
            # one rounding of the product with the scale and one of this division
            assert ((hi - lo) <= 2.0 ** -22 * hi).all(), (D, lo, hi)
            norm = g.double().square().sum(0).sqrt()
            # the norm's FP32 partial sums: chains of fewer than 2^16 roundings
            assert ((hi.double() * norm - 1.0).abs() <= 2.0 ** -8).all(), (D, hi, norm)
            del out, ratio
    graph.close()
    scene.close()
