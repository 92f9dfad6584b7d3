"""The walk's kernels on both sides of their rules: few quadrants (two waves
per quadrant) and more than 4096 (one, unless the group has over 32 channels);
channel counts at the edges of the tails, the 32-channel blocks and the groups
of the uplift and the render, rendered groups that share a walk and that do
not; tiles whose lists run over many steps and queues.  Reference: the FP64
oracle, with the parity bars of the uplift and render tests (1e-4 relative to
the sum of magnitudes, alpha 1e-5, counts exact) off the pixels and Gaussians
that an ambiguous decision touches."""
import numpy as np
import pytest
import torch

import oracle
import paper_2410_14462_amd as lv
from helpers import beta_error, counts_match, feature_error
from synth import philox, scenes

pytestmark = pytest.mark.gpu

# (views, W, H): 2 x 120 and 1 x 4480 quadrants
LAUNCHES = [(2, 90, 71), (1, 640, 433)]


@pytest.fixture(scope="module")
def scene():
    sc = scenes.make_scene(71, 6000, -3.2, 0.5, -2.0, 1.0)  # faint: long lists
    return sc, lv.Scene.from_arrays(sc)


def cameras(m, W, H):
    return [scenes.look_at(e, W, H, 50.0) for e in scenes.fibonacci_eyes(m, 4.0)]


@pytest.mark.parametrize("launch", LAUNCHES)
@pytest.mark.parametrize("D", [1, 4, 5, 32, 33, 64, 68])
def test_uplift_both_walks(scene, launch, D):
    sc, gs = scene
    cams = cameras(*launch)
    maps = [scenes.map_uniform(72, v, c.height, c.width, D) for v, c in enumerate(cams)]
    print(f"uplift {launch} D={D}", flush=True)
    acc = lv.Accum(gs, D, counts=True)
    acc.add(cams, [torch.as_tensor(x, device="cuda") for x in maps])
    f, b = acc.finalize()
    c = acc.counts().cpu().numpy().astype(np.int64)
    acc.close()
    ref = oracle.uplift(sc, cams, maps)
    assert feature_error(f.cpu().numpy(), ref).max(initial=0.0) < 1e-4
    assert beta_error(b.cpu().numpy(), ref).max(initial=0.0) < 1e-4
    assert counts_match(c, ref)


@pytest.mark.parametrize("launch,D", [(LAUNCHES[0], d) for d in (3, 32, 33, 64, 65, 128, 129, 257, 384)] +
                                     [(LAUNCHES[1], d) for d in (3, 64, 128, 129, 260)])
def test_render_both_walks(scene, launch, D):
    sc, gs = scene
    cams = cameras(*launch)
    g = philox.normal(73 + D, 0, sc.n * D).reshape(sc.n, D)
    print(f"render {launch} D={D}", flush=True)
    outs, alphas = gs.render(cams, torch.as_tensor(g, device="cuda"))
    for v, cam in enumerate(cams):
        ref, ref_a, amb = oracle.render(sc, cam, g, amb_px=True)
        scale, _ = oracle.render(sc, cam, np.abs(g))
        ok = ~amb
        err = np.abs(outs[v].cpu().numpy().astype(np.float64) - ref) / np.maximum(scale, 1e-30)
        assert amb.sum() <= 0.002 * amb.size
        assert err[ok].max() < 1e-4
        assert np.abs(alphas[v].cpu().numpy() - ref_a)[ok].max() < 1e-5
