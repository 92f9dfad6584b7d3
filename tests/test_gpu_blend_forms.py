"""The one-wave forms of the one-group blend (more than 4096 quadrants and at most
32 channels, or short lists) in every element type and layout, with sets that
skip views, and the deterministic accumulator in both forms.  Reference: the FP64 oracle on the maps
as stored (decoded on the CPU), with the bars of the uplift tests."""
import numpy as np
import pytest
import torch

import oracle
import paper_2410_14462_amd as lv
from helpers import beta_error, counts_match, feature_error
from synth import scenes

pytestmark = pytest.mark.gpu

W, H = 640, 433  # 4480 quadrants a view


@pytest.fixture(scope="module")
def scene():
    sc = scenes.make_scene(71, 6000, -3.2, 0.5, -2.0, 1.0)  # faint: long lists
    return sc, lv.Scene.from_arrays(sc)


def cameras(m, w=W, h=H):
    return [scenes.look_at(e, w, h, 50.0) for e in scenes.fibonacci_eyes(m, 4.0)]


def stored(x, elem):
    """The FP32 values that the map holds in `elem`, and its FP8 scales."""
    if elem == "f32":
        return x, None
    y, sc = lv.encode(x, elem)
    if elem == "bf16":
        return y.float(), None
    return y.cpu().view(torch.float8_e4m3fn).float().cuda() * sc, sc


@pytest.mark.parametrize("layout", ["", "_px8"])
@pytest.mark.parametrize("elem", ["f32", "bf16", "fp8"])
@pytest.mark.parametrize("D", [3, 5, 32])
def test_one_wave_storage(scene, D, elem, layout):
    sc, gs = scene
    cams = cameras(1)
    print(f"one wave D={D} {elem}{layout}", flush=True)
    x = torch.as_tensor(scenes.map_uniform(74, 0, H, W, D), device="cuda")
    ref_map, scales = stored(x, elem)
    m = x if elem + layout == "f32" else lv.encode(x, elem + layout)[0]
    acc = lv.Accum(gs, D, counts=True)
    acc.add(cams, [m], dtype=elem + layout, scales=None if scales is None else scales.view(1, D))
    f, b = acc.finalize()
    c = acc.counts().cpu().numpy().astype(np.int64)
    acc.close()
    ref = oracle.uplift(sc, cams, [ref_map.cpu().numpy()])
    assert feature_error(f.cpu().numpy(), ref).max(initial=0.0) < 1e-4
    assert beta_error(b.cpu().numpy(), ref).max(initial=0.0) < 1e-4
    assert counts_match(c, ref)


@pytest.mark.parametrize("dtype", ["f32", "bf16", "fp8", "f32_px8", "bf16_px8", "fp8_px8"])
@pytest.mark.parametrize("n", [500, 20_000])  # lists below and above the rule's 128 in the mean
@pytest.mark.parametrize("D", [33, 64, 67])
def test_wide_groups_short_and_long_lists(D, n, dtype):
    sc = scenes.make_scene(78, n, -3.2, 0.5, -2.0, 1.0)
    gs = lv.Scene.from_arrays(sc)
    cams = cameras(1)
    print(f"lists n={n} D={D} {dtype}", flush=True)
    x = torch.as_tensor(scenes.map_uniform(79, 0, H, W, D), device="cuda")
    ref_map, scales = stored(x, dtype.split("_")[0])
    m = x if dtype == "f32" else lv.encode(x, dtype)[0]
    acc = lv.Accum(gs, D, counts=True)
    acc.add(cams, [m], dtype=dtype, scales=None if scales is None else scales.view(1, D))
    f, b = acc.finalize()
    c = acc.counts().cpu().numpy().astype(np.int64)
    tiles = ((W + 15) // 16) * ((H + 15) // 16)
    assert (acc.stats()["pairs"] >= 128 * tiles) == (n > 500)
    acc.close()
    ref = oracle.uplift(sc, cams, [ref_map.cpu().numpy()])
    assert feature_error(f.cpu().numpy(), ref).max(initial=0.0) < 1e-4
    assert beta_error(b.cpu().numpy(), ref).max(initial=0.0) < 1e-4
    assert counts_match(c, ref)


def test_one_wave_set_skipping_a_view(scene):
    sc, gs = scene
    cams = cameras(2)
    host = [[scenes.map_uniform(75 + k, v, H, W, D) for v in range(2)] for k, D in enumerate((20, 10))]
    dev = [[torch.as_tensor(x, device="cuda") for x in hm] for hm in host]
    A, B = lv.Accum(gs, 20, counts=True), lv.Accum(gs, 10, counts=True)
    lv.accumulate_sets(cams, [(A, dev[0]), (B, [None, dev[1][1]])])
    for acc, ref in ((A, oracle.uplift(sc, cams, host[0])), (B, oracle.uplift(sc, cams[1:], host[1][1:]))):
        f, b = acc.finalize()
        assert counts_match(acc.counts().cpu().numpy(), ref)
        assert feature_error(f.cpu().numpy(), ref).max() < 1e-4
        assert beta_error(b.cpu().numpy(), ref).max() < 1e-4
        acc.close()


@pytest.mark.parametrize("w,h", [(90, 71), (W, H)])
@pytest.mark.parametrize("D", [3, 32, 64])
def test_deterministic_accumulator(scene, D, w, h):
    sc, gs = scene
    cams = cameras(2, w, h)
    host = [scenes.map_uniform(77, v, h, w, D) for v in range(2)]
    maps = [torch.as_tensor(x, device="cuda") for x in host]

    def run(groups):
        acc = lv.Accum(gs, D, counts=True, deterministic=True)
        for g in groups:
            acc.add([cams[v] for v in g], [maps[v] for v in g])
        f, b, u = acc.finalize(want_sum=True)
        out = [x.cpu().numpy() for x in (f, b, u, acc.counts())]
        acc.close()
        return out

    one, two = run([[0, 1]]), run([[1], [0]])
    assert all(np.array_equal(x, y) for x, y in zip(one, two))
    ref = oracle.uplift(sc, cams, host)
    # each partial sum is rounded to 2^-36 more than in FP32
    assert feature_error(one[0], ref)[ref.beta[(ref.beta > 0) & ref.strict] > 1e-3].max() < 1e-4
    assert beta_error(one[1], ref).max() < 1e-4
    assert counts_match(one[3], ref)
