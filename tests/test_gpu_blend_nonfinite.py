"""A map with an infinite or NaN pixel: a Gaussian that no pixel counts (it lies
behind others that end every ray of its quadrants) takes nothing from the view,
for every form of the blend (tail channels, one wave and two, several groups),
element type and layout.  Opaque sheets of Gaussians cover the image; the
hidden ones behind them follow in the same lists."""
import numpy as np
import pytest
import torch

import paper_2410_14462_amd as lv
from synth import scenes

pytestmark = pytest.mark.gpu

HIDDEN = 40


def sheets(W, H):
    """Camera on +z looking at the origin; six opaque Gaussians much wider than
    the image in front (the second one ends every ray), HIDDEN small ones behind."""
    cam = scenes.look_at(np.array([0.0, 0.0, 4.0]), W, H, 40.0)
    rng = np.random.default_rng(W)
    front = np.zeros((6, 3))
    front[:, 2] = np.linspace(1.0, 0.5, 6)
    back = np.stack([rng.uniform(-0.8, 0.8, HIDDEN), rng.uniform(-0.5, 0.5, HIDDEN),
                     rng.uniform(-1.0, -0.5, HIDDEN)], 1)
    x = np.concatenate([front, back])
    s = np.concatenate([np.full((6, 3), 60.0), np.full((HIDDEN, 3), 0.1)])
    s[:6, 2] = 0.01
    q = np.tile([1.0, 0.0, 0.0, 0.0], (len(x), 1))
    o = np.concatenate([np.full(6, 0.999), np.full(HIDDEN, 0.9)])
    d = lambda a: torch.as_tensor(np.ascontiguousarray(a, np.float32), device="cuda")
    return lv.Scene(d(x), d(s), d(q), d(o)), cam


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
@pytest.mark.parametrize("dtype", ["f32", "bf16", "f32_px8", "bf16_px8", "fp8_px8"])
@pytest.mark.parametrize("W,H", [(90, 71), (640, 433)])  # below and above 4096 quadrants
@pytest.mark.parametrize("D", [1, 5, 32, 64, 100])
def test_uncounted_gaussians_take_nothing(D, W, H, dtype, bad):
    print(f"nonfinite D={D} {W}x{H} {dtype} {bad}", flush=True)
    scene, cam = sheets(W, H)
    rear = scenes.look_at(np.array([0.0, 0.0, -4.0]), W, H, 40.0)
    good = torch.full((H, W, D), 0.5, device="cuda")
    m = good.clone()
    scales = None
    if dtype.startswith("fp8"):  # no code is infinite; an infinite scale has the same effect
        m, sc = lv.encode(good, dtype)
        good, scales = m, torch.stack([torch.full_like(sc, bad), sc])
    else:
        m[H // 2 - 8:H // 2 + 8, W // 2 - 8:W // 2 + 8] = bad
        if dtype != "f32":
            good, m = lv.encode(good, dtype)[0], lv.encode(m, dtype)[0]
    acc = lv.Accum(scene, D, counts=True)
    acc.add([cam], [m], dtype=dtype, scales=scales[:1] if scales is not None else None)
    f, b, u = acc.finalize(want_sum=True)
    c = acc.counts().cpu().numpy()
    assert c[0] > 0 and (c[6:] == 0).all()
    assert (b[6:] == 0).all()
    assert (u[6:] == 0).all(), u[6:]  # NaN is not 0
    # seen in a finite view as well, they have that view's feature (weights of
    # one sign: a sum of at most 2^16 products, each within 2^-16)
    acc.add([rear], [good], dtype=dtype, scales=scales[1:] if scales is not None else None)
    f, b = acc.finalize()
    acc.close()
    seen = b[6:] > 0
    assert seen.any()
    assert ((f[6:][seen] - 0.5).abs() <= 0.5 * 2.0 ** -12).all(), f[6:][seen]
