"""FP8 and pixel-block encoding at the edges of their kernels: channel counts
with and without four-channel loads, sources and destinations that are not
16-byte aligned, ragged widths, quotients at the midpoints of the codes,
zeros of both signs, channels whose scale is outside the range of the fused
division.  Codes and scales are compared bit for bit with the FP32 division
and torch's E4M3FN rounding on the CPU."""
import pytest
import torch

import paper_2410_14462_amd as lv

pytestmark = pytest.mark.gpu


def source(H, W, D, shift):
    g = torch.Generator().manual_seed(H * 1000 + D)
    x = torch.randn((H, W, D), generator=g)
    # midpoints between codes, times the channel's scale
    mid = torch.randint(0, 3584, (H, W, D), generator=g).float() / 8.0
    top = torch.rand((D,), generator=g) + 0.5
    sign = torch.where(torch.rand((H, W, D), generator=g) < 0.5, -1.0, 1.0)
    ties = torch.minimum(mid * (top / 448.0), top) * sign
    ties[0, 0] = top
    x = torch.where(torch.arange(D) % 3 == 1, ties, x)
    x[1] = torch.where(torch.arange(D) % 2 == 0, 0.0, -0.0)  # zeros of both signs
    if D > 2:
        x[:, :, 0] *= 1e-35  # scales below and above what the fused division takes
        x[:, :, 2] *= 1e33
    buf = torch.empty(H * W * D + shift, device="cuda")
    return x, buf[shift:].view(H, W, D).copy_(x)


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("H,W,D", [(5, 7, 1), (9, 8, 3), (6, 9, 4), (4, 33, 12), (33, 100, 40), (3, 17, 1028)])
def test_codes_and_layouts_bit_exact(H, W, D, shift):
    x, d = source(H, W, D, shift)
    amax = x.abs().amax(dim=(0, 1))
    scale = torch.where(amax > 0, (amax.double() / 448.0).float(), torch.ones_like(amax))
    code = (x / scale).clamp(-448.0, 448.0).to(torch.float8_e4m3fn).view(torch.uint8)
    blocks = lambda t: torch.nn.functional.pad(t, (0, 0, 0, -W % 8)).view(H, -1, 8, D).transpose(2, 3)
    y, sc = lv.encode(d, "fp8")
    assert torch.equal(sc.cpu(), scale) and torch.equal(y.cpu(), code)
    y, sc = lv.encode(d, "fp8_px8")
    assert torch.equal(sc.cpu(), scale) and torch.equal(y.cpu(), blocks(code))
    y, _ = lv.encode(d, "bf16_px8")
    assert torch.equal(y.cpu().view(torch.int16), blocks(x.to(torch.bfloat16)).contiguous().view(torch.int16))
    y, _ = lv.encode(d, "f32_px8")
    assert torch.equal(y.cpu().view(torch.int32), blocks(x).contiguous().view(torch.int32))
