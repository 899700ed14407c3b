"""The 3x3 max-pool's wide loads against the definition, bit for bit: maps that end inside a window, one-pixel maps, widths that take the narrow
kernel, padding 0 to 2, values where a comparison decides nothing (NaN, equal values, both zeros)."""
import pytest
import torch

from test_gpu_ops import B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("n,h,w,c,stride,pad", [(2, 112, 111, 64, 2, 1), (3, 7, 8, 8, 2, 1), (1, 1, 1, 16, 1, 1), (2, 5, 9, 12, 1, 2), (2, 9, 5, 24, 3, 0),
                                                (1, 2, 30, 8, 2, 1)])
def test_three_by_three(n, h, w, c, stride, pad, dtype):
    gen = torch.Generator(device="cuda").manual_seed(h * w + c)
    x = torch.randn((n, h, w, c), generator=gen, device="cuda").to(dtype)
    x[:, h // 2, w // 2, 1] = float("nan")
    x[:, :, :, 2] = 0.0
    x[:, 0, :, 2] = -0.0
    x[:, :, :, 3] = -float("inf")
    ho, wo = (h + 2 * pad - 3) // stride + 1, (w + 2 * pad - 3) // stride + 1
    y = torch.full((n, ho, wo, c), 7.0, device="cuda", dtype=dtype)
    B().op_maxpool_fwd(x, y, 3, stride, pad)
    torch.cuda.synchronize()
    xc, want = x.cpu(), torch.empty((n, ho, wo, c), dtype=dtype)
    for p in range(ho):
        for q in range(wo):
            best = None
            for a in range(3):
                for b in range(3):
                    yy, xx = p * stride + a - pad, q * stride + b - pad
                    if 0 <= yy < h and 0 <= xx < w:
                        v = xc[:, yy, xx]
                        best = v.clone() if best is None else torch.where(v > best, v, best)
            want[:, p, q] = best
    bits = torch.int32 if dtype == torch.float32 else torch.int16
    assert torch.equal(y.cpu().view(bits), want.view(bits))
