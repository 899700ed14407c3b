"""bf16 data gradients that read the layer's filter as it lies, w[c][r][s][n], instead of a flipped copy of it: every tiling, filters of every kind,
columns that fill no tile, 1x1 with a stride, accumulation.  The products and their order are those of a forward pass with the flipped
filter, so the bits are; and nothing is written to the workspace."""
import pytest
import torch

import test_gpu_igemm_bf16_taps as T
from test_gpu_igemm_bf16_heights import CASES as HEIGHTS

pytestmark = pytest.mark.gpu

# n, h, w, channels reduced over, channels of the result, filter, padding
CASES = [c[:5] + (3, 1) for c in T.CASES + HEIGHTS if c[3] % 64 == 0] + [
    (3, 9, 11, 64, 8, 1, 0), (64, 14, 14, 256, 1024, 1, 0), (1, 7, 7, 2048, 512, 1, 0), (2, 5, 6, 128, 40, 5, 2), (5, 8, 8, 192, 72, 2, 1),
    (4, 13, 7, 64, 200, 4, 1), (1, 3, 3, 320, 24, 5, 1), (6, 12, 12, 64, 16, 3, 0), (40, 28, 28, 512, 128, 1, 0), (9, 31, 30, 96, 64, 3, 1), (2, 6, 6, 32, 32, 3, 1),
]


def data_gradient(dy, w, h, wd, stride, pad, accumulate_to=None):
    n, c = dy.shape[0], w.shape[3]
    need = T.B().op_conv_workspace(n, h, wd, c, w.shape[0], w.shape[1], stride, pad)
    ws = torch.full((need,), 173, dtype=torch.uint8, device="cuda")
    dx = torch.full((n, h, wd, c), float("nan"), device="cuda", dtype=torch.bfloat16) if accumulate_to is None else accumulate_to.clone()
    T.B().op_conv_dgrad(dy, w, dx, stride, pad, ws, accumulate_to is not None)
    return dx, bool((ws == 173).all())


@pytest.mark.parametrize("case", CASES)
def test_the_bits_of_the_flipped_filter(case):
    n, h, w, c, m, r, pad = case
    p, q = h + 2 * pad - r + 1, w + 2 * pad - r + 1
    dy, wt = T.randn(1, (n, p, q, c)), T.randn(2, (c, r, r, m), (2.0 / (r * r * c)) ** 0.5)
    dx, untouched = data_gradient(dy, wt, h, w, 1, pad)
    back = wt.flip(1, 2).permute(3, 1, 2, 0).contiguous()
    want = torch.full((n, h, w, m), float("nan"), device="cuda", dtype=torch.bfloat16)
    T.B().op_conv_fwd(dy, back, want, 1, r - 1 - pad)
    assert torch.isfinite(want).all() and torch.equal(dx, want)
    if c % 64 == 0:                       # whole chunks whatever the tiling
        assert untouched
    base = T.randn(3, (n, h, w, m))
    got, _ = data_gradient(dy, wt, h, w, 1, pad, base)
    # one rounding here, one in `want`, each as large as T.close() allows
    ref = want.double() + base.double()
    d = got.double() - ref
    assert d.norm() <= 2 * 2.3e-3 * max(ref.norm(), want.double().norm()) and d.abs().max() <= 2 * 2.0 ** -8 * ref.abs().max()


@pytest.mark.parametrize("n,h,w,c,m,stride", [(4, 14, 14, 128, 64, 2), (3, 15, 13, 256, 72, 3), (33, 28, 28, 512, 256, 2)])
def test_1x1_with_a_stride(n, h, w, c, m, stride):
    p, q = (h - 1) // stride + 1, (w - 1) // stride + 1
    dy, wt = T.randn(1, (n, p, q, c)), T.randn(2, (c, 1, 1, m), (1.0 / c) ** 0.5)
    dx, untouched = data_gradient(dy, wt, h, w, stride, 0)
    ref = torch.zeros((n, h, w, m), dtype=torch.float64, device="cuda")
    ref[:, ::stride, ::stride] = (dy.double().reshape(-1, c) @ wt.double().view(c, m)).view(n, p, q, m)
    T.close(dx, ref)
    assert untouched and (dx[ref == 0] == 0).all()


def test_infinities_and_nan_stay_in_their_places():
    dy, wt = T.randn(1, (2, 8, 8, 64)), T.randn(2, (64, 3, 3, 40), 0.05)
    dy[0, 3, 4, 5] = float("inf")
    dy[1, 0, 0, 63] = float("nan")
    dx, _ = data_gradient(dy, wt, 8, 8, 1, 1)
    bad = ~torch.isfinite(dx).all(3)
    want = torch.zeros_like(bad)
    want[0, 2:5, 3:6] = True
    want[1, :2, :2] = True
    assert torch.equal(bad, want)
