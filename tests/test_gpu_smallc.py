"""GPU parity of the kernels for a handful of input channels (the first layer of a network), of the strip-wise max-pool
gradient and of the pooling kernels, at the sizes where they can go wrong.

Tolerance: as in test_gpu_x3.py for fp32 storage (2e-6 in the l2 norm); with bf16 storage 8e-3 for a stored bf16 result
(one rounding, 2^-9, plus the rounding of the oracle's own bf16 operands, which is none) and 1e-5 for the fp32 weight
gradient of bf16 operands, whose products are exact."""
import numpy as np
import pytest
import torch

import oracle as O
from test_gpu_ops import B, close, dev, nchw, nhwc, ohwi, rnd

pytestmark = pytest.mark.gpu

CASES = [  # n, h, w, cin, cout, r, stride, pad: at least 16384 output positions
    (6, 112, 112, 3, 64, 7, 2, 3),     # the stem
    (5, 131, 123, 3, 72, 7, 2, 3),     # odd sizes, a second block of output channels, ragged rows and columns
    (2, 97, 93, 3, 64, 3, 1, 1),       # VGG's first layer: odd word offsets
    (17, 33, 31, 1, 40, 5, 1, 2),      # one channel, columns that fill no block
    (9, 64, 70, 2, 16, 4, 1, 0),       # no padding
    (300, 8, 9, 3, 24, 3, 1, 1),       # images of one group of rows
    (3, 150, 600, 3, 32, 5, 2, 2),     # wide rows: fewer of them fit
]
# the same where the kernels for few channels take both storage types: f = forward, w = weight gradient in fp32 too (bf16: always)
TAKEN = [
    (26, 112, 112, 3, 64, 7, 2, 3, "fw"),
    (20, 131, 123, 3, 72, 7, 2, 3, "fw"),
    (12, 97, 93, 3, 64, 3, 1, 1, "f"),
    (29, 33, 40, 1, 40, 5, 1, 2, "f"),
    (18, 64, 70, 2, 16, 4, 1, 0, "f"),
    (150, 8, 41, 3, 24, 3, 1, 1, "f"),
    (8, 150, 600, 3, 32, 5, 2, 2, "f"),
    (34, 50, 49, 2, 40, 7, 1, 3, "fw"),
]


def bf16(a):
    return torch.from_numpy(np.ascontiguousarray(a)).bfloat16().float().numpy()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", CASES + TAKEN)
def test_small_channel_conv(case, dtype):
    n, h, w, cin, cout, r, stride, pad = case[:8]
    if len(case) > 8:
        kernel = lambda role: B().op_conv_kernel(role, *case[:8], B().F32 if dtype == "f32" else B().BF16)
        assert kernel("fwd") == "smallc" and (kernel("wgrad") == "smallc") == (dtype == "bf16" or "w" in case[8])
    x = rnd(1, n, cin, h, w)
    wt = rnd(2, cout, cin, r, r) * np.float32(np.sqrt(2.0 / (cin * r * r)))
    ho, wo = O.out_dim(h, r, stride, pad), O.out_dim(w, r, stride, pad)
    assert n * ho * wo >= 16384
    dy = rnd(3, n, cout, ho, wo)
    if dtype == "bf16":
        x, wt, dy = bf16(x), bf16(wt), bf16(dy)
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    y = torch.full((n, ho, wo, cout), float("nan"), device="cuda", dtype=td)
    B().op_conv_fwd(dev(nhwc(x)).to(td), dev(ohwi(wt)).to(td), y, stride, pad)
    ws = torch.empty(max(B().op_conv_workspace(n, h, w, cin, cout, r, stride, pad), 256), dtype=torch.uint8, device="cuda")
    dw = torch.full((cout, r, r, cin), float("nan"), device="cuda")
    B().op_conv_wgrad(dev(nhwc(x)).to(td), dev(nhwc(dy)).to(td), dw, stride, pad, ws)
    torch.cuda.synchronize()
    ref = O.conv_fwd(x, wt, stride, pad).astype(np.float64)
    err = np.linalg.norm(nchw(y.float().cpu().numpy()) - ref) / np.linalg.norm(ref)
    assert err <= (2e-6 if dtype == "f32" else 8e-3), err
    refw = O.conv_wgrad(x, dy, wt.shape, stride, pad).astype(np.float64)
    errw = np.linalg.norm(dw.cpu().numpy().transpose(0, 3, 1, 2) - refw) / np.linalg.norm(refw)
    assert errw <= (2e-6 if dtype == "f32" else 1e-5), errw


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", [CASES[0], TAKEN[0]])
def test_small_channel_conv_keeps_infinities_and_nan(case, dtype):
    """A non-finite input reaches exactly the outputs and the filter gradients that read it (the kernels also touch the
    values beside a window, times zeros)."""
    n, h, w, cin, cout, r, stride, pad = case[:8]
    x, wt = bf16(rnd(1, n, cin, h, w)), bf16(rnd(2, cout, cin, r, r))
    dy = bf16(rnd(3, n, cout, 56, 56))
    wt[:, 1] = 0.5
    x[1, 1, 20, 30] = np.inf
    x[2, 0, 111, 111] = np.nan
    x[4, 2, 0, 0] = -np.inf
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    y = torch.zeros((n, 56, 56, cout), device="cuda", dtype=td)
    B().op_conv_fwd(dev(nhwc(x)).to(td), dev(ohwi(wt)).to(td), y, stride, pad)
    ws = torch.empty(B().op_conv_workspace(n, h, w, cin, cout, r, stride, pad), dtype=torch.uint8, device="cuda")
    dw = torch.zeros((cout, r, r, cin), device="cuda")
    B().op_conv_wgrad(dev(nhwc(x)).to(td), dev(nhwc(dy)).to(td), dw, stride, pad, ws)
    torch.cuda.synchronize()
    with np.errstate(invalid="ignore", over="ignore"):
        ref = torch.nn.functional.conv2d(torch.from_numpy(x).double(), torch.from_numpy(wt).double(), stride=stride, padding=pad).numpy()
        cols = torch.nn.functional.unfold(torch.from_numpy(x).double(), r, padding=pad, stride=stride)
        refw = torch.einsum("ncp,nkp->ck", torch.from_numpy(dy).double().reshape(n, cout, -1), cols).reshape(wt.shape).numpy()
    for got, want in ((nchw(y.float().cpu().numpy()), ref), (dw.cpu().numpy().transpose(0, 3, 1, 2), refw)):
        assert np.isnan(want).any()
        assert np.array_equal(np.isnan(got), np.isnan(want))
        assert np.array_equal(np.where(np.isinf(want), got, 0), np.where(np.isinf(want), want, 0).astype(got.dtype))
        ok = np.isfinite(want)
        assert np.abs(got[ok] - want[ok]).max() <= 2e-2 * np.abs(want[ok]).max()


# n, c, h, w; then strips of two, four, eight (fp32) blocks: 200 thousand, 0.55 million, 1.4 million blocks of 2 x 2
@pytest.mark.parametrize("shape", [(2, 8, 33, 17), (1, 4, 3, 3), (3, 20, 16, 31), (2, 4, 1, 6), (1, 64, 37, 2),
                                   (42, 128, 33, 17), (121, 128, 35, 15), (290, 128, 33, 17), (1300, 64, 3, 31)])
@pytest.mark.parametrize("accumulate", [False, True])
def test_maxpool_gradient_in_strips(shape, accumulate):
    """Heights around the length of a strip, maps of one row or column of blocks, ties."""
    n, c, h, w = shape
    x = np.round(rnd(11, n, c, h, w) * 2) / np.float32(2)
    y, arg = O.maxpool_fwd(x, 3, 2, 1)
    dy = rnd(12, *y.shape)
    base = rnd(13, n, c, h, w)
    dx = dev(nhwc(base)) if accumulate else torch.full((n, h, w, c), float("nan"), device="cuda")
    B().op_maxpool_bwd(dev(nhwc(x)), dev(nhwc(dy)), dx, 3, 2, 1, accumulate=accumulate)
    torch.cuda.synchronize()
    ref = O.maxpool_bwd(dy, arg, x.shape).astype(np.float64) + (base if accumulate else 0.0)
    close(nchw(dx.cpu().numpy()), ref, f"maxpool_bwd {shape}", 1e-6)
    if not accumulate:      # bf16: sums of up to four values, rounded once
        x16, dy16 = dev(nhwc(x)).bfloat16(), dev(nhwc(dy)).bfloat16()
        dx16 = torch.full((n, h, w, c), float("nan"), device="cuda", dtype=torch.bfloat16)
        B().op_maxpool_bwd(x16, dy16, dx16, 3, 2, 1)
        ref = O.maxpool_bwd(nchw(dy16.float().cpu().numpy()), arg, x.shape)      # (the halves of x are exact in bf16)
        torch.cuda.synchronize()
        assert np.abs(nchw(dx16.float().cpu().numpy()) - ref).max() <= 2.0 ** -8 * np.abs(ref).max()


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("case", [(2, 16, 16, 64), (3, 1, 1, 8), (2, 9, 5, 1032), (5, 3, 3, 6), (1, 40, 31, 4)])
def test_pooling_mean_wide_and_narrow(case, offset):
    """Four channels at a time, and channel counts or addresses (offset: elements) that do not allow it."""
    n, h, w, c = case
    x = rnd(14, n, c, h, w)
    xt = torch.empty(x.size + offset, device="cuda")[offset:].view(n, h, w, c).copy_(dev(nhwc(x)))
    y = torch.full((n * c + offset,), float("nan"), device="cuda")[offset:].view(n, c)
    B().op_gap_fwd(xt, y)
    dx = torch.full((n * h * w * c + offset,), 2.0, device="cuda")[offset:].view(n, h, w, c)
    B().op_gap_bwd(y, dx, accumulate=True)
    torch.cuda.synchronize()
    ref = O.gap_fwd(x)
    close(y.cpu().numpy(), ref, f"gap_fwd {case}", 1e-6 * 4)
    close(nchw(dx.cpu().numpy()), O.gap_bwd(ref.reshape(n, c), x.shape).astype(np.float64) + 2.0, f"gap_bwd {case}", 1e-6)


@pytest.mark.parametrize("scales", [(-116, 90), (-140, 110), (90, -116), (100, -130)])
@pytest.mark.parametrize("case", TAKEN[:2])
def test_small_channel_conv_tiny_operands(case, scales):
    """fp32 operands whose lowest bits lie below the smallest bf16 are held in all their bits."""
    n, h, w, cin, cout, r, stride, pad = case[:8]
    ho, wo = O.out_dim(h, r, stride, pad), O.out_dim(w, r, stride, pad)
    small = lambda a, e: torch.from_numpy(np.ldexp(a.astype(np.float64), e).astype(np.float32))
    x, wt, dy = small(rnd(1, n, cin, h, w), scales[0]), small(rnd(2, cout, cin, r, r), scales[1]), small(rnd(3, n, cout, ho, wo), scales[1])
    y = torch.full((n, ho, wo, cout), float("nan"), device="cuda")
    B().op_conv_fwd(dev(nhwc(x.numpy())), dev(ohwi(wt.numpy())), y, stride, pad)
    ws = torch.empty(max(B().op_conv_workspace(n, h, w, cin, cout, r, stride, pad), 256), dtype=torch.uint8, device="cuda")
    dw = torch.full((cout, r, r, cin), float("nan"), device="cuda")
    B().op_conv_wgrad(dev(nhwc(x.numpy())), dev(nhwc(dy.numpy())), dw, stride, pad, ws)
    torch.cuda.synchronize()
    ref = torch.nn.functional.conv2d(x.double(), wt.double(), stride=stride, padding=pad)
    cols = torch.nn.functional.unfold(x.double(), r, padding=pad, stride=stride)
    refw = sum(d @ c.t() for d, c in zip(dy.double().reshape(n, cout, -1), cols)).reshape(wt.shape)
    got, gotw = torch.from_numpy(nchw(y.cpu().numpy())).double(), dw.cpu().double().permute(0, 3, 1, 2)
    assert ((got - ref).norm() / ref.norm()).item() <= 2e-6
    assert ((gotw - refw).norm() / refw.norm()).item() <= 2e-6


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("n,hw", [(2 ** 24 + 3, 1), (2 ** 20 + 1, 2)])
def test_pooling_mean_of_many_images(n, hw, dtype):
    """More images than a launch may have workgroups; whole numbers, exact."""
    x = torch.randint(-8, 9, (n, 1, hw, 4), device="cuda").to(dtype) * hw
    y = torch.full((n, 4), float("nan"), device="cuda", dtype=dtype)
    B().op_gap_fwd(x, y)
    dx = torch.full_like(x, 2.0)
    B().op_gap_bwd(y * hw, dx, accumulate=True)
    torch.cuda.synchronize()
    mean = (x.float().sum((1, 2)) / hw).to(dtype)
    assert torch.equal(y, mean)
    assert torch.equal(dx, (2.0 + mean.float())[:, None, None, :].expand(n, 1, hw, 4).to(dtype))
