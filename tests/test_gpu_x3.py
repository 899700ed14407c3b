"""GPU parity of the fp32 convolutions on the bf16 matrix cores (every value split into three bf16 parts, see split3.h) at the
sizes where their kernels can go wrong: ragged row and column tiles, reductions that deal unevenly to the groups
of waves, windows of the largest width, one-chunk reductions; and values the split cannot represent.

Tolerance: the parts left out of a product are below 2^-25 of it, and a result is rounded 6 times per 16 products,
at most 6 * K / 16 * 2^-24 of the sum of magnitudes (K = 3024: 7e-5) if every rounding went the same way; they do
not, and 2e-6 in the l2 norm is what the fp32 matrix instruction (up to 8e-7 measured) stays below as well."""
import numpy as np
import pytest
import torch

import oracle as O
from test_gpu_ops import B, close, dev, nchw, nhwc, ohwi, rnd

pytestmark = pytest.mark.gpu

X128, X64, D2x1, D2x2, D1x1 = "igemm_x3 128x128", "igemm_x3 64x64", "igemm_x3_deep 128x64", "igemm_x3_deep 128x128", "igemm_x3_deep 64x64"
WINDOW, PARTS, GENERIC = "igemm_x3_deep window 128x64", "igemm_x3_parts 64x64", "igemm generic 64x64"
DIRECT, DIRECT2 = "igemm direct 64x64", "igemm direct 64x64, two groups"
# n, h, w, cin, cout, r, stride, the kernels of the forward pass and of the data gradient (test_conv_routes.py holds them to it)
CASES = [
    (41, 14, 14, 144, 1000, 1, 1, X128, D2x1),     # ragged rows and columns, nine steps
    (13, 31, 30, 112, 264, 1, 1, X64, X64),        # seven steps
    (7, 9, 9, 16, 24, 1, 1, X64, X64),             # a single step
    (5, 61, 62, 64, 144, 3, 1, WINDOW, WINDOW),    # window of the largest width (61 x 62 map: 254 of 256 rows)
    (23, 14, 14, 336, 272, 3, 1, WINDOW, WINDOW),  # window, 189 steps over four groups (48 + 47 + 47 + 47)
    (30, 14, 14, 528, 136, 1, 1, D2x1, D2x2),      # four groups of waves, 33 steps
    (20, 28, 28, 272, 250, 1, 1, D2x2, GENERIC),   # two groups of waves, 17 steps
    (3, 62, 64, 64, 144, 3, 1, D2x2, D1x1),        # 3x3 on a map too wide for the window
    (9, 31, 29, 80, 80, 3, 1, D1x1, D1x1),         # eight groups of one wave, 45 steps
    (6, 15, 17, 48, 48, 3, 2, D1x1, PARTS),        # strided: forward gathers, data gradient in four parts
    (2, 11, 10, 16, 48, 5, 1, D1x1, D1x1),         # 5x5 taps
    (41, 1, 1, 516, 1000, 1, 1, D1x1, D1x1),       # fully connected: both reductions end inside a step (516 = 32 * 16 + 4, 1000 = 62 * 16 + 8)
    (9, 12, 11, 20, 260, 1, 1, X64, D1x1),         # the same with 64 x 64 tiles
    (64, 14, 14, 148, 620, 1, 1, X128, D2x2),      # and with 128 x 128 tiles
    (60, 28, 27, 144, 272, 3, 2, D2x1, PARTS),     # strided gather in four groups of waves
    (11, 20, 20, 272, 144, 3, 1, D1x1, WINDOW),
    # launches that stay with the fp32 instruction
    (2, 56, 55, 256, 72, 1, 1, DIRECT2, X64),      # ragged rows and columns, two groups of waves
    (13, 40, 40, 96, 64, 1, 1, DIRECT, DIRECT),
    (1, 9, 9, 64, 64, 3, 1, DIRECT2, DIRECT2),
]


@pytest.mark.parametrize("case", CASES)
def test_split_conv(case):
    n, h, w, cin, cout, r, stride = case[:7]
    pad = r // 2
    x = rnd(1, n, cin, h, w)
    wt = rnd(2, cout, cin, r, r) * np.float32(np.sqrt(2.0 / (cin * r * r)))
    ref = O.conv_fwd(x, wt, stride, pad)
    y = torch.full((n, ref.shape[2], ref.shape[3], cout), float("nan"), device="cuda")
    B().op_conv_fwd(dev(nhwc(x)), dev(ohwi(wt)), y, stride, pad)
    torch.cuda.synchronize()
    close(nchw(y.cpu().numpy()), ref, f"conv_fwd {case}", 2e-6 * 4)
    err = np.linalg.norm(nchw(y.cpu().numpy()).astype(np.float64) - ref) / np.linalg.norm(ref.astype(np.float64))
    assert err <= 2e-6, err


@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("case", CASES)
def test_split_dgrad(case, accumulate):
    n, h, w, cin, cout, r, stride = case[:7]
    pad = r // 2
    wt = rnd(2, cout, cin, r, r) * np.float32(np.sqrt(2.0 / (cin * r * r)))
    dy = rnd(3, n, cout, O.out_dim(h, r, stride, pad), O.out_dim(w, r, stride, pad))
    base = rnd(4, n, cin, h, w) if accumulate else np.zeros((n, cin, h, w), np.float32)
    refd = O.conv_dgrad(dy, wt, (n, cin, h, w), stride, pad).astype(np.float64) + base
    ws = torch.empty(max(B().op_conv_workspace(n, h, w, cin, cout, r, stride, pad), 256), dtype=torch.uint8, device="cuda")
    dx = dev(nhwc(base)) if accumulate else torch.full((n, h, w, cin), float("nan"), device="cuda")
    B().op_conv_dgrad(dev(nhwc(dy)), dev(ohwi(wt)), dx, stride, pad, ws, accumulate)
    torch.cuda.synchronize()
    err = np.linalg.norm(nchw(dx.cpu().numpy()).astype(np.float64) - refd) / np.linalg.norm(refd)
    assert err <= 2e-6, err


@pytest.mark.parametrize("case", [CASES[i] for i in (1, 4, 6, 8, 12)])
def test_split_conv_keeps_infinities_nan_and_the_largest_values(case):
    """As the fp32 instruction: an infinity times a nonzero weight is an infinity (also where a part of the weight
    is zero), a NaN stays in the outputs that read it, values next to the largest finite one do not overflow."""
    n, h, w, cin, cout, r, stride = case[:7]
    pad = r // 2
    x = rnd(1, n, cin, h, w)
    wt = rnd(2, cout, cin, r, r) * np.float32(np.sqrt(2.0 / (cin * r * r)))
    wt[:, 3] = 0.5                                    # exact in one bf16: its other parts are zero
    x[0, 3, 2, 1] = np.inf
    x[n - 1, 3, h - 1, w - 1] = -np.inf
    x[n // 2, cin - 1, 3, 4] = np.nan
    x[n // 2, 3, h - 2, 2] = np.float32(3.4028e38)    # rounds to an infinite bf16; times 0.5 it is finite
    with np.errstate(invalid="ignore", over="ignore"):
        ref = torch.nn.functional.conv2d(torch.from_numpy(x).double(), torch.from_numpy(wt).double(), stride=stride,
                                         padding=pad).numpy()
    y = torch.zeros((n, ref.shape[2], ref.shape[3], cout), device="cuda")
    B().op_conv_fwd(dev(nhwc(x)), dev(ohwi(wt)), y, stride, pad)
    torch.cuda.synchronize()
    got = nchw(y.cpu().numpy()).astype(np.float64)
    assert np.isinf(ref).any() and np.isnan(ref).any() and (np.abs(ref[np.isfinite(ref)]) > 1e38).any()
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(np.where(np.isinf(ref), got, 0.0), np.where(np.isinf(ref), ref, 0.0))
    ok = np.isfinite(ref)
    scale = np.maximum(np.abs(ref[ok]), 1.0)
    assert (np.abs(got[ok] - ref[ok]) / scale).max() <= 1e-4


WX64, WX128, WDIRECT = "wgrad_x3 64x64", "wgrad_x3 128x128", "wgrad direct 64x64"
WGRAD_CASES = [  # n, h, w, cin, cout, r, stride, kernel
    (9, 13, 11, 132, 260, 1, 1, WX64),       # ragged tiles
    (7, 14, 14, 36, 44, 3, 1, WX64),         # channels that fill no block, taps that change inside one
    (2, 9, 9, 60, 64, 1, 1, WX64),           # 162 positions: the fewest this kernel takes
    (5, 21, 3, 32, 40, 3, 1, WX64),          # rows of three positions: several wraps inside a thread's four
    (11, 2, 20, 32, 32, 3, 1, WX64),         # images of two rows
    (6, 31, 29, 48, 20, 3, 2, WX64),         # strided gather
    (60, 28, 28, 68, 260, 1, 2, WX64),       # strided 1x1
    (23, 14, 14, 256, 256, 3, 1, WX128),     # several parts, a ragged last step
    (64, 28, 27, 260, 268, 1, 1, WX128),     # ragged 128 x 128 tiles
    (30, 27, 29, 132, 260, 3, 2, WX128),     # the same, strided, channels that fill no block
    # small layers that stay with the fp32 instruction
    (2, 9, 9, 64, 64, 1, 1, WDIRECT),
    (9, 21, 3, 64, 44, 3, 1, WDIRECT),       # rows of three positions
    (3, 28, 27, 64, 252, 1, 2, WDIRECT),     # strided
    (2, 31, 29, 128, 68, 3, 2, WDIRECT),
]


def wgrad(case, x, dy):
    n, h, w, cin, cout, r, stride = case[:7]
    ws = torch.empty(max(B().op_conv_workspace(n, h, w, cin, cout, r, stride, r // 2), 256), dtype=torch.uint8, device="cuda")
    dw = torch.full((cout, r, r, cin), float("nan"), device="cuda")
    B().op_conv_wgrad(dev(nhwc(x)), dev(nhwc(dy)), dw, stride, r // 2, ws)
    torch.cuda.synchronize()
    return dw.cpu().numpy().transpose(0, 3, 1, 2).astype(np.float64)


@pytest.mark.parametrize("case", WGRAD_CASES)
def test_split_wgrad(case):
    n, h, w, cin, cout, r, stride = case[:7]
    x = rnd(1, n, cin, h, w)
    dy = rnd(3, n, cout, O.out_dim(h, r, stride, r // 2), O.out_dim(w, r, stride, r // 2))
    ref = O.conv_wgrad(x, dy, (cout, cin, r, r), stride, r // 2).astype(np.float64)
    got = wgrad(case, x, dy)
    assert np.linalg.norm(got - ref) <= 2e-6 * np.linalg.norm(ref)
    assert np.abs(got - ref).max() <= 1e-5 * np.abs(ref).max()


@pytest.mark.parametrize("case", [WGRAD_CASES[i] for i in (0, 1, 7)])
def test_split_wgrad_keeps_infinities_nan_and_the_largest_values(case):
    n, h, w, cin, cout, r, stride = case[:7]
    x = rnd(1, n, cin, h, w)
    dy = rnd(3, n, cout, O.out_dim(h, r, stride, r // 2), O.out_dim(w, r, stride, r // 2))
    dy[0, 5] = 0.25                                   # exact in one bf16
    x[0, 7, 1, 1] = np.inf
    x[n - 1, 3, h - 1, 2] = np.nan
    x[0, 9, 1, 2] = np.float32(3.4028e38)
    dy[:, 8:] = np.where(np.abs(dy[:, 8:]) > 0.9, 0.9, dy[:, 8:])
    xt, dt = torch.from_numpy(x).double(), torch.from_numpy(dy).double()
    cols = torch.nn.functional.unfold(xt, r, padding=r // 2, stride=stride)          # [n, cin*r*r, positions]
    with np.errstate(invalid="ignore", over="ignore"):
        ref = torch.einsum("ncp,nkp->ck", dt.reshape(n, cout, -1), cols).reshape(cout, cin, r, r).numpy()
    got = wgrad(case, x, dy)
    fit = np.abs(np.where(np.isfinite(ref), ref, 0.0)) < 3.3e38                      # the others overflow or not by their order
    assert np.isinf(ref).any() and np.isnan(ref).any()
    assert np.array_equal(np.isnan(got[fit]), np.isnan(ref[fit]))
    inf = np.isinf(ref) & fit
    assert np.array_equal(got[inf], ref[inf])
    ok = np.isfinite(ref) & fit & (np.abs(ref) < 1e30)
    assert np.abs(got[ok] - ref[ok]).max() <= 1e-4 * np.abs(ref[ok]).max()


# Operands whose lowest bits lie below the smallest bf16 (2^-133), subnormal ones among them, against others that bring the result
# back into range: held in all their bits as before.  One operand at a time, then results far below one.
TINY = [(-116, 90), (-124, 100), (-140, 110), (90, -116), (100, -130), (-50, -60)]


@pytest.mark.parametrize("scales", TINY)
@pytest.mark.parametrize("case", [CASES[i] for i in (0, 1, 4, 5, 6, 8, 9)])
def test_split_conv_tiny_operands(case, scales):
    n, h, w, cin, cout, r, stride = case[:7]
    n, pad = min(n, 12), r // 2
    x = torch.ldexp(torch.from_numpy(rnd(1, n, cin, h, w)).double(), torch.tensor(scales[0])).float()
    wt = torch.ldexp(torch.from_numpy(rnd(2, cout, cin, r, r)).double() * (2.0 / (cin * r * r)) ** 0.5, torch.tensor(scales[1])).float()
    ref = torch.nn.functional.conv2d(x.double(), wt.double(), stride=stride, padding=pad)
    y = torch.full((n, ref.shape[2], ref.shape[3], cout), float("nan"), device="cuda")
    B().op_conv_fwd(dev(nhwc(x.numpy())), dev(ohwi(wt.numpy())), y, stride, pad)
    torch.cuda.synchronize()
    got = torch.from_numpy(nchw(y.cpu().numpy())).double()
    assert ((got - ref).norm() / ref.norm()).item() <= 2e-6


@pytest.mark.parametrize("scales", TINY)
@pytest.mark.parametrize("case", [WGRAD_CASES[i] for i in (0, 1, 7)])
def test_split_wgrad_tiny_operands(case, scales):
    n, h, w, cin, cout, r, stride = case[:7]
    x = np.ldexp(rnd(1, n, cin, h, w).astype(np.float64), scales[0]).astype(np.float32)
    dy = np.ldexp(rnd(3, n, cout, O.out_dim(h, r, stride, r // 2), O.out_dim(w, r, stride, r // 2)).astype(np.float64), scales[1]).astype(np.float32)
    cols = torch.nn.functional.unfold(torch.from_numpy(x).double(), r, padding=r // 2, stride=stride)
    ref = sum(d @ c.t() for d, c in zip(torch.from_numpy(dy).double().reshape(n, cout, -1), cols)).reshape(cout, cin, r, r).numpy()
    got = wgrad(case, x, dy)
    assert np.linalg.norm(got - ref) <= 2e-6 * np.linalg.norm(ref)


@pytest.mark.parametrize("case,parts", [(WGRAD_CASES[7], 3), ((64, 14, 14, 132, 260, 1, 1, WX128), 49)])
def test_split_wgrad_in_the_least_workspace(case, parts):
    """More parts are taken where the workspace holds them; the fewest (those of the fp32 kernel's launch, one round of workgroups) are
    enough, and less is refused."""
    n, h, w, cin, cout, r, stride = case[:7]
    x, dy = rnd(1, n, cin, h, w), rnd(3, n, cout, O.out_dim(h, r, stride, r // 2), O.out_dim(w, r, stride, r // 2))
    ref = O.conv_wgrad(x, dy, (cout, cin, r, r), stride, r // 2).astype(np.float64)
    least = parts * cout * cin * r * r * 4
    ws = torch.empty(least, dtype=torch.uint8, device="cuda")
    dw = torch.full((cout, r, r, cin), float("nan"), device="cuda")
    B().op_conv_wgrad(dev(nhwc(x)), dev(nhwc(dy)), dw, stride, r // 2, ws)
    torch.cuda.synchronize()
    assert np.linalg.norm(dw.cpu().numpy().transpose(0, 3, 1, 2) - ref) <= 2e-6 * np.linalg.norm(ref)
    with pytest.raises(B().AccError):
        B().op_conv_wgrad(dev(nhwc(x)), dev(nhwc(dy)), dw, stride, r // 2, ws[: least - 16])
