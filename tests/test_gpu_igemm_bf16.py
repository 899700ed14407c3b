"""GPU parity of the bf16 convolutions at the sizes where their kernels can go wrong: ragged row and column tiles, widths
that end inside a chunk of K or span two taps with it, reductions that deal unevenly to the groups of waves or leave
some without a chunk, strided gathers and scattered results, accumulation (the tilings that these data gradients do not reach:
test_gpu_igemm_bf16_taps.py, which names them for both directions).

Tolerance: the operands are bf16 on both sides and their products exact in fp32; the result is rounded once to bf16 (eight
significant bits: 2^-8 of a value at most, 2^-8 / sqrt(3) = 2.3e-3 in the l2 norm if every value were the worst one of its
binade), the fp32 sums add less than 1e-5 of it."""
import numpy as np
import pytest
import torch

import oracle as O
from test_gpu_ops import B, dev, nchw, nhwc, ohwi, rnd

KERNELS = ["256x256", "128x256", "256x128", "128x128", "128x64", "64x64", "64x64, four stages", "64x64, four pairs", "64x64, four waves",
           "32x32, eight waves"]
# n, h, w, cin, cout, r, stride, kernel of the forward pass (None: whichever)
CASES = [
    (22, 31, 29, 64, 528, 1, 1, "256x256"),
    (87, 21, 18, 72, 136, 1, 1, "256x256"),          # 72 channels: a chunk of 64 and a part
    (66, 14, 15, 200, 200, 3, 1, None),              # 1800 values of K: 28 chunks and a part, most of them across two taps
    (99, 17, 14, 192, 144, 1, 1, "128x256"),
    (35, 16, 13, 72, 528, 1, 1, "128x256"),
    (48, 36, 33, 64, 272, 1, 1, "256x128"),
    (17, 38, 35, 32, 16, 1, 1, "256x128"),
    (94, 36, 36, 64, 8, 1, 1, "128x128"),
    (18, 38, 35, 72, 136, 1, 1, "128x128"),
    (17, 38, 35, 64, 16, 1, 1, "128x64"),
    (80, 26, 26, 104, 8, 1, 1, "128x64"),
    (2, 9, 6, 64, 8, 1, 1, "64x64"),
    (1, 9, 8, 72, 32, 1, 1, "64x64"),
    (12, 25, 25, 320, 8, 1, 1, "64x64, four stages"),
    (75, 13, 11, 120, 8, 1, 1, "64x64, four stages"),
    (15, 27, 27, 256, 8, 3, 1, "64x64, four pairs"),
    (52, 15, 13, 272, 8, 3, 1, "64x64, four pairs"),
    (47, 14, 14, 128, 8, 3, 1, "64x64, four waves"),
    (45, 18, 17, 32, 8, 1, 1, "64x64, four waves"),   # one chunk: three waves of four have none
    (3, 5, 5, 192, 16, 1, 1, "32x32, eight waves"),   # six chunks for eight waves
    (2, 7, 7, 328, 40, 3, 1, "32x32, eight waves"),
    (1, 8, 5, 48, 8, 1, 1, "32x32, eight waves"),
    (6, 15, 17, 72, 88, 3, 2, None),                  # strided: data gradient in four parts
    (5, 20, 21, 96, 40, 1, 2, None),                  # strided 1x1: scattered result
    (2, 11, 10, 40, 48, 5, 1, None),
]


def test_every_kernel_is_reached():
    got = [B().op_conv_kernel("fwd", n, h, w, cin, cout, r, stride, r // 2, B().BF16) for n, h, w, cin, cout, r, stride, _ in CASES]
    assert [g if c[7] else None for g, c in zip(got, CASES)] == ["igemm_bf16 " + c[7] if c[7] else None for c in CASES]
    assert set(g for g in got) == set("igemm_bf16 " + k for k in KERNELS)


def bf16(a):
    return torch.from_numpy(a).bfloat16().float().numpy()


def close(got, ref, what):
    err = np.linalg.norm(got.astype(np.float64) - ref) / np.linalg.norm(ref.astype(np.float64))
    assert err <= 2.3e-3, (what, err)
    assert np.abs(got - ref).max() <= 2.0 ** -8 * np.abs(ref).max(), what


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES)
def test_bf16_conv(case):
    n, h, w, cin, cout, r, stride = case[:7]
    pad = r // 2
    x = bf16(rnd(1, n, cin, h, w))
    wt = bf16(rnd(2, cout, cin, r, r) * np.float32(np.sqrt(2.0 / (cin * r * r))))
    ref = O.conv_fwd(x, wt, stride, pad)
    y = torch.full((n, ref.shape[2], ref.shape[3], cout), float("nan"), device="cuda", dtype=torch.bfloat16)
    B().op_conv_fwd(dev(nhwc(x)).bfloat16(), dev(ohwi(wt)).bfloat16(), y, stride, pad)
    torch.cuda.synchronize()
    close(nchw(y.float().cpu().numpy()), ref, f"conv_fwd {case}")


@pytest.mark.gpu
@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("case", CASES)
def test_bf16_dgrad(case, accumulate):
    n, h, w, cin, cout, r, stride = case[:7]
    pad = r // 2
    wt = bf16(rnd(2, cout, cin, r, r) * np.float32(np.sqrt(2.0 / (cin * r * r))))
    dy = bf16(rnd(3, n, cout, O.out_dim(h, r, stride, pad), O.out_dim(w, r, stride, pad)))
    base = bf16(rnd(4, n, cin, h, w)) if accumulate else np.zeros((n, cin, h, w), np.float32)
    ref = O.conv_dgrad(dy, wt, (n, cin, h, w), stride, pad).astype(np.float64) + base
    ws = torch.empty(max(B().op_conv_workspace(n, h, w, cin, cout, r, stride, pad), 256), dtype=torch.uint8, device="cuda")
    dx = dev(nhwc(base)).bfloat16() if accumulate else torch.full((n, h, w, cin), float("nan"), device="cuda", dtype=torch.bfloat16)
    B().op_conv_dgrad(dev(nhwc(dy)).bfloat16(), dev(ohwi(wt)).bfloat16(), dx, stride, pad, ws, accumulate)
    torch.cuda.synchronize()
    close(nchw(dx.float().cpu().numpy()), ref, f"conv_dgrad {case}")
