"""GPU parity of bf16 convolutions whose last rows run in lower tiles behind those of 256 x 256: one and several columns of tiles, a last tile
that is nearly empty, nearly full and whole, whole and ragged chunks, strided and scattered results, accumulation, bias + ReLU.

Tolerances as for the other tilings: one rounding of the result to bf16."""
import pytest
import torch

import test_gpu_igemm_bf16_taps as T
from test_gpu_ops import B

# n, h, w, channels reduced over, channels of the result, height of the lower tiles
CASES = [
    (90, 30, 30, 128, 136, 64),         # 65536 rows and 241 tiles of 64 and a piece
    (73, 30, 30, 136, 248, 64),         # 164 rows
    (110, 30, 30, 136, 256, 192),      # 33464 = 174 * 192 + 56
    (128, 28, 28, 256, 256, 192),       # 30464 = 158 * 192 + 128
    (60, 29, 29, 200, 504, 192),        # two columns of tiles
    (80, 30, 30, 128, 504, 64),
    (50, 26, 26, 160, 768, 192),        # three
    (220, 28, 28, 128, 136, 192),       # two rounds of 192 behind one of 256
]


def name(low):
    return f"igemm_bf16 256x256 and {low}x256"


@pytest.mark.parametrize("case", CASES)
def test_routes(case):
    n, h, w, c, m, low = case
    assert B().op_conv_kernel("fwd", n, h, w, c, m, 3, 1, 1, B().BF16) == name(low)
    assert B().op_conv_kernel("dgrad", n, h, w, m, c, 3, 1, 1, B().BF16) == name(low)


def test_routes_one_height():
    # a round that is full, less than one round, results that wait for memory, fewer than 3 % of many rounds saved
    for case in ((128, 16, 32, 128, 256, 3), (60, 32, 32, 128, 256, 3), (128, 56, 56, 64, 256, 1), (164, 54, 52, 1024, 768, 1),
                 (164, 42, 44, 1024, 1208, 1)):
        n, h, w, c, m, r = case
        assert B().op_conv_kernel("fwd", n, h, w, c, m, r, 1, r // 2, B().BF16) == "igemm_bf16 256x256", case


def test_routes_of_measured_layers():
    for case, low in (((512, 14, 14, 256, 256, 3), 192), ((200, 28, 28, 256, 256, 3), 192), ((256, 28, 28, 128, 256, 3), 64),
                      ((128, 28, 28, 1024, 512, 1), 64)):
        n, h, w, c, m, r = case
        assert B().op_conv_kernel("fwd", n, h, w, c, m, r, 1, r // 2, B().BF16) == name(low), case


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES)
def test_forward_and_data_gradient(case):
    T.test_forward_and_data_gradient(case)


@pytest.mark.gpu
@pytest.mark.parametrize("case", [CASES[1], CASES[4]])
def test_bias_and_relu_in_the_launch(case):
    T.test_bias_and_relu_in_the_launch(case, True)


@pytest.mark.gpu
@pytest.mark.parametrize("n,h,w,low", [(130, 56, 56, 192), (92, 55, 56, 64)])
def test_strided(n, h, w, low):
    """3x3 stride 2: the forward pass jumps over pixels, a part of the data gradient writes every second one."""
    c = m = 256
    p, q = (h + 1) // 2, (w + 1) // 2
    assert B().op_conv_kernel("fwd", n, h, w, c, m, 3, 2, 1, B().BF16) == name(low)
    x, wt, dy = T.randn(1, (n, h, w, c)), T.randn(2, (m, 3, 3, c), (2.0 / (9 * c)) ** 0.5), T.randn(3, (n, p, q, m))
    y = torch.full((n, p, q, m), float("nan"), device="cuda", dtype=torch.bfloat16)
    B().op_conv_fwd(x, wt, y, 2, 1)
    T.close(y, T.conv64(x, wt)[:, ::2, ::2])
    ws = torch.empty(B().op_conv_workspace(n, h, w, c, m, 3, 2, 1), dtype=torch.uint8, device="cuda")
    dx = torch.full((n, h, w, c), float("nan"), device="cuda", dtype=torch.bfloat16)
    B().op_conv_dgrad(dy, wt, dx, 2, 1, ws)
    spread = torch.zeros((n, h, w, m), device="cuda", dtype=torch.bfloat16)
    spread[:, ::2, ::2] = dy
    T.close(dx, T.conv64(spread, wt.flip(1, 2).permute(3, 1, 2, 0).contiguous()))
