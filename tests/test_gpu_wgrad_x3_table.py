"""GPU parity of the fp32 weight gradient where a wave works out the offsets of 64 positions at a time (64 channels of one filter tap): maps smaller
than 64 positions (a position's successor lies images further on), maps of one row or column, strides, paddings, filters of every
kind, ranges of positions that end inside a group of 64, output channels that fill no block, 1x1 strided filters of any width.

Tolerance: six of the nine bf16 products of the parts of two fp32 values, the rest below 2^-25 of the product, fp32 sums: less than 1e-5 of the l2
norm; whole numbers below 2^24 are exact in any order."""
import pytest
import torch

# n, h, w, cin, cout, r, stride, pad
CASES = [
    (4, 28, 28, 128, 128, 3, 1, 1),
    (41, 14, 14, 64, 136, 3, 1, 1),
    (85, 7, 7, 128, 256, 3, 1, 1),          # 49 positions
    (510, 2, 3, 192, 64, 3, 1, 1),          # six
    (4501, 1, 1, 64, 128, 3, 1, 1),          # one
    (50, 1, 97, 64, 100, 3, 1, 1),
    (12, 101, 1, 64, 68, 3, 1, 1),
    (17, 29, 31, 64, 260, 3, 2, 1),
    (75, 15, 14, 128, 64, 5, 3, 2),
    (119, 13, 12, 64, 64, 2, 1, 1),
    (1275, 9, 8, 64, 72, 3, 4, 0),
    (12, 27, 28, 256, 512, 1, 2, 0),
    (30, 19, 17, 100, 68, 1, 2, 0),         # no whole block of 64 channels, one tap all the same
    (30, 19, 17, 36, 132, 1, 3, 0),
    (57, 17, 11, 64, 64, 3, 1, 1),          # 10659 positions
]


def b():
    from paper_1901_06773_amd import binding
    return binding


@pytest.mark.parametrize("case", CASES)
def test_routes(case):
    assert b().op_conv_kernel("wgrad", *case, b().F32).startswith("wgrad_x3"), case


@pytest.mark.gpu
@pytest.mark.parametrize("whole", [False, True])
@pytest.mark.parametrize("case", CASES)
def test_wgrad(case, whole):
    n, h, w, ci, co, r, st, pad = case
    ho, wo = (h + 2 * pad - r) // st + 1, (w + 2 * pad - r) // st + 1
    gen = torch.Generator(device="cuda").manual_seed(n * h + w + ci)

    def at_end(*shape):                      # NaN behind the operand
        t = torch.randint(-9, 10, shape, generator=gen, device="cuda").float() if whole else torch.randn(shape, generator=gen, device="cuda")
        buf = torch.full((t.numel() + 4096,), float("nan"), device="cuda")
        buf[:t.numel()] = t.reshape(-1)
        return buf[:t.numel()].view(shape)
    x, dy = at_end(n, h, w, ci), at_end(n, ho, wo, co)
    ws = torch.empty(b().op_conv_workspace(n, h, w, ci, co, r, st, pad), dtype=torch.uint8, device="cuda")
    dw = torch.full((co, r, r, ci), float("nan"), device="cuda")
    b().op_conv_wgrad(x, dy, dw, st, pad, ws)
    xp = torch.nn.functional.pad(x.double(), (0, 0, pad, pad, pad, pad))
    g = dy.double().reshape(-1, co).t().contiguous()
    ref = torch.empty(co, r, r, ci, dtype=torch.float64, device="cuda")
    for i in range(r):
        for j in range(r):
            ref[:, i, j] = g @ xp[:, i:i + (ho - 1) * st + 1:st, j:j + (wo - 1) * st + 1:st].reshape(-1, ci)
    if whole:
        assert torch.equal(dw.double(), ref)
    else:
        assert float((dw.double() - ref).norm() / ref.norm()) < 1e-5
