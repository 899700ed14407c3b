"""Strided data gradients: one launch for the parts (64- and 128-wide tiles) or one for each, rows of positions shorter than the
epilogue's counting needs, more parts than one launch takes, positions without a tap; overwriting and accumulating."""
import pytest
import torch

pytestmark = pytest.mark.gpu

CASES = [  # n, h, w, cin, cout, r, stride, pad
    (3, 7, 8, 48, 32, 3, 2, 1),         # one launch; four positions a row: a division per row
    (5, 13, 11, 80, 48, 3, 2, 1),       # one launch; rows of six and five, ragged tiles both ways
    (96, 28, 27, 192, 256, 3, 2, 1),    # one launch, 64-wide tiles, many of them
    (45, 55, 54, 116, 112, 3, 2, 1),    # one launch, 128-wide tiles, ragged both ways
    (64, 14, 13, 960, 960, 3, 2, 1),    # long reductions: the parts on their own
    (4, 13, 14, 32, 32, 5, 3, 2),       # nine parts
    (2, 10, 9, 16, 32, 2, 3, 0),        # four parts, five classes of positions without a tap
    (4, 9, 9, 32, 20, 3, 2, 1),         # reductions that are not whole steps of 16: the per-element kernel
]


# the kernel of the fp32 calls (of the first part, where the parts run one by one)
KERNELS = ["igemm_x3_parts 64x64", "igemm_x3_parts 64x64", "igemm_x3_parts 64x64", "igemm_x3_parts 128x128", "igemm_x3_deep 128x128",
           "igemm_x3 64x64", "igemm_x3_parts 64x64", "igemm_x3 64x64"]


@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_strided_dgrad(case, dtype, accumulate):
    from paper_1901_06773_amd import binding as b
    n, h, w, cin, cout, r, stride, pad = case
    gen = torch.Generator().manual_seed(h * w + r)
    ho, wo = (h + 2 * pad - r) // stride + 1, (w + 2 * pad - r) // stride + 1
    dy = torch.randn(n, ho, wo, cout, generator=gen).to(dtype)
    wt = (torch.randn(cout, r, r, cin, generator=gen) * (2.0 / (cout * r * r)) ** 0.5).to(dtype)
    old = torch.randn(n, h, w, cin, generator=gen).to(dtype)
    dx = old.cuda() if accumulate else torch.full((n, h, w, cin), float("nan"), device="cuda", dtype=dtype)
    # (the workspace of the forward, data-gradient and weight-gradient calls of this shape)
    ws = torch.empty(max(b.op_conv_workspace(n, h, w, cin, cout, r, stride, pad), cin * cout * r * r * 4 + 256 * 16), dtype=torch.uint8,
                     device="cuda")
    b.op_conv_dgrad(dy.cuda(), wt.cuda(), dx, stride, pad, ws, accumulate)
    torch.cuda.synchronize()
    ref = torch.nn.grad.conv2d_input((n, cin, h, w), wt.double().permute(0, 3, 1, 2).contiguous(),
                                     dy.double().permute(0, 3, 1, 2).contiguous(), stride, pad).permute(0, 2, 3, 1)
    if accumulate:
        ref = ref + old.double()
    err = ((dx.cpu().double() - ref).norm() / ref.norm()).item()
    # fp32: 2e-6 in the l2 norm, above what the fp32 matrix instruction shows (up to 8e-7); bf16: a result is rounded once to eight
    # bits, at most 2^-9 of itself
    assert err <= (2e-6 if dtype == torch.float32 else 2.0 ** -9), err
