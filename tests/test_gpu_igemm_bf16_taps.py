"""GPU parity of every bf16 tiling on the path of the networks' 3x3 layers: several taps of several chunks of channels (whole chunks, and
widths that span two taps with one), ragged tiles in both directions; forward, data gradient with and without accumulation, and bias + ReLU
in the launch, which only an iteration reaches.

Tolerance: bf16 operands on both sides, products exact in fp32, one rounding of the result to bf16: 2^-8 / sqrt(3) = 2.3e-3 of it in the l2 norm
if every value were the worst one of its binade, 2^-8 of the largest at most; the fp32 sums add less than 1e-5."""
import numpy as np
import pytest
import torch

import synth as S
from test_gpu_ops import B

# n, h, w, channels reduced over, channels of the result, tiling
CASES = [
    (87, 21, 21, 128, 136, "256x256"),
    (45, 31, 29, 136, 136, "256x256"),
    (201, 14, 14, 256, 248, "256x256"),
    (220, 10, 10, 128, 136, "128x256"),
    (21, 33, 33, 136, 144, "128x256"),
    (249, 12, 11, 96, 72, "256x128"),
    (24, 37, 37, 72, 80, "256x128"),
    (44, 34, 33, 128, 72, "128x128"),
    (121, 22, 20, 168, 72, "128x128"),
    (119, 22, 19, 128, 32, "128x64"),
    (80, 25, 25, 136, 32, "128x64"),
    (120, 17, 17, 128, 32, "64x64"),
    (25, 38, 35, 152, 32, "64x64"),
    (34, 23, 21, 128, 32, "64x64, four stages"),
    (3, 39, 37, 144, 40, "64x64, four stages"),
    (34, 11, 11, 256, 40, "64x64, four pairs"),
    (3, 38, 37, 272, 40, "64x64, four pairs"),
    (9, 22, 21, 96, 40, "64x64, four waves"),
    (9, 22, 21, 80, 40, "64x64, four waves"),
    (1, 7, 4, 64, 32, "32x32, eight waves"),
    (1, 5, 5, 72, 40, "32x32, eight waves"),
]


@pytest.mark.parametrize("case", CASES)
def test_routes(case):
    n, h, w, c, m, name = case
    assert B().op_conv_kernel("fwd", n, h, w, c, m, 3, 1, 1, B().BF16) == "igemm_bf16 " + name
    assert B().op_conv_kernel("dgrad", n, h, w, m, c, 3, 1, 1, B().BF16) == "igemm_bf16 " + name


def randn(seed, shape, scale=1.0):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return (torch.randn(shape, generator=g, device="cuda") * scale).bfloat16()


def conv64(x, w):
    """3x3, padding 1; NHWC x, O-H-W-I w, as float64: one product per tap."""
    n, h, wd, c = x.shape
    xp = torch.nn.functional.pad(x.double(), (0, 0, 1, 1, 1, 1))
    y = torch.zeros((n * h * wd, w.shape[0]), dtype=torch.float64, device=x.device)
    for a in range(3):
        for b in range(3):
            y += xp[:, a:a + h, b:b + wd].reshape(-1, c) @ w[:, a, b].double().t().contiguous()
    return y.view(n, h, wd, -1)


def close(got, ref):
    d = got.double() - ref
    assert torch.isfinite(d).all()
    assert d.norm() <= 2.3e-3 * ref.norm(), float(d.norm() / ref.norm())
    assert d.abs().max() <= 2.0 ** -8 * ref.abs().max()


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES)
def test_forward_and_data_gradient(case):
    n, h, w, c, m, _ = case
    x, wt = randn(1, (n, h, w, c)), randn(2, (m, 3, 3, c), (2.0 / (9 * c)) ** 0.5)
    y = torch.full((n, h, w, m), float("nan"), device="cuda", dtype=torch.bfloat16)
    B().op_conv_fwd(x, wt, y, 1, 1)
    ref = conv64(x, wt)
    close(y, ref)
    # the layer whose data gradient is this product: its filter is this one flipped and transposed
    wl = wt.flip(1, 2).permute(3, 1, 2, 0).contiguous()
    ws = torch.empty(B().op_conv_workspace(n, h, w, m, c, 3, 1, 1), dtype=torch.uint8, device="cuda")
    dx = torch.full((n, h, w, m), float("nan"), device="cuda", dtype=torch.bfloat16)
    B().op_conv_dgrad(x, wl, dx, 1, 1, ws)
    assert torch.equal(dx, y)                                   # the same kernel on the same numbers
    base = randn(3, (n, h, w, m))
    dx = base.clone()
    B().op_conv_dgrad(x, wl, dx, 1, 1, ws, True)
    close(dx, ref + base.double())


@pytest.mark.gpu
@pytest.mark.parametrize("relu", [True, False])
@pytest.mark.parametrize("case", CASES)
def test_bias_and_relu_in_the_launch(case, relu):
    n, h, w, c, m, _ = case
    net = S.NetSpec("one_layer", c, h, w, 4)
    x = net.add(S.Layer(S.CONV, in0=-1, cin=c, cout=m, r=3, s=3, stride=1, pad=1))
    x = net.add(S.Layer(S.BIAS, in0=x, cin=m, cout=m))
    if relu:
        x = net.add(S.Layer(S.RELU, in0=x, cin=m, cout=m))
    out = x
    x = net.add(S.Layer(S.GAP, in0=x, cin=m, cout=m))
    x = net.add(S.Layer(S.FC, in0=x, cin=m, cout=4))
    net.add(S.Layer(S.SOFTMAX_CE, in0=x, cin=4, cout=1))
    img = randn(4, (n, c, h, w)).float()                        # NCHW, bf16 values
    wt, bias = randn(5, (m, c, 3, 3), (2.0 / (9 * c)) ** 0.5).float(), torch.randn(m, generator=torch.Generator().manual_seed(6))
    params = [np.zeros(0, np.float32)] * len(net.layers)
    params[0], params[1] = wt.cpu().numpy().ravel(), bias.numpy()
    params[-2] = np.zeros(4 * m + 4, np.float32)
    b = B()
    probe = b.Context(net.as_array(), (c, h, w), dtype=b.BF16)
    need = probe.plan_swaps(n, 1 << 38, b.PLAN_NONE)["peak_bytes"]
    probe.close()
    ctx = b.Context(net.as_array(), (c, h, w), pool_bytes=int(need * 1.1) + (8 << 20), host_bytes=1 << 20, dtype=b.BF16)
    ctx.set_weights(params)
    ctx.plan_swaps(n, int(need * 1.1) + (8 << 20), b.PLAN_NONE)
    got = ctx.capture_outputs([out], {out: (m, h, w)}, n)[out]
    ctx.train_step(img, np.zeros(n, np.int32), 0.0)
    ctx.stop_captures()
    ref = conv64(img.permute(0, 2, 3, 1).contiguous(), wt.permute(0, 2, 3, 1).contiguous()) + bias.cuda().double()
    close(got.cuda(), ref.relu() if relu else ref)
    ctx.close()
