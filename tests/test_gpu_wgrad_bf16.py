"""GPU parity of the bf16 weight gradient at the edges of its five tilings, on 1x1 filters and on others: tiles that the channels fill whole, by a remainder or by eight channels,
columns of a tile that span filter taps, fewer positions than a chunk, one more and one fewer than whole chunks, maps smaller than a chunk (a
row's position wraps over whole images), strides, paddings and filters of every kind, one part and many.

Tolerance: bf16 products are exact in fp32, so only the fp32 sums round: at most (terms of the longest chain) * 2^-24 of the sum of magnitudes.
Normal values make that less than 1e-5 of the l2 norm for the sizes here; whole numbers below 2^24 are exact in any order."""
import pytest
import torch

# n, h, w, cin, cout, r, stride, pad, tiling
CASES = [
    (20, 14, 14, 256, 256, 3, 1, 1, "64x64"),    # whole tiles
    (9, 15, 13, 264, 136, 3, 1, 1, "64x64"),     # remainders of eight in both directions, columns that span taps
    (64, 7, 7, 512, 512, 3, 1, 1, "128x256"),      # maps of 49 positions, chunks of 64 and 128
    (31, 28, 28, 512, 128, 1, 1, 0, "64x64 plain"),
    (40, 28, 28, 128, 512, 1, 1, 0, "64x64 plain"),
    (16, 56, 56, 64, 64, 1, 1, 0, "64x64 plain"),      # few elements in many parts
    (16, 55, 56, 64, 64, 3, 1, 1, "64x64"),
    (8, 56, 55, 64, 256, 1, 2, 0, "64x64"),      # strided, smaller than its stride
    (5, 27, 29, 128, 128, 3, 2, 1, "64x64"),
    (3, 30, 31, 40, 72, 3, 2, 1, "64x64"),
    (1, 1, 1, 64, 64, 1, 1, 0, "64x128 plain"),         # one position
    (1, 3, 21, 64, 128, 1, 1, 0, "64x128 plain"),       # 63, 64, 65, 127, 129 positions
    (1, 8, 8, 128, 64, 1, 1, 0, "64x128 plain"),
    (1, 5, 13, 72, 64, 1, 1, 0, "64x128 plain"),
    (1, 1, 127, 64, 8, 3, 1, 1, "64x64"),
    (1, 3, 43, 8, 200, 3, 1, 1, "64x64"),
    (200, 1, 1, 2048, 1000, 1, 1, 0, "128x64 plain"),   # a fully connected layer
    (70, 1, 2, 24, 40, 3, 1, 1, "64x64"),        # maps of two positions
    (50, 2, 3, 32, 32, 5, 3, 2, "64x128"),
    (2, 33, 17, 16, 48, 5, 1, 2, "64x64"),
    (3, 12, 12, 32, 136, 3, 4, 0, "64x128"),
    (4, 16, 16, 136, 264, 2, 1, 1, "128x64"),     # even filters
    (2, 9, 70, 384, 24, 2, 1, 0, "64x64"),
    # the two large tilings, in several parts
    (512, 14, 14, 256, 256, 3, 1, 1, "256x128"),   # whole tiles, fourteen parts of 112 whole chunks
    (301, 13, 11, 200, 504, 3, 1, 1, "256x128"),   # both directions end inside a tile, the range inside a chunk
    (301, 13, 11, 264, 136, 3, 1, 1, "256x128"),   # one tile, half of its channels there
    (257, 7, 7, 512, 512, 3, 1, 1, "256x128"),     # an image is less than a chunk
    (301, 13, 11, 512, 512, 3, 2, 1, "256x128"),
    (256, 28, 28, 320, 392, 1, 2, 0, "256x128"),
    (130, 28, 27, 200, 504, 1, 1, 0, "256x128 plain"),
    (512, 14, 14, 264, 136, 1, 1, 0, "256x128 plain"),
    (301, 13, 11, 136, 520, 3, 1, 1, "128x256"),
    (257, 7, 7, 200, 504, 3, 1, 1, "128x256"),
    (63, 28, 27, 448, 208, 2, 1, 0, "256x128"),
    (256, 28, 28, 136, 520, 1, 2, 0, "128x256"),
    (256, 28, 28, 512, 128, 1, 1, 0, "128x256 plain"),
    (301, 13, 11, 136, 520, 1, 1, 0, "128x256 plain"),
    (51, 33, 30, 456, 200, 1, 1, 0, "128x256 plain"),
    # 64 x 128 and 128 x 64 in several parts
    (75, 17, 15, 416, 160, 3, 2, 1, "64x128"),
    (33, 39, 39, 352, 80, 1, 1, 0, "64x128 plain"),
    (37, 21, 20, 104, 304, 3, 1, 1, "128x64"),
    (33, 27, 26, 488, 424, 1, 1, 0, "128x64 plain"),
]


@pytest.mark.parametrize("case", CASES)
def test_tiling(case):
    from paper_1901_06773_amd import binding as b
    assert b.op_conv_kernel("wgrad", *case[:8], b.BF16) == "wgrad_bf16 " + case[8]


def test_every_tiling_has_cases():
    assert {c[8] for c in CASES} == {t + f for t in ("256x128", "128x256", "64x64", "64x128", "128x64") for f in ("", " plain")}


@pytest.mark.gpu
@pytest.mark.parametrize("whole", [False, True])
@pytest.mark.parametrize("case", CASES)
def test_wgrad_bf16(case, whole):
    from paper_1901_06773_amd import binding as b
    n, h, w, ci, co, r, st, pad = case[:8]
    ho, wo = (h + 2 * pad - r) // st + 1, (w + 2 * pad - r) // st + 1
    gen = torch.Generator(device="cuda").manual_seed(n * h + w + ci)
    def values(*shape):
        t = torch.randint(-3, 4, shape, generator=gen, device="cuda").float() if whole else torch.randn(shape, generator=gen, device="cuda")
        return t.to(torch.bfloat16)
    # operands end where their memory does, with NaN behind them
    def at_end(t):
        buf = torch.full((t.numel() + 4096,), float("nan"), dtype=t.dtype, device="cuda")
        buf[:t.numel()] = t.reshape(-1)
        return buf[:t.numel()].view(t.shape)
    x, dy = at_end(values(n, h, w, ci)), at_end(values(n, ho, wo, co))
    need = b.op_conv_workspace(n, h, w, ci, co, r, st, pad)
    ws = torch.full((need // 4 + 1024,), float("nan"), device="cuda")
    dw = torch.full((co, r, r, ci), float("nan"), device="cuda")
    b.op_conv_wgrad(x, dy, dw, st, pad, ws.view(torch.uint8)[:need])
    torch.cuda.synchronize()
    xp = torch.nn.functional.pad(x.double(), (0, 0, pad, pad, pad, pad))
    g = dy.double().reshape(-1, co).t().contiguous()
    ref = torch.empty(co, r, r, ci, dtype=torch.float64, device="cuda")
    for a in range(r):
        for c in range(r):
            ref[:, a, c] = g @ xp[:, a:a + (ho - 1) * st + 1:st, c:c + (wo - 1) * st + 1:st].reshape(-1, ci)
    assert bool(ws[(need + 3) // 4:].isnan().all())          # nothing written behind the workspace
    if whole:
        assert torch.equal(dw.double(), ref)
    else:
        assert float((dw.double() - ref).norm() / ref.norm()) < 1e-5
