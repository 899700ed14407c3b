"""bf16 weight gradient on maps of millions of rows or columns, and of a few rows or columns on either side of 4096: a thread counts the pixels of its
rows on from chunk to chunk, by whole images, rows and columns with one wrap of each at most, and that has to hold for any map.  Every
position counts, the ones at the ends of a row above all.

The operands are whole numbers up to 2 at a few thousand positions, zero elsewhere, so every sum is a whole number below 2^24 and the
result is exact in any order."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,w", [(1, 7561049), (7561049, 1), (1, 9000001), (4099, 5), (3, 4097), (4096, 4), (70, 4096)])
def test_wgrad_bf16_far(h, w):
    from paper_1901_06773_amd import binding as b
    c, m = 8, h * w
    gen = torch.Generator().manual_seed(m)
    at = torch.cat([torch.arange(0, 200), torch.arange(m - 200, m), torch.arange(w - 1, m, max(w, m // 997)),
                    torch.randint(0, m, (2000,), generator=gen)]).clamp(0, m - 1).unique()
    x, dy = torch.zeros(m, c), torch.zeros(m, c)
    x[at] = torch.randint(-2, 3, (at.numel(), c), generator=gen).float()
    dy[at] = torch.randint(-2, 3, (at.numel(), c), generator=gen).float()
    ws = torch.empty(b.op_conv_workspace(1, h, w, c, c, 3, 1, 1), dtype=torch.uint8, device="cuda")
    dw = torch.full((c, 3, 3, c), float("nan"), device="cuda")
    b.op_conv_wgrad(x.to(torch.bfloat16).cuda().view(1, h, w, c), dy.to(torch.bfloat16).cuda().view(1, h, w, c), dw, 1, 1, ws)
    torch.cuda.synchronize()
    ref = torch.zeros(c, 3, 3, c)
    p, q = at // w, at % w
    for kr in range(3):
        for kt in range(3):
            iy, ix = p + kr - 1, q + kt - 1
            ok = (iy >= 0) & (iy < h) & (ix >= 0) & (ix < w)
            ref[:, kr, kt, :] = dy[at[ok]].t() @ x[(iy * w + ix)[ok]]
    assert ref.abs().max() < 2 ** 24 and ref[:, 1, 1].abs().sum() > 0
    assert torch.equal(dw.cpu(), ref)
