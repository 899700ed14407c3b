"""Gradient of 3x3 max-pooling at stride 2 in bf16: the first maximum of every window by rank, against a plain scan."""
import numpy as np
import pytest
import torch

from paper_1901_06773_amd import binding as B

pytestmark = pytest.mark.gpu


def scan(x, dy, dx):
    """First maximum by ">" over the positions of a window that lie in the map; sums in window order, fp32, rounded once."""
    n, h, w, c = x.shape
    ho, wo = dy.shape[1:3]
    acc = np.zeros(x.shape, np.float32)
    i, k = np.ogrid[:n, :c]
    for p in range(ho):
        for q in range(wo):
            best = at = None
            for y in range(max(2 * p - 1, 0), min(2 * p + 2, h)):
                for z in range(max(2 * q - 1, 0), min(2 * q + 2, w)):
                    v = x[:, y, z]
                    more = np.ones(v.shape, bool) if best is None else v > best
                    at = np.where(more, y * w + z, 0 if at is None else at)
                    best = np.where(more, v, 0 if best is None else best)
            acc[i, at // w, at % w, k] += dy[:, p, q]
    return torch.from_numpy(acc if dx is None else dx + acc).bfloat16()


# strips of one, two and four blocks (160 thousand and 512 thousand blocks of 2 x 2 positions and four channels on), odd and even edges
@pytest.mark.parametrize("shape", [(2, 1, 1, 4), (3, 8, 7, 8), (2, 9, 12, 64), (700, 12, 13, 24), (2100, 11, 9, 44)])
@pytest.mark.parametrize("values", ["ties", "special"])
@pytest.mark.parametrize("accumulate", [False, True])
def test_first_maximum(shape, values, accumulate):
    n, h, w, c = shape
    g = np.random.default_rng(3)
    some = [-1.0, -0.5, -0.0, 0.0, 0.5, 2.0 ** -130, -2.0 ** -130] if values == "ties" else [
        -np.inf, -np.inf, -3e38, -1.0, -0.0, 0.0, 1.0, 3e38, np.inf, np.nan, -np.nan]
    x = torch.from_numpy(g.choice(np.array(some, np.float32), shape)).bfloat16()
    if values == "special":                       # most rows without a NaN
        keep = torch.from_numpy(g.random((n, h, 1, 1)) < 0.3)
        x = torch.where(torch.isnan(x) & ~keep, torch.ones((), dtype=x.dtype), x)
    dy = torch.from_numpy(g.standard_normal((n, (h - 1) // 2 + 1, (w - 1) // 2 + 1, c), dtype=np.float32)).bfloat16()
    base = torch.from_numpy(g.standard_normal(shape, dtype=np.float32)).bfloat16()
    dx = base.cuda() if accumulate else torch.full(shape, float("nan"), dtype=torch.bfloat16, device="cuda")
    B.op_maxpool_bwd(x.cuda(), dy.cuda(), dx, 3, 2, 1, accumulate=accumulate)
    torch.cuda.synchronize()
    assert torch.equal(dx.cpu(), scan(x.float().numpy(), dy.float().numpy(), base.float().numpy() if accumulate else None))
