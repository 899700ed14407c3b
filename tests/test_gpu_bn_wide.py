"""Batch norm in bf16 over more rows than the slice kernels take: eight channels per thread (16-byte accesses) and four."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

ROWS = 16384 + 1 + 2 * 23      # one row more than the slice kernels' last, and a ragged tail of the row loops


def _tensor(flat):
    return flat.to(torch.bfloat16).cuda().view(1, 1, *flat.shape)


# Eight channels per thread from 4 Mi elements on: 520 (65 threads across a row, in slices of 33 and 32), 8 and 24 (one and three
# threads), 256 (a last workgroup that is not full).  Four: fewer elements; 12, 260 and 1028: channels not in eights.
@pytest.mark.parametrize("ROWS,c", [(ROWS, 8), (ROWS, 24), (ROWS, 520), (ROWS, 12), (ROWS, 260), (ROWS, 1028), (524288 + 47, 8),
                                    (174763, 24), (16385, 256)])
@pytest.mark.parametrize("relu", [False, True])
def test_bn_bf16_many_rows(ROWS, c, relu):
    from paper_1901_06773_amd import binding as b
    g = torch.Generator().manual_seed(c)
    x, dy, res = ((torch.randn(ROWS, c, generator=g) * 1.5 + 0.3).to(torch.bfloat16) for _ in range(3))
    gamma, beta = torch.rand(c, generator=g) + 0.5, torch.randn(c, generator=g)
    xd, dyd, resd = _tensor(x), _tensor(dy), _tensor(res)
    y, dx = _tensor(torch.zeros(ROWS, c)), _tensor(torch.zeros(ROWS, c))
    ws = torch.empty(b.op_bn_workspace(c), dtype=torch.uint8, device="cuda")
    mean, istd, dg, db = (torch.empty(c, device="cuda") for _ in range(4))
    b.op_bn_fwd(xd, gamma.cuda(), beta.cuda(), resd if relu else None, y, mean, istd, relu, 1e-5, ws)
    b.op_bn_bwd(xd, dyd, y if relu else None, gamma.cuda(), mean, istd, dx, dg, db, dyd if relu else None, ws)
    torch.cuda.synchronize()

    xs, gs = x.double(), dy.double()
    mu, inv = xs.mean(0), (xs.var(0, unbiased=False) + 1e-5).rsqrt()
    ref = (xs - mu) * inv * gamma.double() + beta.double()
    if relu:
        ref = (ref + res.double()).clamp_min(0)
        gs = gs * (y.cpu().view(ROWS, c) > 0)      # the decisions of the stored output
    xhat = (xs - mu) * inv
    ref_dg, ref_db = (gs * xhat).sum(0), gs.sum(0)
    ref_dx = gamma.double() * inv * (gs - ref_db / ROWS - xhat * ref_dg / ROWS)
    # stored values: one rounding to bf16 (2^-9 of the value) on top of a few fp32 roundings of terms up to ~20
    tol = lambda r: r.abs() * 2.0 ** -8 + 20 * 2.0 ** -20
    got_y, got_dx = y.cpu().double().view(ROWS, c), dx.cpu().double().view(ROWS, c)
    assert ((got_y - ref).abs() <= tol(ref)).all()
    assert ((got_dx - ref_dx).abs() <= tol(ref_dx)).all()
    # sums over 16431 values in fp64 of terms rounded in fp32: ROWS * 2^-23 * |term|, |term| on average below 2
    assert np.abs((dg.cpu().double() - ref_dg).numpy()).max() <= ROWS * 2.0 ** -22
    assert np.abs((db.cpu().double() - ref_db).numpy()).max() <= ROWS * 2.0 ** -22
    if relu:
        assert torch.equal(dyd.cpu().view(ROWS, c).double(), gs)
