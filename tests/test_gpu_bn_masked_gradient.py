"""Batch norm's backward pass where the masked gradient is wanted: from 2^20 elements on the pass that sums stores it.  Row
counts that leave the last trip of rows short, in one place and out of place; below the line the other pass stores it."""
import pytest
import torch

pytestmark = pytest.mark.gpu


# threads across a row x channels of a thread: 64 x 4, 11 x 4, 64 x 8 (bf16, large) and 25 x 8
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("rows,c", [(4096, 256), (4095, 256), (23833, 44), (16385 + 7, 512), (32769, 200), (1025, 1024)])
@pytest.mark.parametrize("in_place", [False, True])
def test_bn_bwd_masked_gradient(rows, c, dtype, in_place):
    from paper_1901_06773_amd import binding as b
    g = torch.Generator().manual_seed(rows + c)
    x, dy, y = (torch.randn(1, 1, rows, c, generator=g).to(dtype).cuda() for _ in range(3))
    gamma = (torch.rand(c, generator=g) + 0.5).cuda()
    mean, istd = x.double().reshape(rows, c).mean(0).float(), (x.double().reshape(rows, c).var(0, unbiased=False) + 1e-5).rsqrt().float()
    dx, dg, db = torch.empty_like(x), torch.empty(c, device="cuda"), torch.empty(c, device="cuda")
    ws = torch.empty(b.op_bn_workspace(c), dtype=torch.uint8, device="cuda")
    d_in, g_out = dy.clone(), torch.full_like(x, float("nan"))
    if in_place:
        g_out = d_in
    b.op_bn_bwd(x, d_in, y, gamma, mean, istd, dx, dg, db, g_out, ws)
    torch.cuda.synchronize()
    want_g = torch.where(y > 0, dy, torch.zeros_like(dy))
    assert torch.equal(g_out, want_g)                                     # stored values, selected and not computed
    gd, xh = want_g.double().view(rows, c), (x.double().view(rows, c) - mean.double()) * istd.double()
    ref_db, ref_dg = gd.sum(0), (gd * xh).sum(0)
    ref = gamma.double() * istd.double() * (gd - ref_db / rows - xh * ref_dg / rows)
    # sums in fp64 of products rounded a few times in fp32 (2^-23 of a term below 25, on average below 1); one rounding to storage at the end
    assert (db.double() - ref_db).abs().max() <= rows * 2.0 ** -22 and (dg.double() - ref_dg).abs().max() <= rows * 2.0 ** -22
    eps = 2.0 ** -8 if dtype == torch.bfloat16 else 2.0 ** -21
    assert ((dx.double().view(rows, c) - ref).abs() <= ref.abs() * eps + 20 * 2.0 ** -21).all()


@pytest.mark.parametrize("over", ["x", "y"])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_bn_bwd_masked_gradient_over_an_input(over, dtype):
    """The masked gradient may lie over a tensor that the call has read: the same bits as in a place of its own."""
    from paper_1901_06773_amd import binding as b
    rows, c = 8200, 256
    g = torch.Generator().manual_seed(3)
    x, dy, y = (torch.randn(1, 1, rows, c, generator=g).to(dtype).cuda() for _ in range(3))
    gamma = (torch.rand(c, generator=g) + 0.5).cuda()
    mean, istd = x.double().reshape(rows, c).mean(0).float(), (x.double().reshape(rows, c).var(0, unbiased=False) + 1e-5).rsqrt().float()
    ws = torch.empty(b.op_bn_workspace(c), dtype=torch.uint8, device="cuda")
    want_g = torch.where(y > 0, dy, torch.zeros_like(dy))
    gd, xh = want_g.double().view(rows, c), (x.double().view(rows, c) - mean.double()) * istd.double()
    ref = gamma.double() * istd.double() * (gd - gd.mean(0) - xh * (gd * xh).mean(0))
    dx, dg, db = torch.empty_like(x), torch.empty(c, device="cuda"), torch.empty(c, device="cuda")
    b.op_bn_bwd(x, dy, y, gamma, mean, istd, dx, dg, db, x if over == "x" else y, ws)
    torch.cuda.synchronize()
    assert torch.equal(x if over == "x" else y, want_g)
    eps = 2.0 ** -8 if dtype == torch.bfloat16 else 2.0 ** -21
    assert ((dx.double().view(rows, c) - ref).abs() <= ref.abs() * eps + 20 * 2.0 ** -21).all()
