"""GPU parity of the softmax cross-entropy where its rows stop fitting a thread's registers, and of the sums that take sixteen rows at a time.
Tolerances: fp32 results carry a few roundings of 2^-24 (1e-6); a bf16 gradient one of 2^-9."""
import numpy as np
import pytest
import torch

from test_gpu_ops import B, dev, rnd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n,classes", [(1, 1), (2, 255), (16, 256), (17, 257), (5, 1023), (33, 1024), (3, 1025), (2, 5000)])
def test_loss_and_gradient_together_apart_and_in_place(n, classes, dtype):
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    z = dev(rnd(1, n, classes) * np.float32(8.0)).to(td)
    lab = torch.arange(n, dtype=torch.int32, device="cuda") * 7 % classes
    zd = z.double()
    p = torch.log_softmax(zd, 1)
    ref_rows = -p.gather(1, lab.long()[:, None])[:, 0]
    ref_dz = p.exp()
    ref_dz[torch.arange(n, device="cuda"), lab.long()] -= 1.0
    ref_dz /= n
    rows, loss, dz, alone = torch.empty(n, device="cuda"), torch.empty(1, device="cuda"), torch.empty_like(z), torch.empty_like(z)
    B().op_softmax_ce(z, lab, rows, loss, dz)
    B().op_softmax_ce(z, lab, None, None, alone)
    place = z.clone()
    rows2, loss2 = torch.empty(n, device="cuda"), torch.empty(1, device="cuda")
    B().op_softmax_ce(place, lab, rows2, loss2, place)
    torch.cuda.synchronize()
    assert (rows.double() - ref_rows).abs().max() <= 4e-6 * max(1.0, ref_rows.abs().max().item())
    assert abs(loss.double() - ref_rows.mean()).item() <= 4e-6 * max(1.0, ref_rows.mean().item())
    assert (dz.double() - ref_dz).norm() <= (2e-6 if dtype == "f32" else 4e-3) * ref_dz.norm() + 1e-7
    assert torch.equal(dz, alone) and torch.equal(dz, place) and torch.equal(rows, rows2) and torch.equal(loss, loss2)


def test_a_label_that_does_not_exist():
    z, lab = dev(rnd(2, 3, 40)), torch.tensor([1, 40, -1], dtype=torch.int32, device="cuda")
    rows, loss, dz = torch.zeros(3, device="cuda"), torch.zeros(1, device="cuda"), torch.empty_like(z)
    B().op_softmax_ce(z, lab, rows, loss, dz)
    assert torch.isnan(rows).tolist() == [False, True, True] and bool(torch.isnan(loss))
    assert torch.allclose(dz[1:], torch.softmax(z[1:], 1) / 3, atol=1e-7)


@pytest.mark.parametrize("rows,c", [(16384, 128), (16385, 128), (16384, 132), (90, 256), (7, 252), (8036, 256), (5000, 124), (3, 260)])
def test_batch_norm_in_two_slices_of_channels(rows, c):
    x, dy = dev(rnd(3, rows, c)), dev(rnd(4, rows, c))
    gamma, beta = dev(rnd(5, c) * 0.1 + 1), dev(rnd(6, c))
    y, dx = torch.empty_like(x), torch.empty_like(x)
    mean, istd, dg, db = (torch.empty(c, device="cuda") for _ in range(4))
    ws = torch.empty(B().op_bn_workspace(c), dtype=torch.uint8, device="cuda")
    B().op_bn_fwd(x.view(rows, 1, 1, c), gamma, beta, None, y.view(rows, 1, 1, c), mean, istd, True, 1e-5, ws)
    B().op_bn_bwd(x.view(rows, 1, 1, c), dy.view(rows, 1, 1, c), y.view(rows, 1, 1, c), gamma, mean, istd, dx.view(rows, 1, 1, c), dg, db, None, ws)
    torch.cuda.synchronize()
    xd, m, i = x.double(), mean.double(), istd.double()
    assert (m - xd.mean(0)).abs().max() <= 1e-6
    assert ((xd.var(0, unbiased=False) + 1e-5).rsqrt() / i - 1).abs().max() <= 1e-6
    xh, g = (xd - m) * i, torch.where(y > 0, dy, torch.zeros_like(dy)).double()
    refs = ((y, (xh * gamma.double() + beta.double()).relu()), (db, g.sum(0)), (dg, (g * xh).sum(0)),
            (dx, gamma.double() * i * (g - g.mean(0) - xh * (g * xh).mean(0))))
    for got, ref in refs:
        assert (got.double() - ref).norm() <= 2e-6 * ref.norm() + 1e-6 * ref.numel() ** 0.5 * 1e-1
