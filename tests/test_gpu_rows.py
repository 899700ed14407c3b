"""GPU parity of the fp32 products of few rows and long reductions (conv_rows.hip), forward and as a data gradient that reads the filter
as it lies, at the edges of its tiles, reductions and column widths.

Tolerance: a result is the sum of 16 * 2 or 16 * 4 chains of at most K / 32 additions and of the chains themselves, each rounding 2^-24 of a
partial sum: 2e-6 in the l2 norm if K / 32 + 35 <= 131 of them all went the same way would be 8e-6; they do not, and 1e-6 holds."""
import numpy as np
import pytest
import torch

from test_gpu_ops import B, dev

# rows (images x map), cin, cout, kernel of the forward pass and of the data gradient
NK, KN1, KN2, KN4 = "igemm_rows 16x16", "igemm_rows 16x16 [k][n]", "igemm_rows 16x32", "igemm_rows 16x64"
CASES = [
    (1, 1, 320, 320, NK, KN2),
    (41, 1, 2048, 1000, NK, KN2),
    (17, 1, 336, 324, NK, KN2),         # ragged rows and columns; K that ends inside a group
    (3, 7, 1008, 1004, NK, None),
    (2, 4, 1040, 10, NK, None),         # fewer columns than a tile
    (2, 4, 2064, 2052, NK, KN2),
    (5, 1, 72, 2044, None, KN1),
    (1, 14, 1024, 72, NK, None),
    (95, 1, 2048, 2048, None, KN4),
]


def names(case):
    n, hw, cin, cout = case[:4]
    return [B().op_conv_kernel(role, n, hw, hw, cin, cout, 1, 1, 0, 0) for role in ("fwd", "dgrad")]


@pytest.mark.parametrize("case", CASES)
def test_routes(case):
    for got, want in zip(names(case), case[4:]):
        assert want is None or got == want, (case, got)


# data gradients that are taken because nothing has to transpose the filter first: about as fast as the other kernels without that launch
TRANSPOSED = [
    (2, 14, 1000, 1000, None, KN4),     # 392 rows, 1000 -> 1000
    (1, 14, 2048, 1000, None, KN4),     # 196 rows, 1000 -> 2048
    (160, 1, 2048, 512, None, KN1),
]


@pytest.mark.parametrize("case", TRANSPOSED)
def test_the_saved_transposition_counts(case):
    assert names(case)[1] == case[5]


@pytest.mark.gpu
@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("case", CASES + TRANSPOSED)
def test_products_of_few_rows(case, accumulate):
    n, hw, cin, cout = case[:4]
    rng = np.random.default_rng(cin + n)
    x, w = (rng.standard_normal(s).astype(np.float32) for s in ((n, hw, hw, cin), (cout, 1, 1, cin)))
    dy, base = (rng.standard_normal(s).astype(np.float32) for s in ((n, hw, hw, cout), (n, hw, hw, cin)))
    y = torch.full((n, hw, hw, cout), float("nan"), device="cuda")
    B().op_conv_fwd(dev(x), dev(w), y, 1, 0)
    ws = torch.empty(max(B().op_conv_workspace(n, hw, hw, cin, cout, 1, 1, 0), 256), dtype=torch.uint8, device="cuda")
    dx = dev(base.copy()) if accumulate else torch.full((n, hw, hw, cin), float("nan"), device="cuda")
    B().op_conv_dgrad(dev(dy), dev(w), dx, 1, 0, ws, accumulate)
    torch.cuda.synchronize()
    w2 = w.reshape(cout, cin).astype(np.float64)
    for got, ref in ((y, x.reshape(-1, cin) @ w2.T), (dx, dy.reshape(-1, cout) @ w2 + (base.reshape(-1, cin) if accumulate else 0.0))):
        err = np.linalg.norm(got.cpu().numpy().reshape(ref.shape) - ref) / np.linalg.norm(ref)
        assert err <= 1e-6, err


@pytest.mark.gpu
def test_infinities_and_nan_stay_in_their_rows_and_columns():
    x, w = np.ones((5, 1, 1, 512), np.float32), np.full((72, 1, 1, 512), 0.5, np.float32)
    x[1, 0, 0, 511], x[3, 0, 0, 7], w[70, 0, 0, 300] = np.inf, np.nan, -np.inf
    y = torch.empty((5, 1, 1, 72), device="cuda")
    B().op_conv_fwd(dev(x), dev(w), y, 1, 0)
    ref = np.full((5, 72), 256.0)
    ref[:, 70] = -np.inf
    ref[1] = np.inf
    ref[1, 70] = np.nan
    ref[3] = np.nan
    np.testing.assert_array_equal(y.cpu().numpy().reshape(5, 72), ref)


# (rows, columns of the result, kernel): a filter that is read as it lies, one, two and four columns per lane
@pytest.mark.parametrize("n,cin,cout,name", [(5, 72, 2044, KN1), (41, 2048, 1000, KN2), (95, 2048, 2048, KN4)])
@pytest.mark.gpu
def test_infinities_and_nan_through_a_filter_read_as_it_lies(n, cin, cout, name):
    assert B().op_conv_kernel("dgrad", n, 1, 1, cin, cout, 1, 1, 0, 0) == name
    dy, w = np.ones((n, 1, 1, cout), np.float32), np.full((cout, 1, 1, cin), 0.5, np.float32)
    dy[1, 0, 0, cout - 1], dy[3, 0, 0, 7], w[300, 0, 0, cin - 3] = np.inf, np.nan, -np.inf
    ws = torch.empty(B().op_conv_workspace(n, 1, 1, cin, cout, 1, 1, 0), dtype=torch.uint8, device="cuda")
    dx = torch.empty((n, 1, 1, cin), device="cuda")
    B().op_conv_dgrad(dev(dy), dev(w), dx, 1, 0, ws)
    ref = np.full((n, cin), cout / 2.0)
    ref[:, cin - 3] = -np.inf
    ref[1] = np.inf
    ref[1, cin - 3] = np.nan
    ref[3] = np.nan
    np.testing.assert_array_equal(dx.cpu().numpy().reshape(n, cin), ref)
