"""GPU parity of the first layer's forward kernel where the width decides how many rows a workgroup holds: pairs of rows held as bf16 parts,
one pair, and rows held as words when a pair does not fit.  Tolerances: those of test_gpu_smallc.py."""
import numpy as np
import pytest
import torch

import oracle as O
from test_gpu_ops import B, dev, nchw, nhwc, ohwi, rnd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", [
    (48, 40, 330, 3, 64, 7, 2, 3),      # six rows of words, four rows of parts
    (21, 61, 449, 3, 40, 7, 2, 3),       # one pair, an odd number of rows and columns
    (4, 80, 880, 3, 24, 7, 2, 3),       # fp32: a single row of words
    (36, 25, 521, 3, 33, 5, 1, 2),       # positions an odd number of values apart
])
def test_wide_images(case, dtype):
    n, h, w, cin, cout, r, stride, pad = case
    assert B().op_conv_kernel("fwd", *case, B().F32 if dtype == "f32" else B().BF16) == "smallc"
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    x = torch.from_numpy(rnd(1, n, cin, h, w)).to(td).float().numpy()
    wt = torch.from_numpy(rnd(2, cout, cin, r, r) * np.float32(np.sqrt(2.0 / (cin * r * r)))).to(td).float().numpy()
    ref = O.conv_fwd(x, wt, stride, pad).astype(np.float64)
    y = torch.full((n, ref.shape[2], ref.shape[3], cout), float("nan"), device="cuda", dtype=td)
    B().op_conv_fwd(dev(nhwc(x)).to(td), dev(ohwi(wt)).to(td), y, stride, pad)
    torch.cuda.synchronize()
    err = np.linalg.norm(nchw(y.float().cpu().numpy()) - ref) / np.linalg.norm(ref)
    assert err <= (2e-6 if dtype == "f32" else 8e-3), err
