"""GPU parity of weight gradients with few elements in many parts (one thread adds up the parts of one element): a last wave that is not full,
an element count that does not divide by four, the largest count.  Tolerance: sums of n * h * w products in fp32, at most a few thousand
roundings of 2^-24 that do not all go one way; 2e-6 is what the other weight gradient tests hold in the l2 norm."""
import numpy as np
import pytest
import torch

import oracle as O
from test_gpu_ops import B, dev, nhwc, rnd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", [
    (24, 28, 28, 36, 44, 1),     # 1584 elements: 24.75 waves
    (24, 28, 28, 5, 13, 1),      # 65 elements
    (20, 28, 28, 64, 64, 3),     # 36864
    (16, 28, 28, 256, 256, 1),   # 65536, the most
    (16, 28, 28, 260, 256, 1),   # one row of elements more
])
def test_sums_of_many_parts(case):
    n, h, w, cin, cout, r = case
    x, dy = rnd(1, n, cin, h, w), rnd(2, n, cout, h, w)
    ws = torch.empty(B().op_conv_workspace(n, h, w, cin, cout, r, 1, r // 2), dtype=torch.uint8, device="cuda")
    dw = torch.full((cout, r, r, cin), float("nan"), device="cuda")
    B().op_conv_wgrad(dev(nhwc(x)), dev(nhwc(dy)), dw, 1, r // 2, ws)
    torch.cuda.synchronize()
    ref = O.conv_wgrad(x, dy, (cout, cin, r, r), 1, r // 2).astype(np.float64)
    err = np.linalg.norm(dw.cpu().numpy().transpose(0, 3, 1, 2) - ref) / np.linalg.norm(ref)
    assert err <= 2e-6, err
