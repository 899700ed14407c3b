"""Iterations that swap little issue their copies in the compute stream, larger ones on streams of their own with events: on both sides of the
line (1.25 MiB each way) a swapped iteration has the bits of the resident one, also where every byte that is not alive holds a NaN
pattern, with weight gradients on their own stream or not, and where plans of both kinds follow each other in one context."""
import pytest
import torch

import synth as S

pytestmark = pytest.mark.gpu


def run(ctx, b, net, k, mode, budget, poison, overlap):
    ctx.set_weights(S.init_params(net))
    ctx.set_wgrad_overlap(overlap)
    summ = ctx.plan_swaps(k, budget, mode)
    ctx.set_debug(poison)
    losses = [ctx.train_step(torch.from_numpy(img).pin_memory(), lab, 0.1) for img, lab in (S.make_batch(net, k, s) for s in range(3))]
    ctx.set_debug(False)
    return summ, losses, ctx.get_weights(), ctx.get_grads()


@pytest.mark.parametrize("overlap", [True, False])
@pytest.mark.parametrize("dtype", ["F32", "BF16"])
def test_both_sides_of_the_line(dtype, overlap):
    from paper_1901_06773_amd import binding as b
    net = S.bottleneck_unit(64, 16, 16, 10)
    shape, code = (net.in_c, net.in_h, net.in_w), getattr(b, dtype)
    probe = b.Context(net.as_array(), shape, dtype=code)
    ks = (1, 4, 5, 6) if dtype == "F32" else (1, 9, 10, 13)
    out = [probe.plan_swaps(k, 1 << 38, b.PLAN_NAIVE_ALL)["host_bytes"] for k in ks]
    assert out[1] <= 5 << 18 < out[2] or out[2] <= 5 << 18 < out[3]      # the line lies between
    budget = int(probe.plan_swaps(ks[-1], 1 << 38, b.PLAN_NONE)["peak_bytes"] * 1.2) + (8 << 20)
    probe.close()
    ctx = b.Context(net.as_array(), shape, pool_bytes=budget, host_bytes=out[-1] + 4096, dtype=code)
    for k in ks + ks[:1]:
        summ, losses, weights, grads = run(ctx, b, net, k, b.PLAN_NONE, budget, False, overlap)
        assert summ["n_swapped"] == 0
        for poison in (False, True):
            s2, l2, w2, g2 = run(ctx, b, net, k, b.PLAN_NAIVE_ALL, budget, poison, overlap)
            assert s2["n_swapped"] == s2["n_maps"] > 0
            assert l2 == losses, (k, poison)
            for i, (a, r) in enumerate(zip(list(w2) + list(g2), list(weights) + list(grads))):
                assert (a == r).all(), (k, poison, i)
    ctx.close()
