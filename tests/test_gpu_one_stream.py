"""Iterations that swap eight maps or more, of at most 1.25 MiB in all, issue their copies in the compute stream, others on streams of their own
with events: on both sides of both lines a swapped iteration has the bits of the resident one, also where every byte that is not alive holds a
NaN pattern and where steps and copies are timed, with weight gradients on their own stream or not, and where plans of both kinds follow each
other in one context.  The input comes behind what the caller has queued on the swap-in stream either way."""
import pytest
import torch

import synth as S

pytestmark = pytest.mark.gpu


def run(ctx, b, net, k, swap, budget, how, overlap):
    """swap: how many maps, the first ones.  how: "", "poison" or "timed"."""
    from paper_1901_06773_amd import validate as V
    ctx.set_weights(S.init_params(net))
    ctx.set_wgrad_overlap(overlap)
    summ = ctx.plan_explicit(k, budget, [i < swap for i in range(ctx.plan_swaps(k, budget, b.PLAN_NONE)["n_maps"])])
    ctx.set_debug(how == "poison")
    ctx.set_profiling(1 if how == "timed" else 0)
    losses = [ctx.train_step(torch.from_numpy(img).pin_memory(), lab, 0.1) for img, lab in (S.make_batch(net, k, s) for s in range(3))]
    ctx.set_debug(False)
    ctx.set_profiling(0)
    if how == "timed":
        assert V.dependency_violations(ctx, ctx.timeline(observed=True)) == []
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
        summ, losses, weights, grads = run(ctx, b, net, k, 0, budget, "", overlap)
        assert summ["n_swapped"] == 0 and ctx.stats()["copies_in_order"] == 0
        for swap, how in ((9, ""), (9, "poison"), (9, "timed"), (8, ""), (8, "poison"), (7, ""), (7, "poison"), (9, "")):
            s2, l2, w2, g2 = run(ctx, b, net, k, swap, budget, how, overlap)
            assert s2["n_maps"] == 9 and s2["n_swapped"] == swap
            assert ctx.stats()["copies_in_order"] == (swap >= 8 and s2["bytes_swapped"] <= 5 << 18)
            assert l2 == losses, (k, swap, how)
            for i, (a, r) in enumerate(zip(list(w2) + list(g2), list(weights) + list(grads))):
                assert (a == r).all(), (k, swap, how, i)
    ctx.close()


@pytest.mark.parametrize("k", [2, 8])
def test_an_input_prepared_on_the_swap_in_stream_is_complete(k):
    """Work that the caller has queued on the swap-in stream comes before the input load, whichever stream carries the other copies."""
    from paper_1901_06773_amd import binding as b
    net = S.bottleneck_unit(64, 16, 16, 10)
    ctx = b.Context(net.as_array(), (net.in_c, net.in_h, net.in_w), pool_bytes=64 << 20, host_bytes=16 << 20)
    params = S.init_params(net)
    img, lab = S.make_batch(net, k, 0)
    batch = torch.from_numpy(img).cuda()
    ctx.set_weights(params)
    ctx.plan_swaps(k, 64 << 20, b.PLAN_NAIVE_ALL)
    want = ctx.train_step(batch, lab, 0.1), ctx.get_weights()
    assert ctx.stats()["copies_in_order"] == (k == 2)
    late, a = torch.full_like(batch, float("nan")), torch.randn(4096, 4096, device="cuda")
    torch.cuda.synchronize()
    for _ in range(3):
        ctx.set_weights(params)
        late.fill_(float("nan"))
        torch.cuda.synchronize()
        with torch.cuda.stream(ctx.streams[2]):
            for _ in range(8):
                a = (a @ a).mul_(1e-3).clamp_(-1, 1)
            late.copy_(batch)
        got = ctx.train_step(late, lab, 0.1), ctx.get_weights()
        assert got[0] == want[0] and all((x == y).all() for x, y in zip(got[1], want[1]))
    ctx.close()
