"""What the speed of this library is measured on: calls of its public entry points, over the sizes,
storage types and directions that training the networks of synth/netspec.py puts them to.

A case is one layer (or a group of layers that only occur together) in every direction that an
iteration runs it in, through the acc_op_* calls, or one whole iteration through Context.train_step.
Sizes are those of the ResNets at 224 x 224 at the minibatches the tests and bench.py use, and, drawn,
anything of that range including ragged ones."""
import numpy as np
import torch

from paper_1901_06773_amd import binding as B
import synth as S

DEV = "cuda:0"
LR = 0.001                     # small: two such steps then differ by what rounding does to the gradients, not to the path
_DT = {"f32": torch.float32, "bf16": torch.bfloat16}


# ---------------------------------------------------------------------------------- the cases
def listed():
    return [
        # the end of a ResNet (global average pool, fully connected layer, softmax cross-entropy) at the
        # minibatch bench.py's tuner picks: a chain of small launches
        dict(name="head_f32_k41", kind="head", dtype="f32", n=41, hw=7, c=2048, classes=1000),
        # batch norm + ReLU of a conv4 bottleneck, forward and backward: 8 MB, latency matters
        dict(name="bn_f32_256_14x14_k41", kind="bn", dtype="f32", n=41, h=14, w=14, c=256, residual=False),
        # batch norm behind a shortcut (adds it, hands its gradient on) at a large bf16 minibatch: bandwidth
        dict(name="bn_bf16_512_28x28_k256_res", kind="bn", dtype="bf16", n=256, h=28, w=28, c=512, residual=True),
        # start of every ResNet: 7x7/2 convolution of the 3-channel images (no data gradient) and the 3x3/2 max-pool
        dict(name="stem_f32_224_k32", kind="stem", dtype="f32", n=32, h=224, w=224, cin=3, cout=64),
        # the layer with the largest share of ResNet-152's work, at bench.py's minibatch
        dict(name="conv3x3_f32_256_14x14_k41", kind="conv", dtype="f32", n=41, h=14, w=14, cin=256, cout=256, r=3, stride=1),
        # 1x1 expansion on large maps: short reductions, much memory traffic
        dict(name="conv1x1_f32_64to256_56x56_k32", kind="conv", dtype="f32", n=32, h=56, w=56, cin=64, cout=256, r=1, stride=1),
        # strided 3x3 of the basic-block and v1.5 networks on an odd map and minibatch (data gradient in parts)
        dict(name="conv3x3s2_f32_128_55x55_k19", kind="conv", dtype="f32", n=19, h=55, w=55, cin=128, cout=128, r=3, stride=2),
        # the same two kinds of layer at the bf16 minibatches
        dict(name="conv3x3_bf16_256_14x14_k512", kind="conv", dtype="bf16", n=512, h=14, w=14, cin=256, cout=256, r=3, stride=1),
        dict(name="conv1x1_bf16_512to128_28x28_k256", kind="conv", dtype="bf16", n=256, h=28, w=28, cin=512, cout=128, r=1, stride=1),
        # one iteration of a single bottleneck block with every feature map swapped out and back in
        dict(name="step_bottleneck_f32_k2_swap", kind="step", net="bottleneck", dtype="f32", k=2, hw=16, swap=True),
        # one iteration of ResNet-50 at minibatch 32, nothing swapped
        dict(name="step_resnet50_f32_k32", kind="step", net="resnet50", dtype="f32", k=32, hw=224, swap=False),
        # the same network in bf16 storage at a larger minibatch
        dict(name="step_resnet50_bf16_k128", kind="step", net="resnet50", dtype="bf16", k=128, hw=224, swap=False),
    ]


def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["conv"] * 6 + ["bn"] * 3 + ["stem", "head", "step"])
    dtype = rng.choice(["f32", "f32", "bf16"])
    if kind == "conv":
        r = rng.choice([1, 1, 3])
        step = 4 if dtype == "f32" else 8
        # usual widths, and widths that fill no tile
        cin, cout = (rng.choice([64, 128, 256, 512, rng.randrange(32, 513) // step * step]) for _ in range(2))
        h = _log(rng, 7, 56)
        w = h if rng.random() < 0.6 else max(7, h - rng.randrange(4))
        stride = 2 if rng.random() < 0.2 else 1
        most = 2.5e11 if dtype == "f32" else 1e12                  # flops of the three products
        cap = int(most / (6.0 * h * w * cin * cout * r * r / stride ** 2))
        n = _log(rng, 1, max(1, min(256, cap, int(1.6e9 / (4 * h * w * max(cin, cout))))))
        return dict(kind=kind, dtype=dtype, n=n, h=h, w=w, cin=cin, cout=cout, r=r, stride=stride)
    if kind == "bn":
        h = _log(rng, 7, 112)
        c = rng.choice([64, 128, 256, 512, 1024, 2048, rng.randrange(16, 1025) // 4 * 4])
        n = _log(rng, 1, max(1, min(512, int(1e8 / (h * h * c)))))
        return dict(kind=kind, dtype=dtype, n=n, h=h, w=h, c=c, residual=rng.random() < 0.4)
    if kind == "stem":
        h = rng.choice([224, 192, 224 - rng.randrange(60)])
        return dict(kind=kind, dtype=dtype, n=_log(rng, 2, 40), h=h, w=h, cin=3, cout=64)
    if kind == "head":
        return dict(kind=kind, dtype=dtype, n=_log(rng, 2, 256), hw=rng.choice([4, 6, 7, 8]),
                    c=rng.choice([512, 1024, 2048]), classes=rng.choice([10, 100, 1000]))
    if rng.random() < 0.5:
        hw = rng.randrange(8, 57)
        return dict(kind="step", net="bottleneck", dtype=dtype, k=_log(rng, 2, max(2, 16384 // hw ** 2)), hw=hw, swap=rng.random() < 0.5)
    return dict(kind="step", net=rng.choice(["resnet18", "resnet34"]), dtype=dtype, k=rng.randrange(16, 33),
                hw=rng.choice([128, 160, 192, 224]), swap=False)


# ---------------------------------------------------------------------------------- inputs
def _gen(seed, salt):
    return torch.Generator(device=DEV).manual_seed((int(seed) * 1000003 + salt) % (1 << 62))


def _randn(seed, salt, shape, dtype, scale=1.0, shift=0.0):
    t = torch.randn(shape, generator=_gen(seed, salt), device=DEV, dtype=torch.float32)
    return t.mul_(scale).add_(shift).to(dtype)


def _out(x, r, stride, pad):
    return (x + 2 * pad - r) // stride + 1


def _conv_inputs(case, seed):
    n, h, w, cin, cout, r, stride = (case[k] for k in ("n", "h", "w", "cin", "cout", "r", "stride"))
    dt, pad = _DT[case["dtype"]], r // 2
    ho, wo = _out(h, r, stride, pad), _out(w, r, stride, pad)
    x = _randn(seed, 1, (n, h, w, cin), dt).relu_()                           # what a ReLU hands on
    wt = _randn(seed, 2, (cout, r, r, cin), dt, (2.0 / (cin * r * r)) ** 0.5)   # He-normal, O-H-W-I
    dy = _randn(seed, 3, (n, ho, wo, cout), dt, 1e-3)
    return x, wt, dy, pad


def _bn_inputs(case, seed):
    n, h, w, c = (case[k] for k in ("n", "h", "w", "c"))
    dt = _DT[case["dtype"]]
    x = _randn(seed, 1, (n, h, w, c), dt, 1.0, 0.1)
    gamma = _randn(seed, 2, (c,), torch.float32, 0.1, 1.0)
    beta = _randn(seed, 3, (c,), torch.float32, 0.1)
    res = _randn(seed, 4, (n, h, w, c), dt) if case["residual"] else None
    dy = _randn(seed, 5, (n, h, w, c), dt, 1e-3)
    # what an earlier forward pass of such a layer has saved for the backward pass
    xf = x.float().reshape(-1, c)
    mean = xf.mean(0)
    istd = (xf.var(0, unbiased=False) + 1e-5).rsqrt()
    y = ((x.float() - mean) * istd * gamma + beta + (res.float() if res is not None else 0.0)).relu().to(dt)
    return x, gamma, beta, res, dy, mean, istd, y


def _stem_inputs(case, seed):
    n, h, w, cin, cout = (case[k] for k in ("n", "h", "w", "cin", "cout"))
    dt = _DT[case["dtype"]]
    ho, wo = _out(h, 7, 2, 3), _out(w, 7, 2, 3)
    po, qo = _out(ho, 3, 2, 1), _out(wo, 3, 2, 1)
    x = _randn(seed, 1, (n, h, w, cin), dt)
    wt = _randn(seed, 2, (cout, 7, 7, cin), dt, (2.0 / (cin * 49)) ** 0.5)
    dy = _randn(seed, 3, (n, ho, wo, cout), dt, 1e-3)
    act = _randn(seed, 4, (n, ho, wo, cout), dt).relu_()                      # what the batch norm between the two hands on
    dp = _randn(seed, 5, (n, po, qo, cout), dt, 1e-3)
    return x, wt, dy, act, dp


def _head_inputs(case, seed):
    n, hw, c, classes = (case[k] for k in ("n", "hw", "c", "classes"))
    dt = _DT[case["dtype"]]
    x = _randn(seed, 1, (n, hw, hw, c), dt).relu_()
    wt = _randn(seed, 2, (classes, 1, 1, c), dt, (2.0 / c) ** 0.5)
    labels = torch.randint(0, classes, (n,), generator=_gen(seed, 3), device=DEV, dtype=torch.int32)
    feat = _randn(seed, 4, (n, 1, 1, c), dt, 0.1, 0.4)                        # saved for the weight gradient
    dz = _randn(seed, 5, (n, 1, 1, classes), dt, 1e-3)
    return x, wt, labels, feat, dz


def _net(case):
    if case["net"] == "bottleneck":
        return S.bottleneck_unit(64, 16, case["hw"], 10)
    return getattr(S, case["net"])(in_hw=case["hw"])


def _step_inputs(case, seed):
    net, k = _net(case), case["k"]
    params = []
    for i, l in enumerate(net.layers):                                        # He-normal, gamma 1, beta and bias 0; host, OIHW
        if l.kind in (S.CONV, S.FC):
            fan_in = l.cin * (l.r * l.s if l.kind == S.CONV else 1)
            p = _randn(seed, 100 + i, (l.cout * fan_in,), torch.float32, (2.0 / fan_in) ** 0.5).cpu().numpy()
            params.append(p if l.kind == S.CONV else np.concatenate([p, np.zeros(l.cout, np.float32)]))
        elif l.kind == S.BN:
            params.append(np.concatenate([np.ones(l.cin, np.float32), np.zeros(l.cin, np.float32)]))
        else:
            params.append(np.zeros(0, np.float32))
    images = _randn(seed, 1, (k, net.in_c, net.in_h, net.in_w), torch.float32)
    labels = torch.randint(0, net.classes, (k,), generator=_gen(seed, 2), device=DEV, dtype=torch.int32).cpu().numpy()
    return net, params, images, labels


def prepare(case, seed):
    kind, dt = case["kind"], _DT[case["dtype"]]
    s = dict(case=case)
    if kind == "conv":
        x, wt, dy, pad = _conv_inputs(case, seed)
        n, h, w, cin = x.shape
        ws = B.op_conv_workspace(n, h, w, cin, wt.shape[0], wt.shape[1], case["stride"], pad)
        s.update(x=x, w=wt, dy=dy, pad=pad, y=torch.empty_like(dy), dx=torch.empty_like(x),
                 dw=torch.empty(wt.shape, device=DEV), ws=torch.empty(max(ws, 256), dtype=torch.uint8, device=DEV))
    elif kind == "bn":
        x, gamma, beta, res, dy, mean, istd, y = _bn_inputs(case, seed)
        c = case["c"]
        f = [torch.empty(c, device=DEV) for _ in range(4)]
        s.update(x=x, gamma=gamma, beta=beta, res=res, dy=dy, mean=mean, istd=istd, y_saved=y, y=torch.empty_like(x),
                 dx=torch.empty_like(x), g=torch.empty_like(x) if res is not None else None, f=f,
                 ws=torch.empty(B.op_bn_workspace(c), dtype=torch.uint8, device=DEV))
    elif kind == "stem":
        x, wt, dy, act, dp = _stem_inputs(case, seed)
        n, h, w, cin = x.shape
        ws = B.op_conv_workspace(n, h, w, cin, wt.shape[0], 7, 2, 3)
        s.update(x=x, w=wt, dy=dy, act=act, dp=dp, y=torch.empty_like(dy), p=torch.empty_like(dp), da=torch.empty_like(act),
                 dw=torch.empty(wt.shape, device=DEV), ws=torch.empty(max(ws, 256), dtype=torch.uint8, device=DEV))
    elif kind == "head":
        x, wt, labels, feat, dz = _head_inputs(case, seed)
        n, classes, c = x.shape[0], wt.shape[0], x.shape[3]
        ws = B.op_conv_workspace(n, 1, 1, c, classes, 1, 1, 0)
        s.update(x=x, w=wt, labels=labels, feat=feat, dz=dz, f=torch.empty((n, 1, 1, c), dtype=dt, device=DEV),
                 z=torch.empty((n, 1, 1, classes), dtype=dt, device=DEV), rows=torch.empty(n, device=DEV),
                 loss=torch.empty(1, device=DEV), sz=torch.empty((n, classes), dtype=dt, device=DEV),
                 df=torch.empty((n, 1, 1, c), dtype=dt, device=DEV), dx=torch.empty_like(x),
                 dw=torch.empty(wt.shape, device=DEV), ws=torch.empty(max(ws, 256), dtype=torch.uint8, device=DEV))
    else:
        net, params, images, labels = _step_inputs(case, seed)
        code = B.BF16 if case["dtype"] == "bf16" else B.F32
        probe = B.Context(net.as_array(), (net.in_c, net.in_h, net.in_w), dtype=code)
        need = probe.plan_swaps(case["k"], 1 << 38, B.PLAN_NONE)["peak_bytes"]
        maps = probe.plan_swaps(case["k"], 1 << 38, B.PLAN_NAIVE_ALL)["host_bytes"] if case["swap"] else 0
        probe.close()
        pool = (int(need * 1.1) + (8 << 20)) // 256 * 256
        ctx = B.Context(net.as_array(), (net.in_c, net.in_h, net.in_w), pool_bytes=pool, host_bytes=int(maps) + 4096, dtype=code)
        ctx.set_weights(params)
        ctx.plan_swaps(case["k"], pool, B.PLAN_NAIVE_ALL if case["swap"] else B.PLAN_NONE)
        # the caller owns the pool; the fp32 weights lie at its start, the gradients behind them (each tensor
        # rounded up to 64 elements)
        elems = sum((n + 63) // 64 * 64 for n in net.param_sizes())
        view = ctx.pool[: 8 * elems].view(torch.float32)
        torch.cuda.synchronize()
        s.update(ctx=ctx, images=images, labels=labels, weights=view[:elems], grads=view[elems:])
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "conv":
        B.op_conv_fwd(s["x"], s["w"], s["y"], case["stride"], s["pad"])
        B.op_conv_dgrad(s["dy"], s["w"], s["dx"], case["stride"], s["pad"], s["ws"])
        B.op_conv_wgrad(s["x"], s["dy"], s["dw"], case["stride"], s["pad"], s["ws"])
        return s["y"], s["dx"], s["dw"]
    if kind == "bn":
        mean, istd, dgamma, dbeta = s["f"]
        B.op_bn_fwd(s["x"], s["gamma"], s["beta"], s["res"], s["y"], mean, istd, True, 1e-5, s["ws"])
        B.op_bn_bwd(s["x"], s["dy"], s["y_saved"], s["gamma"], s["mean"], s["istd"], s["dx"], dgamma, dbeta, s["g"], s["ws"])
        return (s["y"], mean, istd, s["dx"], dgamma, dbeta) + ((s["g"],) if s["g"] is not None else ())
    if kind == "stem":
        B.op_conv_fwd(s["x"], s["w"], s["y"], 2, 3)
        B.op_maxpool_fwd(s["act"], s["p"], 3, 2, 1)
        B.op_maxpool_bwd(s["act"], s["dp"], s["da"], 3, 2, 1)
        B.op_conv_wgrad(s["x"], s["dy"], s["dw"], 2, 3, s["ws"])
        return s["y"], s["p"], s["da"], s["dw"]
    if kind == "head":
        n, classes = s["z"].shape[0], s["z"].shape[3]
        B.op_gap_fwd(s["x"], s["f"].view(n, -1))
        B.op_conv_fwd(s["f"], s["w"], s["z"], 1, 0)
        B.op_softmax_ce(s["z"].view(n, classes), s["labels"], s["rows"], s["loss"], s["sz"])
        B.op_conv_wgrad(s["feat"], s["dz"], s["dw"], 1, 0, s["ws"])
        B.op_conv_dgrad(s["dz"], s["w"], s["df"], 1, 0, s["ws"])
        B.op_gap_bwd(s["df"].view(n, -1), s["dx"])
        return s["f"], s["z"], s["rows"], s["loss"], s["sz"], s["dw"], s["df"], s["dx"]
    loss = s["ctx"].train_step(s["images"], s["labels"], LR)
    # a gradient tensor depends on ReLU decisions within rounding of zero, on which no two implementations
    # agree where there are many (two per cent in ResNet-50): large steps return the updated weights only
    return (loss, s["weights"], s["grads"]) if _few_decisions(case) else (loss, s["weights"])


def _few_decisions(case):
    return case["dtype"] == "f32" and case["net"] == "bottleneck" and case["k"] * case["hw"] ** 2 <= 1024


# ---------------------------------------------------------------------------------- what a pass cannot do without
def _layer_shapes(net):
    """(layer, input (c, h, w), output (c, h, w)) of every layer."""
    shp, out = [], []
    for l in net.layers:
        c, h, w = shp[l.in0] if l.in0 >= 0 else (net.in_c, net.in_h, net.in_w)
        if l.kind in (S.CONV, S.MAXPOOL):
            o = (l.cout, _out(h, l.r, l.stride, l.pad), _out(w, l.s, l.stride, l.pad))
        elif l.kind in (S.GAP, S.FC):
            o = (l.cout if l.kind == S.FC else c, 1, 1)
        else:
            o = (c, h, w)
        shp.append(o)
        out.append((l, (c, h, w), o))
    return out


def work(case):
    es = 2 if case["dtype"] == "bf16" else 4
    kind = case["kind"]
    if kind == "conv":
        n, h, w, cin, cout, r, st = (case[k] for k in ("n", "h", "w", "cin", "cout", "r", "stride"))
        m = n * _out(h, r, st, r // 2) * _out(w, r, st, r // 2)
        x, y, f = n * h * w * cin, m * cout, cin * cout * r * r
        return {"bytes": es * (2 * x + 2 * y + f) + 4 * f, "flops": 6.0 * m * f}
    if kind == "bn":
        e = case["n"] * case["h"] * case["w"] * case["c"]
        # forward x (+ shortcut) -> y; backward x, dy, y -> dx (+ masked gradient); x is one input
        return {"bytes": es * e * (7 if case["residual"] else 5) + 32 * case["c"], "flops": 20.0 * e}
    if kind == "stem":
        n, cin, cout = case["n"], case["cin"], case["cout"]
        ho, wo = _out(case["h"], 7, 2, 3), _out(case["w"], 7, 2, 3)
        po, qo = _out(ho, 3, 2, 1), _out(wo, 3, 2, 1)
        f = cout * 49 * cin
        return {"bytes": es * (n * case["h"] * case["w"] * cin + 4 * n * ho * wo * cout + 2 * n * po * qo * cout + f) + 4 * f,
                "flops": 4.0 * n * ho * wo * f}
    if kind == "head":
        n, c, cl, p = case["n"], case["c"], case["classes"], case["hw"] ** 2
        return {"bytes": es * (2 * n * p * c + 3 * n * c + 3 * n * cl + c * cl) + 4 * c * cl + 12 * n, "flops": 6.0 * n * c * cl}
    net, k = _net(case), case["k"]
    flops = bytes_ = 0.0
    for l, (ci, hi, wi), (co, ho, wo) in _layer_shapes(net):
        if l.kind in (S.CONV, S.FC):
            fl = 2.0 * k * ho * wo * co * ci * (l.r * l.s if l.kind == S.CONV else 1)
            flops += fl * (2 if l.in0 < 0 else 3)
            bytes_ += es * k * 2 * co * ho * wo            # output written, gradient read (inputs: the batch norms' outputs)
        elif l.kind == S.BN:
            bytes_ += es * k * 5 * co * ho * wo            # forward x -> y, backward x, dy -> dx
    bytes_ += 12.0 * sum(net.param_sizes()) + 4.0 * k * net.in_c * net.in_h * net.in_w
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    if case["kind"] == "step":
        if case["dtype"] == "bf16":
            return {"rel": 1e-2, "max": 0.2}
        return {"rel": 1e-5} if case["net"] == "bottleneck" else {"rel": 1e-3, "max": 0.1}
    return {"rel": 1e-5} if case["dtype"] == "f32" else {"rel": 8e-3, "max": 0.1}


# ---------------------------------------------------------------------------------- the same in 64 bits
def _conv64(x, w, stride, pad):
    """NHWC x, O-H-W-I w, float64: one product per filter tap."""
    n, h, wd, c = x.shape
    cout, r, s, _ = w.shape
    ho, wo = _out(h, r, stride, pad), _out(wd, s, stride, pad)
    xp = torch.nn.functional.pad(x, (0, 0, pad, pad, pad, pad)) if pad else x
    y = None
    for a in range(r):
        for b in range(s):
            v = xp[:, a:a + (ho - 1) * stride + 1:stride, b:b + (wo - 1) * stride + 1:stride, :].reshape(-1, c)
            t = v @ w[:, a, b, :].t()
            y = t if y is None else y + t
    return y.view(n, ho, wo, cout)


def _conv64_grads(x, w, dy, stride, pad, need_dx=True):
    n, h, wd, c = x.shape
    cout, r, s, _ = w.shape
    ho, wo = dy.shape[1:3]
    xp = torch.nn.functional.pad(x, (0, 0, pad, pad, pad, pad)) if pad else x
    dxp = torch.zeros_like(xp) if need_dx else None
    dw = torch.empty_like(w)
    g = dy.reshape(-1, cout)
    for a in range(r):
        for b in range(s):
            at = (slice(None), slice(a, a + (ho - 1) * stride + 1, stride), slice(b, b + (wo - 1) * stride + 1, stride))
            dw[:, a, b, :] = g.t() @ xp[at].reshape(-1, c)
            if need_dx:
                dxp[at] += (g @ w[:, a, b, :]).view(n, ho, wo, c)
    return (dxp[:, pad:pad + h, pad:pad + wd, :].contiguous() if need_dx else None), dw


def _pool64(x):
    """3x3 / 2 max-pool, padding 1, and for every output the index of its first maximum in scan order."""
    v = torch.nn.functional.pad(x.permute(0, 3, 1, 2), (1, 1, 1, 1), value=-float("inf"))
    n, c, h, w = v.shape
    ho, wo = (h - 3) // 2 + 1, (w - 3) // 2 + 1
    best, at = None, None
    for a in range(3):
        for b in range(3):
            t = v[:, :, a:a + 2 * ho - 1:2, b:b + 2 * wo - 1:2]
            if best is None:
                best, at = t.clone(), torch.zeros(t.shape, dtype=torch.int64, device=t.device)
            else:
                more = t > best
                best = torch.where(more, t, best)
                at = torch.where(more, torch.full_like(at, 3 * a + b), at)
    return best, at


def _step64(case, seed):
    net, params, images, labels = _step_inputs(case, seed)
    leaves, vals = [], []
    for l, p in zip(net.layers, params):
        t = torch.from_numpy(p).to(DEV).double()
        if l.kind == S.CONV:
            t = t.view(l.cout, l.cin, l.r, l.s).permute(0, 2, 3, 1).contiguous()
        leaves.append(t.requires_grad_(t.numel() > 0))
    x_in = images.double().permute(0, 2, 3, 1).contiguous()
    loss = None
    for l, p in zip(net.layers, leaves):
        x = vals[l.in0] if l.in0 >= 0 else x_in
        if l.kind == S.CONV:
            y = _conv64(x, p, l.stride, l.pad)
        elif l.kind == S.BN:
            c = l.cin
            f = x.reshape(-1, c)
            mean = f.mean(0)
            var = (f - mean).square().mean(0)
            y = (x - mean) * (var + 1e-5).rsqrt() * p[:c] + p[c:]
        elif l.kind == S.RELU:
            y = x.relu()
        elif l.kind == S.ADD:
            y = x + (vals[l.in1] if l.in1 >= 0 else x_in)
        elif l.kind == S.MAXPOOL:
            n, h, w, c = x.shape
            y = torch.nn.functional.max_pool2d(x.permute(0, 3, 1, 2), l.r, l.stride, l.pad).permute(0, 2, 3, 1).contiguous()
        elif l.kind == S.GAP:
            y = x.mean((1, 2))
        elif l.kind == S.FC:
            y = x.reshape(x.shape[0], -1) @ p[: l.cout * l.cin].view(l.cout, l.cin).t() + p[l.cout * l.cin:]
        else:
            loss = torch.nn.functional.cross_entropy(x, torch.from_numpy(labels).to(DEV).long())
            y = loss
        vals.append(y)
    loss.backward()

    def flat(ts):
        out = []
        for t in ts:
            t = t.reshape(-1)
            out.append(torch.nn.functional.pad(t, (0, (-t.numel()) % 64)))
        return torch.cat(out)
    some = [t for t in leaves if t.numel()]
    grads = flat([t.grad for t in some])
    weights = flat([t.detach() for t in some]) - LR * grads
    # the loss is one number, and its distance from this one draw of the rounding
    first = (None, weights)
    return first + (grads,) if _few_decisions(case) else first


def exact(case, seed):
    kind = case["kind"]
    if kind == "conv":
        x, w, dy, pad = _conv_inputs(case, seed)
        x, w, dy = x.double(), w.double(), dy.double()
        y = _conv64(x, w, case["stride"], pad)
        dx, dw = _conv64_grads(x, w, dy, case["stride"], pad)
        return y, dx, dw
    if kind == "bn":
        x, gamma, beta, res, dy, mean, istd, y_saved = (t.double() if t is not None else None for t in _bn_inputs(case, seed))
        c = case["c"]
        f = x.reshape(-1, c)
        m = f.mean(0)
        i = ((f - m).square().mean(0) + 1e-5).rsqrt()
        y = ((x - m) * i * gamma + beta + (res if res is not None else 0.0)).relu()
        g = torch.where(y_saved > 0, dy, torch.zeros_like(dy))
        xh = (x - mean) * istd
        dbeta = g.reshape(-1, c).sum(0)
        dgamma = (g * xh).reshape(-1, c).sum(0)
        rows = f.shape[0]
        dx = gamma * istd * (g - dbeta / rows - xh * dgamma / rows)
        return (y, m, i, dx, dgamma, dbeta) + ((g,) if res is not None else ())
    if kind == "stem":
        x, w, dy, act, dp = (t.double() for t in _stem_inputs(case, seed))
        y = _conv64(x, w, 2, 3)
        dw = _conv64_grads(x, w, dy, 2, 3, need_dx=False)[1]
        p, at = _pool64(act)
        n, ho, wo, c = act.shape
        da = torch.zeros((n, c, ho + 2, wo + 2), dtype=torch.float64, device=DEV)
        d = dp.permute(0, 3, 1, 2)
        po, qo = d.shape[2:]
        for a in range(3):
            for b in range(3):
                da[:, :, a:a + 2 * po - 1:2, b:b + 2 * qo - 1:2] += torch.where(at == 3 * a + b, d, torch.zeros_like(d))
        return (y, p.permute(0, 2, 3, 1).contiguous(), da[:, :, 1:1 + ho, 1:1 + wo].permute(0, 2, 3, 1).contiguous(), dw)
    if kind == "head":
        x, w, labels, feat, dz = _head_inputs(case, seed)
        n, c, classes = x.shape[0], x.shape[3], w.shape[0]
        x, w2, feat, dz = x.double(), w.double().view(classes, c), feat.double().view(n, c), dz.double().view(n, classes)
        f = x.mean((1, 2))
        # the fully connected layer and the loss read the stored (rounded) results before them
        z = f.to(_DT[case["dtype"]]).double() @ w2.t()
        lsm = torch.log_softmax(z.to(_DT[case["dtype"]]).double(), 1)
        rows = -lsm.gather(1, labels.long()[:, None])[:, 0]
        sz = lsm.exp()
        sz[torch.arange(n, device=DEV), labels.long()] -= 1.0
        df = dz @ w2
        dx = (df.to(_DT[case["dtype"]]).double() / case["hw"] ** 2).view(n, 1, 1, c).expand(n, case["hw"], case["hw"], c).contiguous()
        return (f.view(n, 1, 1, c), z.view(n, 1, 1, classes), rows, rows.mean().view(1), sz / n, (dz.t() @ feat).view(classes, 1, 1, c),
                df.view(n, 1, 1, c), dx)
    return _step64(case, seed)
