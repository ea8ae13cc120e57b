"""The work whose speed matters in this framework, case by case.

Whole checkpointed training steps of the four network kinds (`train_step`, as
bench.py and a training loop call it) and the layers the bfloat16 ResNet is
composed of (the `op_*` calls): smallest and largest shapes, each plan mode,
forward and backward, float32 and bfloat16.  A step returns the loss and every
parameter gradient; a layer returns every tensor it forms.

Kinds:
  mlp     residual MLP chain, float32
  cifar   CIFAR-shaped basic-block ResNet, float32
  lstm    unrolled LSTM with a softmax head per step, bfloat16 products
  resnet  ImageNet-shaped bottleneck ResNet, bfloat16
  conv    one convolution - batch norm - ReLU layer forward, bfloat16
  grad    one convolution's backward with the batch norm before it, bfloat16
  bn      the masked batch-norm backward of a block's output, bfloat16
"""
import math

import torch

from paper_1604_06174_amd import ckpt as K

DEV = "cuda:0"
EPS = 1e-5


def listed():
    return [
        # 64 blocks of width 256 at batch 64, a boundary every 8: launches and latency
        dict(name="mlp_64x256", kind="mlp", batch=64, depth=64, width=256, plan="sqrt", arg=8),
        # the wide chain of the recursive schedule (width 1024, batch 256), 128 of its 1024 blocks
        dict(name="mlp_128x1024_recursive", kind="mlp", batch=256, depth=128, width=1024, plan="recursive", arg=1),
        # the 110-layer CIFAR network at its training batch
        dict(name="cifar110", kind="cifar", batch=128, blocks=18, base=16, image=32, classes=10, drop=0,
             plan="sqrt", arg=0),
        # a small one with an odd batch, keeping convolution outputs only: a fine-tuning or debugging size
        dict(name="cifar20_b37_drop", kind="cifar", batch=37, blocks=3, base=16, image=32, classes=10, drop=1,
             plan="greedy", arg=25),
        # the speech-sized LSTM (1024 hidden, 10k vocabulary, batch 64), a boundary every 64 steps
        dict(name="lstm_t256", kind="lstm", T=256, batch=64, input=1024, hidden=1024, vocab=10000, plan="sqrt",
             arg=64),
        # a small LSTM with ragged sizes under the recursive plan (single-step segments)
        dict(name="lstm_small_recursive", kind="lstm", T=50, batch=20, input=136, hidden=256, vocab=1000,
             plan="recursive", arg=1),
        # the 1000-layer ResNet's stem and first three stages (most blocks are in the third) at its batch,
        # image and budget; few blocks, since bfloat16 gradients of more are not comparable between
        # implementations
        dict(name="resnet_1_1_2", kind="resnet", batch=32, blocks="1-1-2", width=64, image=224, classes=1000, drop=0,
             plan="greedy", arg=10),
        # its most frequent layer: the 3x3 of stage 3, forward
        dict(name="conv3x3_256_fwd", kind="conv", n=32, side=14, ci=256, co=256, r=3, s=1, res=0),
        # the expansion of stage 1 with the identity shortcut: its largest activations
        dict(name="conv1x1_64_256_fwd", kind="conv", n=32, side=56, ci=64, co=256, r=1, s=1, res=1),
        # backward of a 3x3 of stage 2: data gradient, the batch norm before it, weight gradient
        dict(name="conv3x3_128_bwd", kind="grad", n=32, side=28, ci=128, co=128, r=3, s=1),
        # backward of the expansion of stage 3
        dict(name="conv1x1_256_1024_bwd", kind="grad", n=32, side=14, ci=256, co=1024, r=1, s=1),
        # a block output's batch-norm backward in stage 2
        dict(name="bn_512_bwd", kind="bn", n=32, side=28, c=512),
    ]


def _log(rng, lo, hi):
    """An integer of [lo, hi], uniform in its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _plan(rng, modes, n):
    mode = rng.choice(modes)
    arg = {"sqrt": rng.choice([0, 0, max(1, n // 4)]), "greedy": rng.randint(8, 40), "recursive": rng.choice([1, 1, 3]),
           "none": 0}[mode]
    return dict(plan=mode, arg=arg)


def draw(rng):
    kind = rng.choice(["mlp", "mlp", "cifar", "lstm", "lstm", "resnet", "conv", "conv", "grad", "grad", "bn"])
    if kind == "mlp":
        width = _log(rng, 24, 1024)
        depth = _log(rng, 4, 128)
        return dict(kind=kind, batch=_log(rng, 1, 256), depth=depth, width=width,
                    **_plan(rng, ["sqrt", "recursive", "greedy", "none"], depth))
    if kind == "cifar":
        blocks = _log(rng, 1, 18)
        base = rng.choice([8, 16])
        return dict(kind=kind, batch=_log(rng, 2, 128), blocks=blocks, base=base, image=rng.choice([16, 32]),
                    classes=rng.choice([7, 10, 100]), drop=rng.randint(0, 1),
                    **_plan(rng, ["sqrt", "greedy", "none"], 3 * blocks))
    if kind == "lstm":
        T = _log(rng, 4, 192)
        big = rng.random() < 0.5
        h = 1024 if big else 8 * _log(rng, 4, 96)
        e = h if big or rng.random() < 0.5 else 8 * _log(rng, 4, 96)
        return dict(kind=kind, T=T, batch=64 if big else _log(rng, 1, 64), input=e, hidden=h,
                    vocab=10000 if big else 8 * _log(rng, 8, 1000),
                    **_plan(rng, ["sqrt", "recursive", "greedy", "none"], T))
    if kind == "resnet":
        return dict(kind=kind, batch=_log(rng, 4, 32), 
                    blocks=rng.choice(["1", "2", "1-1", "1-2", "2-1", "1-1-1", "1-1-2"]),
                    width=rng.choice([32, 64]), image=rng.choice([96, 160, 224]), classes=rng.choice([10, 1000]),
                    drop=rng.randint(0, 1), **_plan(rng, ["greedy", "sqrt", "none"], 8))
    stage = rng.randint(0, 3)
    w, side, n = 64 << stage, 56 >> stage, _log(rng, 2, 32)
    if rng.random() < 0.3:
        side = rng.choice([side - 1, side - side // 4, side + 2])
    if kind == "bn":
        return dict(kind=kind, n=n, side=side, c=rng.choice([w, 4 * w]))
    r = rng.choice([1, 3])
    ci, co = (w, w) if r == 3 else rng.choice([(w, 4 * w), (4 * w, w)])
    if kind == "grad":
        return dict(kind=kind, n=n, side=side, ci=ci, co=co, r=r, s=rng.choice([1, 1, 2]) if r == 3 else 1)
    return dict(kind=kind, n=n, side=side, ci=ci, co=co, r=r, s=rng.choice([1, 1, 2]) if r == 3 else 1,
                res=int(co > ci))


# ------------------------------------------------------------------ inputs --
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _randn(g, *shape, scale=1.0):
    return torch.randn(*shape, generator=g, device=DEV) * scale


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device=DEV)


def _labels(g, k, *shape):
    return torch.randint(0, k, shape, generator=g, device=DEV, dtype=torch.int32)


def _he(g, co, r, ci):
    return _randn(g, co, r, r, ci, scale=math.sqrt(2.0 / (r * r * ci)))


def _cifar_blocks(case):
    """(parameter prefix, input channels, output channels, stride) of every basic block."""
    out, cin = [], case["base"]
    for s in range(3):
        for j in range(case["blocks"]):
            cout = case["base"] << s
            out.append(("u%d." % (len(out) + 1), cin, cout, 2 if s > 0 and j == 0 else 1))
            cin = cout
    return out


def _stages(case):
    return [int(b) for b in case["blocks"].split("-")]


def _resnet_blocks(case):
    """(parameter prefix, input channels, inner width, stride, projection) of every bottleneck block."""
    out, cin = [], 64
    for t, nb in enumerate(_stages(case)):
        w = case["width"] << t
        for j in range(nb):
            out.append(("u%d." % (len(out) + 1), cin, w, 2 if t > 0 and j == 0 else 1, j == 0))
            cin = 4 * w
    return out


def _net_inputs(case, seed):
    """The batch and the parameters of a network, by name in their order: He-normal
    convolutions, batch norms at 1 and 0, uniform heads, normal or uniform batches."""
    g = _gen(seed)
    kind, p = case["kind"], {}

    def bn(name, c):
        p[name[0]], p[name[1]] = torch.ones(c, device=DEV), torch.zeros(c, device=DEV)

    def fc(cin, k):
        p["head.W"] = (2 * _rand(g, cin, k) - 1) / math.sqrt(cin)
        p["head.b"] = (2 * _rand(g, k) - 1) / math.sqrt(cin)

    if kind == "mlp":
        x, t = _randn(g, case["batch"], case["width"]), _randn(g, case["batch"], case["width"])
        for i in range(case["depth"]):
            p["u%d.W" % i] = _randn(g, case["width"], case["width"], scale=(case["width"] * case["depth"]) ** -0.5)
            p["u%d.b" % i] = torch.zeros(case["width"], device=DEV)
        return x, t, p
    if kind == "lstm":
        T, B, E, H, V = (case[k] for k in ("T", "batch", "input", "hidden", "vocab"))
        x, t = _randn(g, T, B, E).bfloat16(), _labels(g, V, T, B)
        for name, shape in (("W_x", (E, 4 * H)), ("W_h", (H, 4 * H)), ("b", (4 * H,)), ("W_o", (H, V)), ("b_o", (V,))):
            p[name] = (2 * _rand(g, *shape) - 1) / 32
        return x, t, p
    x = _rand(g, case["batch"], case["image"], case["image"], 3)
    t = _labels(g, case["classes"], case["batch"])
    if kind == "cifar":
        p["u0.W"] = _he(g, case["base"], 3, 3)
        bn(("u0.gamma", "u0.beta"), case["base"])
        for u, ci, co, _ in _cifar_blocks(case):
            p[u + "W1"] = _he(g, co, 3, ci)
            bn((u + "gamma1", u + "beta1"), co)
            p[u + "W2"] = _he(g, co, 3, co)
            bn((u + "gamma2", u + "beta2"), co)
        fc(4 * case["base"], case["classes"])
        return x, t, p
    p["u0.W"] = _he(g, 64, 7, 3)
    bn(("u0.gamma", "u0.beta"), 64)
    for u, ci, w, _, proj in _resnet_blocks(case):
        for k, (co, r, c) in enumerate(((w, 1, ci), (w, 3, w), (4 * w, 1, w))):
            p[u + "W%d" % (k + 1)] = _he(g, co, r, c)
            bn((u + "gamma%d" % (k + 1), u + "beta%d" % (k + 1)), co)
        if proj:
            p[u + "Wp"] = _he(g, 4 * w, 1, ci)
            bn((u + "gammap", u + "betap"), 4 * w)
    fc(4 * w, case["classes"])
    return x.bfloat16(), t, p


def _parts(offs):
    """Where the flat gradient buffer is cut into at most 48 outputs of whole parameters."""
    return offs[::-(-len(offs) // 48)]


def _net(case):
    kind = case["kind"]
    if kind == "mlp":
        return K.net_create(K.NET_MLP, case["batch"], case["depth"], case["width"])
    if kind == "cifar":
        return K.net_create(K.NET_RESNET_BASIC, case["batch"], case["blocks"], case["base"], case["image"],
                            case["classes"], drop_bn_relu=case["drop"])
    if kind == "lstm":
        return K.net_create(K.NET_LSTM, case["batch"], case["T"], case["hidden"], case["input"], case["vocab"])
    return K.net_create(K.NET_RESNET_BOTTLENECK, case["batch"], len(_stages(case)), case["width"], case["image"],
                        case["classes"], stage_blocks=_stages(case), expansion=4, stem_channels=64,
                        drop_bn_relu=case["drop"])


def _prepare_net(case, seed):
    net = _net(case)
    x, t, p = _net_inputs(case, seed)
    flat = torch.zeros(net.param_bytes() // 4, device=DEV)
    grads = torch.zeros_like(flat)
    layout = net.param_layout()
    for name, off, numel in layout:
        flat[off // 4:off // 4 + numel] = p[name].reshape(-1)
    starts = _parts([off // 4 for _, off, _ in layout])
    views = [grads[a:b] for a, b in zip(starts, starts[1:] + [grads.numel()])]
    lb, cb = net.layer_sizes()
    mode = dict(none=K.NONE, sqrt=K.SQRT, greedy=K.GREEDY, recursive=K.RECURSIVE)[case["plan"]]
    plan = K.plan_checkpoints(lb, cb, sum(lb) * case["arg"] // 100 if case["plan"] == "greedy" else case["arg"], mode)
    need = net.workspace_bytes(plan)
    return dict(case=case, net=net, plan=plan, x=x.contiguous(), t=t, params=flat, grads=grads, views=views,
                ws=torch.empty(need, dtype=torch.uint8, device=DEV), need=need, loss=torch.zeros(1, device=DEV))


def _side_out(case):
    return (case["side"] + 2 * (case["r"] // 2) - case["r"]) // case["s"] + 1


def _stats(c):
    """mean | 1/std over the rows of a [rows, channels] matrix."""
    d = c.double()
    m = d.mean(0)
    return torch.cat([m, ((d - m) ** 2).mean(0).add(EPS).rsqrt()]).float()


def _layer_inputs(case, seed):
    g = _gen(seed)
    if case["kind"] == "bn":
        m, c = case["n"] * case["side"] ** 2, case["c"]
        cv = _randn(g, m, c).bfloat16()
        return dict(g=_randn(g, m, c, scale=1e-3), ym=torch.relu(_randn(g, m, c)).bfloat16(), c=cv, st=_stats(cv),
                    gamma=1 + 0.1 * _randn(g, c))
    ci, co, r = case["ci"], case["co"], case["r"]
    mi, mo = case["n"] * case["side"] ** 2, case["n"] * _side_out(case) ** 2
    d = dict(x=torch.relu(_randn(g, mi, ci)).bfloat16(), w=_he(g, co, r, ci).bfloat16())
    if case["kind"] == "conv":
        d.update(gamma=1 + 0.1 * _randn(g, co), beta=0.1 * _randn(g, co))
        if case["res"]:
            d["xr"] = torch.relu(_randn(g, mo, co)).bfloat16()
    else:
        # dy: the gradient at the convolution's output; c: the batch norm's input, whose ReLU output is x
        d.update(dy=_randn(g, mo, co, scale=1e-3).bfloat16(), c=_randn(g, mi, ci).bfloat16(), gamma=1 + 0.1 * _randn(g, ci))
        d["st"] = _stats(d["c"])
    return d


def _prepare_layer(case, seed):
    st = dict(case=case, **_layer_inputs(case, seed))
    f32, f64, b16 = torch.float32, torch.float64, torch.bfloat16

    def buf(dtype, *shape):
        return torch.empty(*shape, dtype=dtype, device=DEV)

    if case["kind"] == "bn":
        m, c = st["c"].shape
        st.update(part=buf(f64, K.op_bnb_partial_blocks(m, c) * 2 * c), sums=buf(f32, 2 * c), dgamma=buf(f32, c),
                  dbeta=buf(f32, c), d=buf(b16, m, c))
        return st
    n, h, ho, ci, co, r, s = case["n"], case["side"], _side_out(case), case["ci"], case["co"], case["r"], case["s"]
    mi, mo = n * h * h, n * ho * ho
    st["geo"] = K.conv_geo(n, h, h, ci, ho, ho, co, r, s, r // 2)
    if case["kind"] == "conv":
        rb, _ = K.op_gemm_bf16_blocks(mo, co)
        st.update(rb=rb, stats=buf(f64, rb * 2 * co), c=buf(b16, mo, co), st=buf(f32, 2 * co), y=buf(b16, mo, co))
        return st
    rb, _ = K.op_gemm_bf16_blocks(mi, ci)
    tiles = ((co + 127) // 128) * ((r * r * ci + 127) // 128)
    splits = max(1, min(512 // tiles, mo // 256))
    st.update(rb=rb, part=buf(f64, rb * 2 * ci), sums=buf(f32, 2 * ci), ds=buf(f32, mi, ci), dgamma=buf(f32, ci),
              dbeta=buf(f32, ci), d=buf(b16, mi, ci), splits=splits, wpart=buf(f32, splits, co * r * r * ci),
              dw=buf(f32, co, r, r, ci))
    return st


def prepare(case, seed):
    if case["kind"] in ("conv", "grad", "bn"):
        return _prepare_layer(case, seed)
    return _prepare_net(case, seed)


# -------------------------------------------------------------------- runs --
def run(state):
    kind = state["case"]["kind"]
    s = torch.cuda.current_stream()
    if kind == "bn":
        m, c = state["c"].shape
        K.op_bnb_backward(m, c, state["g"], state["ym"], state["c"], state["st"], state["gamma"], state["part"],
                          state["sums"], state["dgamma"], state["dbeta"], state["d"], stream=s)
        return [state["d"], state["dgamma"], state["dbeta"]]
    if kind == "conv":
        return _run_conv(state, s)
    if kind == "grad":
        return _run_grad(state, s)
    K.train_step(state["net"], state["params"], state["grads"], state["x"], state["t"], state["plan"], state["ws"],
                 state["need"], stream=s, loss_dev=state["loss"], want_loss=False)
    return [state["loss"]] + state["views"]


def _run_conv(state, s):
    """Convolution with the batch norm's sums, its statistics, then relu(bn(c) [+ shortcut])."""
    case = state["case"]
    mo, co = state["c"].shape
    if case["r"] == 1 and case["s"] == 1:
        ci = case["ci"]
        K.op_gemm_bf16(mo, co, ci, state["x"], ci, True, state["w"], ci, True, None, co, K.EPI_BF16STATS,
                       cb=state["c"], stats=state["stats"], stream=s)
    else:
        K.op_conv_bf16_fwd(state["geo"], state["x"], state["w"], state["c"], state["stats"], stream=s)
    K.op_bn_finalize(False, state["stats"], state["rb"], co, mo, state["st"], stream=s)
    K.op_bnb_apply(K.BNB_RES_ID if case["res"] else K.BNB_RES_NONE, mo, co, state["c"], state["st"], state["gamma"],
                   state["beta"], x=state.get("xr"), y=state["y"], stream=s)
    return [state["c"], state["st"], state["y"]]


def _run_grad(state, s):
    """The convolution's data gradient, masked by the ReLU before it and with the batch norm's
    sums, that batch norm's backward, and the convolution's weight gradient."""
    case = state["case"]
    mo, co = state["dy"].shape
    mi, ci = state["x"].shape
    one = case["r"] == 1 and case["s"] == 1
    if one:
        K.op_gemm_bf16(mi, ci, co, state["dy"], co, True, state["w"], ci, False, state["ds"], ci, K.EPI_BNBWD,
                       mask=state["x"], cv=state["c"], bst=state["st"], stats=state["part"], stream=s)
    else:
        K.op_conv_bf16_dgrad(state["geo"], state["dy"], state["w"], state["ds"], K.EPI_BNBWD, mask=state["x"],
                             cv=state["c"], bst=state["st"], stats=state["part"], stream=s)
    K.op_bn_finalize(True, state["part"], state["rb"], ci, mi, state["sums"], state["dgamma"], state["dbeta"], stream=s)
    K.op_bnb_backward_apply(mi, ci, state["ds"], None, state["c"], state["st"], state["gamma"], state["sums"],
                            state["d"], stream=s)
    if not one:
        K.op_conv_bf16_wgrad(state["geo"], state["x"], state["dy"], state["wpart"], state["splits"], state["dw"],
                             stream=s)
    elif state["splits"] == 1:
        K.op_gemm_bf16(co, ci, mo, state["dy"], co, False, state["x"], ci, False, state["dw"], ci, K.EPI_STORE, stream=s)
    else:
        K.op_gemm_bf16(co, ci, mo, state["dy"], co, False, state["x"], ci, False, state["wpart"], ci, K.EPI_STORE,
                       splits=state["splits"], stream=s)
        K.op_sum_partials(state["wpart"], state["splits"], co * ci, state["dw"], stream=s)
    return [state["ds"], state["dgamma"], state["dbeta"], state["d"], state["dw"]]


# -------------------------------------------------------------------- work --
def work(case):
    """Operations and bytes of one pass: each layer's forward as often as the plan
    runs it and its backward once; bytes are the inputs read once and the outputs
    written once."""
    kind = case["kind"]
    if kind == "bn":
        e = case["n"] * case["side"] ** 2 * case["c"]
        return dict(bytes=10 * e, flops=10 * e)
    if kind in ("conv", "grad"):
        mi, mo = case["n"] * case["side"] ** 2, case["n"] * _side_out(case) ** 2
        ci, co, k = case["ci"], case["co"], case["r"] ** 2 * case["ci"]
        if kind == "conv":
            return dict(bytes=2 * (mi * ci + k * co + (2 + case["res"]) * mo * co), flops=2 * mo * k * co)
        # dy, x, c, w; ds (float32), d, dw (float32)
        return dict(bytes=2 * (mo * co + 2 * mi * ci + k * co) + 6 * mi * ci + 4 * k * co, flops=4 * mo * k * co)
    if kind == "mlp":
        n = case["depth"]
        wts, bt = n * case["width"] ** 2, case["batch"] * case["width"] * 8
        unit = 2 * case["batch"] * case["width"] ** 2
        fwd, params = unit * n, 4 * wts
    elif kind == "lstm":
        n = case["T"]
        B, E, H, V = (case[k] for k in ("batch", "input", "hidden", "vocab"))
        params, bt = 4 * ((E + H) * 4 * H + H * V), n * B * (2 * E + 4)
        fwd, head = 2 * n * B * (E + H) * 4 * H, 2 * n * B * H * V
        # backward: all products twice, but for the inputs' own gradient
        return dict(bytes=2 * params + bt,
                    flops=fwd * (1 + _extra(case, n) / n) + head + fwd + 2 * n * B * 4 * H * H + 2 * head)
    elif kind == "cifar":
        n, side = 1 + 3 * case["blocks"], case["image"]
        fwd, params = 2 * side * side * 27 * case["base"], 4 * 27 * case["base"]
        for _, ci, co, s in _cifar_blocks(case):
            side //= s
            fwd += 2 * side * side * 9 * co * (ci + co)
            params += 36 * co * (ci + co)
        fwd *= case["batch"]
        bt = case["batch"] * case["image"] ** 2 * 12
    else:
        side = (case["image"] + 1) // 2
        n, fwd, params = 1 + sum(_stages(case)), 2 * side * side * 147 * 64, 4 * 147 * 64
        side = (side + 1) // 2
        for _, ci, w, s, proj in _resnet_blocks(case):
            fwd += 2 * side * side * ci * w
            side //= s
            fwd += 2 * side * side * (9 * w * w + 4 * w * w + (4 * w * ci if proj else 0))
            params += 4 * (ci * w + 13 * w * w + (4 * w * ci if proj else 0))
        fwd *= case["batch"]
        bt = case["batch"] * case["image"] ** 2 * 6
    return dict(bytes=2 * params + bt, flops=int(fwd * (3 + _extra(case, n) / n)))


def _extra(case, n):
    """Unit forwards beyond the first pass."""
    if case["plan"] == "none":
        return 0
    if case["plan"] != "recursive":
        return n
    k = case["arg"]

    def rec(m):
        if m == 1:
            return 1
        cut = sorted({j * m // (k + 1) for j in range(1, k + 1)} - {0, m})
        parts = [b - a for a, b in zip([0] + cut, cut + [m])]
        return cut[-1] + sum(rec(q) for q in parts)

    top = sorted({j * n // (k + 1) for j in range(1, k + 1)} - {0, n})
    return sum(rec(b - a) for a, b in zip([0] + top, top + [n]))


# --------------------------------------------------------------- tolerance --
def tolerance(case):
    """Four times the largest difference seen between this path, the same sums in another
    order (torch's in float32; for bfloat16 the path with its parameters moved by 1e-7,
    which turns the same roundings) and float64."""
    kind = case["kind"]
    if kind == "mlp":
        # without a changed ReLU decision 2.4e-7; one such decision moves a weight gradient by
        # 0.2 / sqrt(batch width) (1.7e-3 at 64 x 256, 3.4e-4 at 256 x 1024), about one in 2e7 is
        e = case["batch"] * case["width"]
        return {"rel": 0.8 / math.sqrt(e) if e * case["depth"] > 1e5 else 1e-6}
    if kind == "cifar":
        # 1.5e-2 (110 layers) and 1.2e-2 (20 layers) where ReLU decisions change, else 7e-6
        e = case["batch"] * case["image"] ** 2 * case["base"] * case["blocks"]
        return {"rel": 6e-2 if e > 2e4 else 3e-5}
    if kind == "resnet":
        # gradients under a batch norm of bfloat16 values: 0.01, 0.06, 0.15, 0.19 with 1 to 4 blocks
        return {"rel": {1: 0.04, 2: 0.25, 3: 0.6}.get(sum(_stages(case)), 0.75)}
    # bfloat16 operands or results: 3e-3 (LSTM), 2.6e-3 (layer forward), 1.7e-3 (layer backward)
    return {"rel": {"lstm": 1e-2, "conv": 1e-2, "grad": 7e-3, "bn": 7e-3}[kind]}


# ------------------------------------------------------------------- exact --
def _conv64(x, w, s):
    """NHWC convolution with [co, r, r, ci] weights and padding r // 2, as one product per tap."""
    r = w.shape[1]
    p = r // 2
    ho = (x.shape[1] + 2 * p - r) // s + 1
    xp = torch.nn.functional.pad(x, (0, 0, p, p, p, p))
    y = 0
    for a in range(r):
        for b in range(r):
            y = y + xp[:, a:a + s * (ho - 1) + 1:s, b:b + s * (ho - 1) + 1:s] @ w[:, a, b].t()
    return y


def _bn64(c, gamma, beta):
    d = tuple(range(c.dim() - 1))
    m = c.mean(d)
    return gamma * (c - m) * ((c - m) ** 2).mean(d).add(EPS).rsqrt() + beta


def _loss64(case, x, t, p):
    relu = torch.relu
    kind = case["kind"]
    if kind == "mlp":
        for i in range(case["depth"]):
            x = x + relu(x @ p["u%d.W" % i] + p["u%d.b" % i])
        return ((x - t) ** 2).mean()
    if kind == "lstm":
        h = c = torch.zeros(case["batch"], case["hidden"], dtype=x.dtype, device=x.device)
        hs = []
        for xt in x:
            i, f, g, o = (xt @ p["W_x"] + h @ p["W_h"] + p["b"]).chunk(4, 1)
            c = torch.sigmoid(f) * c + torch.sigmoid(i) * torch.tanh(g)
            h = torch.sigmoid(o) * torch.tanh(c)
            hs.append(h)
        logits = torch.cat(hs) @ p["W_o"] + p["b_o"]
        return torch.nn.functional.cross_entropy(logits, t.reshape(-1).long())
    if kind == "cifar":
        x = relu(_bn64(_conv64(x, p["u0.W"], 1), p["u0.gamma"], p["u0.beta"]))
        for u, ci, co, s in _cifar_blocks(case):
            r = relu(_bn64(_conv64(x, p[u + "W1"], s), p[u + "gamma1"], p[u + "beta1"]))
            y = _bn64(_conv64(r, p[u + "W2"], 1), p[u + "gamma2"], p[u + "beta2"])
            x = relu(y + torch.nn.functional.pad(x[:, ::s, ::s], (0, co - ci)))
    else:
        x = relu(_bn64(_conv64(x, p["u0.W"], 2), p["u0.gamma"], p["u0.beta"]))
        x = torch.nn.functional.max_pool2d(x.permute(0, 3, 1, 2), 3, 2, 1).permute(0, 2, 3, 1)
        for u, ci, w, s, proj in _resnet_blocks(case):
            r = x
            for k, st in ((1, 1), (2, s), (3, 1)):
                r = _bn64(_conv64(r, p[u + "W%d" % k], st), p[u + "gamma%d" % k], p[u + "beta%d" % k])
                r = relu(r) if k < 3 else r
            if proj:
                x = _bn64(_conv64(x, p[u + "Wp"], s), p[u + "gammap"], p[u + "betap"])
            x = relu(r + x)
    logits = x.mean((1, 2)) @ p["head.W"] + p["head.b"]
    return torch.nn.functional.cross_entropy(logits, t.long())


def exact(case, seed):
    kind = case["kind"]
    if kind in ("conv", "grad", "bn"):
        d = {k: v.double() for k, v in _layer_inputs(case, seed).items()}
        return _exact_bn(d) if kind == "bn" else _exact_conv(case, d) if kind == "conv" else _exact_grad(case, d)
    x, t, p = _net_inputs(case, seed)
    p = {k: v.double().requires_grad_() for k, v in p.items()}
    loss = _loss64(case, x.double(), t.double() if kind == "mlp" else t, p)
    if kind == "resnet":
        # the gradients that bfloat16 roundings leave are a third off those without any: the layers
        # have exact values, the network's loss too, its gradients none that would compare
        return [loss.detach().reshape(1)] + [None] * len(_parts(list(range(len(p)))))
    flat, offs = [], [0]
    for v in torch.autograd.grad(loss, list(p.values())):
        flat.append(torch.nn.functional.pad(v.reshape(-1), (0, -v.numel() % 64)))  # each parameter on 256 bytes
        offs.append(offs[-1] + flat[-1].numel())
    flat = torch.cat(flat)
    starts = _parts(offs[:-1])
    return [loss.detach().reshape(1)] + [flat[a:b] for a, b in zip(starts, starts[1:] + [flat.numel()])]


def _bn_backward64(ds, c, st, gamma):
    j = c.shape[1]
    xh = (c - st[:j]) * st[j:]
    return gamma * st[j:] * (ds - ds.mean(0) - xh * (ds * xh).mean(0)), (ds * xh).sum(0), ds.sum(0)


def _exact_bn(d):
    return list(_bn_backward64(d["g"] * (d["ym"] > 0), d["c"], d["st"], d["gamma"]))


def _exact_conv(case, d):
    n, h, co = case["n"], case["side"], case["co"]
    c = _conv64(d["x"].reshape(n, h, h, -1), d["w"], case["s"]).reshape(-1, co)
    m = c.mean(0)
    rstd = ((c - m) ** 2).mean(0).add(EPS).rsqrt()
    y = d["gamma"] * (c - m) * rstd + d["beta"]
    return [c, torch.cat([m, rstd]), torch.relu(y + d["xr"] if case["res"] else y)]


def _exact_grad(case, d):
    n, h, ho, co = case["n"], case["side"], _side_out(case), case["co"]
    x = d["x"].reshape(n, h, h, -1).requires_grad_()
    w = d["w"].requires_grad_()
    y = _conv64(x, w, case["s"])
    dx, dw = torch.autograd.grad(y, (x, w), d["dy"].reshape(n, ho, ho, co))
    ds = dx.reshape(d["c"].shape) * (d["x"] > 0)
    dd, dgamma, dbeta = _bn_backward64(ds, d["c"], d["st"], d["gamma"])
    return [ds, dgamma, dbeta, dd, dw]
