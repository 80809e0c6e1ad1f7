"""The work that a program has this library do, as cases that can be measured: what it reads and
writes, how to make its inputs, one pass through the public entry points, and the same in 64 bits.

Sizes are those of the deployed workloads: the linears of a Llama-2-7B decoder layer (the backbone
of the manipulation policy, one launch or several), the ResNet-34 body of the driving policy, and
the operators of training through the quantisers; `draw` gives others of the same ranges.
"""
from __future__ import annotations

import math

import torch
import torch.nn.functional as F

from paper_2412_01034_amd import binding as B

# One decoder layer: fused q/k/v, attention output, fused gate/up, down.
LAYER = "12288x4096+4096x4096+22016x4096+4096x11008"
STAGES = ((64, 3), (128, 4), (256, 6), (512, 3))   # ResNet-34: width and residual blocks per stage
MOST_MACS = 1024 * 202_375_168                      # the largest listed case: the layer at M = 1024
MOST_PIXELS = 32 * 224 * 224


def listed():
    def linear(name, M, linears=LAYER, bits=4, group=128, rank=0):
        return dict(name=name, kind="linear", bits=bits, M=M, linears=linears, group=group, rank=rank)

    return [
        # the smallest call: one linear of a decode step launched alone, as a decoder whose linears
        # wait for each other has to
        linear("linear_m1", 1, "4096x4096"),
        # a decode step of one sequence, the four linears of a layer in one call
        linear("layer_m1", 1),
        # ... with the unmerged rank-32 adapters of a fine-tuned policy
        linear("layer_m1_rank32", 1, rank=32),
        # a decode step of a few environments at once, a ragged number of them
        linear("layer_m7", 7),
        # ... of many
        linear("layer_m48", 48),
        # prefill of one prompt: image patches and instruction, about 288 tokens
        linear("layer_m288", 288),
        # prefill of several prompts or a long one
        linear("layer_m1024", 1024),
        # prefill with the 8-bit backbone
        linear("layer_w8_m288", 288, bits=8),
        # the driving policy looks at one frame: 35 convolutions, 4-bit from end to end
        dict(name="encoder_b1", kind="encoder", batch=1, image=224),
        # ... at the batch its throughput is quoted for
        dict(name="encoder_b32", kind="encoder", batch=32, image=224),
        # one 8-bit layer that gets real-valued activations: find the step, quantise, convolve
        dict(name="conv_w8a8", kind="conv", bits=8, batch=32, height=28, width=28, cin=128, cout=128, taps=3, stride=1),
        # training through the quantisers: weights, activations forward and backward, the policy loss
        dict(name="train_ops", kind="train", rows=4096, cols=4096, group=128, acts=32 * 56 * 56 * 64, batch=256, vocab=32000),
    ]


def _log(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_linear(rng):
    bits = rng.choice((4, 4, 4, 8))
    rank = rng.choice((0, 0, 0, 8, 16, 32, 64)) if bits == 4 else 0
    group = 128 if bits == 8 else rng.choice((64, 128, 128, 128))
    M = _log(rng, 1, 4) if rank else _log(rng, 1, 2048)
    if rng.random() < 0.6:   # a decoder layer of some width; its MLP is about 2.7 times as wide
        h = 256 * rng.randint(4, 20)
        f = 256 * int(round(2.6875 * h / 256))
        linears = "%dx%d+%dx%d+%dx%d+%dx%d" % (3 * h, h, h, h, 2 * f, h, h, f)
    else:                    # one linear, with any number of rows
        linears = "%dx%d" % (_log(rng, 500, 24000), group * 2 * rng.randint(4, 43))
    macs = sum(n * k for n, k in _shapes(linears))
    most = MOST_MACS * 4 // (bits * macs)   # a byte of weight is twice the work of a nibble
    return dict(kind="linear", bits=bits, M=max(1, min(M, most)), linears=linears, group=group, rank=rank)


def draw(rng):
    kind = rng.choice(("linear", "linear", "linear", "linear", "encoder", "conv", "train"))
    if kind == "linear":
        return _draw_linear(rng)
    if kind == "encoder":
        image = 32 * rng.randint(4, 8)
        return dict(kind="encoder", batch=_log(rng, 1, MOST_PIXELS // image ** 2), image=image)
    if kind == "conv":
        cin = 32 * _log(rng, 2, 16)
        size = max(7, 3584 // cin + rng.randint(-6, 6))
        return dict(kind="conv", bits=rng.choice((4, 8)), batch=_log(rng, 1, 32), height=size, width=size + rng.randint(-3, 3),
                    cin=cin, cout=rng.choice((cin, 2 * cin, 4 * _log(rng, 10, 128))), taps=rng.choice((1, 3, 3)), stride=rng.choice((1, 1, 2)))
    group = rng.choice((64, 128))
    return dict(kind="train", rows=_log(rng, 256, 12288), cols=group * rng.randint(8, 32), group=group,
                acts=_log(rng, 30_000, 6_400_000), batch=_log(rng, 8, 512), vocab=_log(rng, 1000, 32000))


# ------------------------------------------------------------------------------------- inputs --

def _rng(seed, stream):
    return torch.Generator(device="cuda").manual_seed(1009 * int(seed) + stream)


def _normal(shape, seed, stream, std=1.0):
    return torch.randn(shape, generator=_rng(seed, stream), device="cuda") * std


def _outliers(t, seed, stream, share, gain):
    """A share of the columns is `gain` times as large: salient channels."""
    cols = torch.randperm(t.shape[1], generator=_rng(seed, stream), device="cuda")[: math.ceil(share * t.shape[1])]
    t[:, cols] *= gain
    return t


def _shapes(linears):
    return [tuple(int(v) for v in s.split("x")) for s in linears.split("+")]


def _linear_inputs(case, seed):
    """fp32 weights, bf16 activations and adapter factors of each linear, one linear at a time."""
    for i, (N, K) in enumerate(_shapes(case["linears"])):
        w = _outliers(_normal((N, K), seed, 10 * i, 0.02), seed, 10 * i + 1, 0.01, 20.0)
        x = _outliers(_normal((case["M"], K), seed, 10 * i + 2), seed, 10 * i + 3, 0.005, 10.0).to(torch.bfloat16)
        r = case["rank"]
        ab = (_normal((r, K), seed, 10 * i + 4, 0.02).to(torch.bfloat16), _normal((N, r), seed, 10 * i + 5, 0.02).to(torch.bfloat16)) if r else None
        yield N, K, w, x, ab


def _quantised(w, group, scheme):
    N, K = w.shape[0], w.numel() // w.shape[0]
    q, s, z = B.qail_packed_sizes(N, K, group, scheme)
    qweight = torch.empty(q // 4, dtype=torch.int32, device="cuda")
    scales = torch.empty(s // 2, dtype=torch.float16, device="cuda") if scheme in (B.QAIL_W4_ASYM_GROUP, B.QAIL_W8_SYM_GROUP) \
        else torch.empty(s // 4, dtype=torch.float32, device="cuda")
    zeros = torch.empty(z // 4, dtype=torch.int32, device="cuda") if z else None
    B.qail_quantize_weights(w, group, scheme, qweight, scales, zeros)
    return qweight, scales, zeros


def _workspace(nbytes):
    return torch.empty(nbytes, dtype=torch.uint8, device="cuda") if nbytes else None


def _prepare_linear(case, seed):
    four = case["bits"] == 4
    entries, loras = [], []
    for N, K, w, x, ab in _linear_inputs(case, seed):
        q, s, z = _quantised(w, case["group"], B.QAIL_W4_ASYM_GROUP if four else B.QAIL_W8_SYM_GROUP)
        entries.append(dict(N=N, K=K, group_size=case["group"], qweight=q, scales=s, zeros=z, x=x,
                            y=torch.empty((case["M"], N), dtype=torch.bfloat16, device="cuda")))
        if ab:
            loras.append(dict(A=ab[0], B=ab[1], r=case["rank"], N=N, K=K, scaling=2.0))
    M, n = case["M"], len(entries)
    st = dict(case=case, entries=entries, loras=loras, M=M, n=n)
    if four:
        st["items"] = B.make_w4a16_items(entries, M)
        if loras:
            st["adapters"] = B.make_loras(loras)
            st["ws"] = _workspace(B.qail_w4a16_lora_workspace(st["items"], st["adapters"], n, M))
        elif n == 1:
            st["ws"] = _workspace(B.qail_w4a16_workspace(entries[0]["N"], entries[0]["K"], case["group"], M))
        else:
            st["ws"] = _workspace(B.qail_w4a16_batch_workspace(st["items"], n, M))
    else:
        st["items"] = B.make_w8a16_items(entries, M)
        st["ws"] = _workspace(B.qail_w8a16_batch_workspace(st["items"], n, M))
    return st


def _run_linear(st):
    M, n, ws = st["M"], st["n"], st["ws"]
    if st["case"]["bits"] == 8:
        B.qail_w8a16_linear_batch(st["items"], n, M, ws)
    elif st["loras"]:
        B.qail_w4a16_linear_lora_batch(st["items"], st["adapters"], n, M, ws)
    elif n == 1:
        e = st["entries"][0]
        B.qail_w4a16_linear(e["N"], e["K"], e["group_size"], e["qweight"], e["scales"], e["zeros"], e["x"], e["y"], M, ws)
    else:
        B.qail_w4a16_linear_batch(st["items"], n, M, ws)
    return [e["y"] for e in st["entries"]]


def _body(case):
    """The convolutions of the encoder in order: (role, H, W, Cin, Cout, taps, stride, block)."""
    h, cin, out, block = case["image"] // 4, 64, [], 0
    for si, (c, blocks) in enumerate(STAGES):
        for bi in range(blocks):
            stride = 2 if si and not bi else 1
            out.append(("first", h, h, cin, c, 3, stride, block))
            if stride == 2:
                out.append(("project", h, h, cin, c, 1, 2, block))
            h = (h - 1) // stride + 1
            out.append(("second", h, h, c, c, 3, 1, block))
            cin, block = c, block + 1
    return out


def _steps(case):
    """Learned activation steps per block: (of its input, of its middle, of its output).  Each block's
    second convolution is scaled down, as trained residual branches are, so that codes fill the range."""
    steps, power = [], 0.5
    for _ in range(sum(n for _, n in STAGES)):
        mid, after = power, 1.15 * power
        steps.append(tuple(4.0 * math.sqrt(2.0 * p) / 15.0 for p in (power, mid, after)))
        power = after
    return steps


def _encoder_inputs(case, seed):
    """4-bit input codes [B, H, W, 64] (values 0..15) and, per convolution, fp32 weights and biases."""
    h = case["image"] // 4
    step = _steps(case)[0][0]
    a = torch.relu(_normal((case["batch"], h, h, 64), seed, 1))
    codes = torch.clamp(torch.round(a / step), max=15.0).to(torch.int32)
    layers = []
    for i, (role, H, W, cin, cout, taps, stride, block) in enumerate(_body(case)):
        std = math.sqrt(2.0 / (taps * taps * cin)) * (0.3 if role == "second" else 1.0)
        layers.append((_normal((cout, taps, taps, cin), seed, 10 + 2 * i, std), _normal((cout,), seed, 11 + 2 * i, 0.1)))
    return codes, layers


def _pack(codes):
    shift = torch.arange(0, 32, 4, device=codes.device, dtype=torch.int64)
    words = (codes.reshape(-1, 8).to(torch.int64) << shift).sum(1)
    return torch.where(words >= 1 << 31, words - (1 << 32), words).to(torch.int32)


def _prepare_encoder(case, seed):
    codes, layers = _encoder_inputs(case, seed)
    steps, nb = _steps(case), case["batch"]
    entering = _pack(codes)
    launches, outputs, keep, shortcut, middle, first = [], [], [entering], None, None, None
    for (role, H, W, cin, cout, taps, stride, block), (w, bias) in zip(_body(case), layers):
        q, s_w, _ = _quantised(w, w.numel() // cout, B.QAIL_W4_SYM_CHANNEL)
        s_in, s_mid, s_out = steps[block]
        e = dict(B=nb, H=H, W=W, Cin=cin, Cout=cout, KH=taps, KW=taps, stride=stride, pad=taps // 2, w_s4=q, bias=bias,
                 scale=s_w * (s_mid if role == "second" else s_in))
        M = nb * ((H - 1) // stride + 1) * ((W - 1) // stride + 1)
        if role == "project":
            shortcut = torch.empty((M, cout), dtype=torch.float32, device="cuda")
            e.update(a_u4=entering, y_out=shortcut)
            outputs.append(shortcut)
            launches[-1] = [first, e]   # opens a stage together with the 3x3 of the same input
        else:
            out = torch.empty(M * cout // 8, dtype=torch.int32, device="cuda")
            outputs.append(out)
            if role == "first":
                e.update(a_u4=entering, out_u4=out, s_out=s_mid)
                middle, first = out, e
            elif shortcut is not None:
                e.update(a_u4=middle, out_u4=out, s_out=s_out, res_f32=shortcut)
                entering, shortcut = out, None
            else:
                e.update(a_u4=middle, out_u4=out, s_out=s_out, res_u4=entering, res_scale=s_in)
                entering = out
            launches.append([e])
        keep.append(e)
    return dict(case=case, outputs=outputs, keep=keep, launches=[(B.make_conv_items(l), len(l)) for l in launches])


def _run_encoder(st):
    for items, count in st["launches"]:
        B.qail_w4a4_conv_batch(items, count)
    return st["outputs"]


def _conv_shape(case):
    p = case["taps"] // 2
    return tuple((case[k] + 2 * p - case["taps"]) // case["stride"] + 1 for k in ("height", "width"))


def _conv_inputs(case, seed):
    cin, cout, taps = case["cin"], case["cout"], case["taps"]
    a = torch.relu(_normal((case["batch"], case["height"], case["width"], cin), seed, 1))
    w = _normal((cout, taps, taps, cin), seed, 2, math.sqrt(2.0 / (taps * taps * cin)))
    return a, w, _normal((cout,), seed, 3, 0.1)


def _prepare_conv(case, seed):
    a, w, bias = _conv_inputs(case, seed)
    eight = case["bits"] == 8
    q, s_w, _ = _quantised(w, w.numel() // case["cout"], B.QAIL_W8_SYM_CHANNEL if eight else B.QAIL_W4_SYM_CHANNEL)
    oh, ow = _conv_shape(case)
    return dict(case=case, a=a, q=q, scale=s_w, bias=bias, step=torch.empty(1, device="cuda"),
                codes=torch.empty(a.numel() * case["bits"] // 32, dtype=torch.int32, device="cuda"),
                y=torch.empty((case["batch"] * oh * ow, case["cout"]), device="cuda"),
                geom=(case["batch"], case["height"], case["width"], case["cin"], case["cout"], case["taps"], case["taps"],
                      case["stride"], case["taps"] // 2))


def _run_conv(st):
    if st["case"]["bits"] == 8:
        B.qail_act_scale_s8(st["a"], st["step"])
        B.qail_quantize_act_s8(st["a"], st["step"], st["codes"])
        B.qail_w8a8_gemm(*st["geom"], st["codes"], st["q"], scale=st["scale"], bias=st["bias"], y_out=st["y"])
    else:
        B.qail_act_scale_u4(st["a"], st["step"])
        B.qail_quantize_act_u4(st["a"], st["step"], st["codes"])
        B.qail_w4a4_gemm(*st["geom"], st["codes"], st["q"], scale=st["scale"], bias=st["bias"], y_out=st["y"])
    return [st["step"], st["codes"], st["y"]]


def _train_inputs(case, seed):
    w = _outliers(_normal((case["rows"], case["cols"]), seed, 1, 0.02), seed, 2, 0.01, 20.0)
    v = torch.relu(_normal((case["acts"],), seed, 3))
    dout = _normal((case["acts"],), seed, 4, 1e-3) + 5e-4 * v   # pulls large activations in: the step's gradient is no sum of noise alone
    lq = _normal((case["batch"], case["vocab"]), seed, 5, 2.0)
    return w, v, dout, lq, lq + _normal((case["batch"], case["vocab"]), seed, 6, 0.3)


def _prepare_train(case, seed):
    w, v, dout, lq, lf = _train_inputs(case, seed)
    one = torch.empty(1, device="cuda")
    return dict(case=case, w=w, v=v, dout=dout, lq=lq, lf=lf, s=torch.full((1,), 0.2, device="cuda"), w_hat=torch.empty_like(w),
                v_hat=torch.empty_like(v), dv=torch.empty_like(v), ds=one, loss=torch.empty_like(one), grad=torch.empty_like(lq),
                ws_lsq=_workspace(B.qail_lsq_backward_workspace()), ws_qbc=_workspace(4 * case["batch"]))


def _grad_scale(case):
    return 1.0 / math.sqrt(15.0 * case["acts"])


def _run_train(st):
    B.qail_fake_quant_w4(st["w"], st["case"]["group"], st["w_hat"])
    B.qail_lsq_forward(st["v"], st["s"], 0, 15, st["v_hat"])
    B.qail_qbc_loss(st["lq"], st["lf"], st["loss"], st["grad"], st["ws_qbc"])
    B.qail_lsq_backward(st["v"], st["dout"], st["s"], 0, 15, _grad_scale(st["case"]), st["dv"], st["ds"], st["ws_lsq"])
    return [st["w_hat"], st["v_hat"], st["loss"], st["grad"], st["dv"], st["ds"]]


def prepare(case, seed):
    return {"linear": _prepare_linear, "encoder": _prepare_encoder, "conv": _prepare_conv, "train": _prepare_train}[case["kind"]](case, seed)


def run(state):
    return {"linear": _run_linear, "encoder": _run_encoder, "conv": _run_conv, "train": _run_train}[state["case"]["kind"]](state)


# ------------------------------------------------------------------------------- what it costs --

def work(case):
    kind, nbytes, flops = case["kind"], 0, 0
    if kind == "linear":
        M, g, r = case["M"], case["group"], case["rank"]
        for N, K in _shapes(case["linears"]):
            nbytes += N * K * case["bits"] // 8 + N * (K // g) * 2 + (N * ((K // g + 7) // 8) * 4 if case["bits"] == 4 else 0)
            nbytes += 2 * M * (N + K) + 2 * r * (N + K)
            flops += 2 * M * N * K + 2 * M * r * (N + K)
    elif kind == "encoder":   # a body: each layer's codes in and out, its weights, its shortcut
        for role, H, W, cin, cout, taps, stride, _ in _body(case):
            M = case["batch"] * ((H - 1) // stride + 1) * ((W - 1) // stride + 1)
            pixels = M if taps == 1 else case["batch"] * H * W
            nbytes += pixels * cin // 2 + cout * taps * taps * cin // 2 + M * cout * (4 if role == "project" else 0.5)
            if role == "second":
                nbytes += M * cout // 2
            flops += 2 * M * cout * taps * taps * cin
    elif kind == "conv":
        oh, ow = _conv_shape(case)
        n, K = case["batch"] * case["height"] * case["width"] * case["cin"], case["taps"] ** 2 * case["cin"]
        nbytes = 4 * n + n * case["bits"] // 8 + case["cout"] * K * case["bits"] // 8 + 4 * case["batch"] * oh * ow * case["cout"]
        flops = 2 * case["batch"] * oh * ow * case["cout"] * K
    else:
        nbytes = 8 * case["rows"] * case["cols"] + 16 * case["acts"] + 12 * case["batch"] * case["vocab"]
        flops = 10 * case["rows"] * case["cols"] + 20 * case["acts"] + 6 * case["batch"] * case["vocab"]
    return dict(bytes=int(nbytes), flops=int(flops))


def tolerance(case):
    if case["kind"] == "linear":
        # measured against `exact`: rel 1.7e-3, max 4.6e-3 (one rounding to bf16); with adapters on several
        # rows, where the sum is rounded again, 2.4e-3 and 7.8e-3
        return dict(rel=1e-2, max=3e-2) if case["rank"] and case["M"] > 1 else dict(rel=7e-3, max=2e-2)
    if case["kind"] == "train":
        # elementwise results are fixed by the formats; the sums are of 32-bit numbers
        return dict(rel=1e-5)
    return "exact"   # integer sums, single roundings


# ----------------------------------------------------------------------------------- in 64 bits --

def _div(a, b):
    """a / b as one rounding to fp32 (a 53-bit quotient rounds to 24 bits like the exact one)."""
    return (a.double() / b.double()).float()


def _dequantised4(w, group):
    """(q - z) s in fp64 of the 4-bit format: fp16 scale rounded up, integer zero-point."""
    v = w.reshape(-1, group)
    lo, hi = v.amin(1).clamp(max=0.0), v.amax(1).clamp(min=0.0)
    fifteen = torch.tensor(15.0, device=w.device)
    s = _div(hi - lo, fifteen)
    h = s.half()
    up = (h.view(torch.int16) + 1).view(torch.float16)
    s = torch.where(h.float() < s, up, h).float().clamp(min=2.0 ** -14)
    s = torch.where(hi == lo, torch.ones_like(s), s)
    z = torch.clamp(torch.round(_div(-lo, s)), 0, 15)
    q = torch.clamp(torch.round(_div(v, s[:, None])) + z[:, None], 0, 15)
    return ((q - z[:, None]).double() * s[:, None].double()).reshape(w.shape)


def _dequantised8(w, group):
    v = w.reshape(-1, group)
    top = v.abs().amax(1)
    s = _div(top, torch.tensor(127.0, device=w.device))
    h = s.half()
    up = (h.view(torch.int16) + 1).view(torch.float16)
    s = torch.where(h.float() < s, up, h).float().clamp(min=2.0 ** -14)
    s = torch.where(top == 0, torch.ones_like(s), s)
    q = torch.clamp(torch.round(_div(v, s[:, None])), -127, 127)
    return (q.double() * s[:, None].double()).reshape(w.shape)


def _exact_linear(case, seed):
    out = []
    for N, K, w, x, ab in _linear_inputs(case, seed):
        w_hat = (_dequantised4 if case["bits"] == 4 else _dequantised8)(w, case["group"])
        y = x.double() @ w_hat.t()
        if ab:
            y += 2.0 * ((x.double() @ ab[0].double().t()) @ ab[1].double().t())
        out.append(y)
    return out


def _channel_codes(w, top, lo):
    """Symmetric codes per output channel and their fp32 steps."""
    v = w.reshape(w.shape[0], -1)
    s = _div(v.abs().amax(1), torch.tensor(float(top), device=w.device))
    s = torch.where(s == 0, torch.ones_like(s), s)
    return torch.clamp(torch.round(_div(v, s[:, None])), lo, top).reshape(w.shape).double(), s


def _conv64(a, w, stride):
    """NHWC codes times [Cout, k, k, Cin] codes -> [M, Cout], exact in fp64."""
    nb, k = a.shape[0], w.shape[1]
    out = []
    for i in range(nb):
        cols = F.unfold(a[i:i + 1].permute(0, 3, 1, 2).contiguous(), k, padding=k // 2, stride=stride)[0]
        out.append(cols.t().contiguous() @ w.permute(0, 3, 1, 2).reshape(w.shape[0], -1).t().contiguous())
    return torch.cat(out)


def _exact_encoder(case, seed):
    if case["batch"] > 4:
        return None   # the same layers; an image at a time takes too long for more
    codes, layers = _encoder_inputs(case, seed)
    entering, middle, shortcut, steps, out = codes.double(), None, None, _steps(case), []
    for (role, H, W, cin, cout, taps, stride, block), (w, bias) in zip(_body(case), layers):
        q, s_w = _channel_codes(w, 7, -8)
        s_in, s_mid, s_out = (torch.tensor(s, dtype=torch.float32, device="cuda") for s in steps[block])
        scale = s_w * (steps[block][1] if role == "second" else steps[block][0])
        acc = _conv64(middle if role == "second" else entering, q, stride)
        if role == "project":
            shortcut = acc * scale.double() + bias.double()
            out.append(shortcut)
            continue
        t = acc.float() * scale + bias
        if role == "second":
            t = t + (shortcut.float() if shortcut is not None else entering.reshape(-1, cout).float() * s_in)
            shortcut = None
        c = torch.clamp(torch.round(_div(torch.relu(t), s_out if role == "second" else s_mid)), max=15.0)
        out.append(_pack(c.to(torch.int32)))
        grid = c.double().reshape(case["batch"], (H - 1) // stride + 1, (W - 1) // stride + 1, cout)
        if role == "second":
            entering = grid
        else:
            middle = grid
    return out


def _exact_conv(case, seed):
    a, w, bias = _conv_inputs(case, seed)
    top, lo = (127, -127) if case["bits"] == 8 else (7, -8)
    q, s_w = _channel_codes(w, top, lo)
    a_top = 127.0 if case["bits"] == 8 else 15.0
    step = _div(a.max(), torch.tensor(a_top, device="cuda"))
    codes = torch.clamp(torch.round(_div(a, step)), max=a_top)
    y = _conv64(codes.double(), q, case["stride"]) * s_w.double() + bias.double()
    return [step.reshape(1), None, y]


def _exact_train(case, seed):
    w, v, dout, lq, lf = _train_inputs(case, seed)
    s = torch.full((1,), 0.2, device="cuda")
    u = _div(v, s)
    code = torch.clamp(torch.round(u), 0, 15)
    inside = u <= 15
    t = torch.where(inside, code.double() - u.double(), torch.full_like(u, 15.0).double())
    diff = lq.double() - lf.double()
    dist = diff.norm(dim=1)
    return [_dequantised4(w, case["group"]), code.double() * s.double(), dist.mean().reshape(1), diff / dist[:, None] / case["batch"],
            torch.where(inside, dout, torch.zeros_like(dout)).double(), (_grad_scale(case) * (dout.double() * t).sum()).reshape(1)]


def exact(case, seed):
    return {"linear": _exact_linear, "encoder": _exact_encoder, "conv": _exact_conv, "train": _exact_train}[case["kind"]](case, seed)
