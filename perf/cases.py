"""Workloads of the quantized-linear library, as a program that runs a UNet of this family calls it.

The layer widths, token counts, prompts and value distributions are those of the repository's own benchmark and tests
(SDXL-shaped UNet: channel levels 320 / 640 / 1280, a [B, 77, 2048] text context, activations N(0, 1) with one entry
in a hundred ten times as large, weights N(0, 0.02^2)).  A case is one of these kinds:

  linear      one layer by the eager call that allocates its own output, weight-only or with 8-bit activations
  kv          the K and V projections of one cross-attention layer, token 0 of each prompt kept in fp16
  kv_stacked  the K and V projections of many layers as one stacked weight, token 0 taken from a stored vector
  block       the linears of one transformer block, one pre-marshalled call per layer
  ff          the two linears of a feed-forward block with the gated product between them
  resblock    the two 3x3 convolutions of a residual block, and (down) the stride-2 convolution behind it
  prepare     quantising and packing the weights of one transformer block, as when a model is loaded
"""
import math

import torch

import paper_2405_17873_amd as mq

T = 77         # text tokens per prompt
CTX = 2048     # width of the text context


def listed():
    return [
        # a residual block's time-embedding projection: a handful of rows, all latency
        dict(name="time_embedding_w8a16", kind="linear", M=4, K=1280, N=1280, bits=8, sym=False, act="none", dtype="f16"),
        # the smallest attention linear at a small image, 8-bit activations with run-time range
        dict(name="small_linear_w8a8", kind="linear", M=256, K=320, N=320, bits=8, sym=True, act="dynamic", dtype="f16"),
        # cross-attention K and V of eight prompts
        dict(name="kv_w8a8_8_prompts", kind="kv", B=8, N=1280, bits=8, sym=True),
        # K and V of all 70 cross-attention layers for one prompt: the weights are read once from memory
        dict(name="kv_all_layers_1_prompt", kind="kv_stacked", B=1, N=166400, bits=8, sym=True),
        # one image, 640-channel level, weight-only in bfloat16 at mixed widths
        dict(name="block640_1_image_bf16", kind="block", B=1, M=4096, C=640, act="none", bits="8 4 3 4 8 4 4 3 4 8", sym=False,
             dtype="bf16"),
        # four images, 640-channel level, weight-only at an average of about 3.66 bits
        dict(name="block640_4_images_w_only", kind="block", B=4, M=16384, C=640, act="none", bits="2 3 4 2 8 4 3 8 4 3", sym=False,
             dtype="f16"),
        # four images, 1280-channel level, 4-bit weights, 8-bit activations with run-time ranges
        dict(name="block1280_4_images_w4a8", kind="block", B=4, M=4096, C=1280, act="dynamic", bits="4", sym=False, dtype="f16"),
        # three images of a format that is not square (26 x 38 positions), 8-bit weights, calibrated activation ranges
        dict(name="block1280_ragged_w8a8_static", kind="block", B=3, M=2964, C=1280, act="static", bits="8", sym=True, dtype="f16"),
        # the feed-forward pair with the activation between its linears kept in 8 bits, run-time ranges
        dict(name="ff640_4_images_w4a8", kind="ff", M=16384, C=640, path="a8_dynamic", bits=4, sym=False),
        # residual block at the 640-channel level, weight-only
        dict(name="resblock640_w4a16", kind="resblock", B=4, H=64, W=64, cin=640, cout=640, act="none", bits=4, sym=False, down=False),
        # residual block and downsampler at the 320-channel level, 8-bit activations
        dict(name="resblock320_down_w4a8", kind="resblock", B=2, H=128, W=128, cin=320, cout=320, act="dynamic", bits=4, sym=False,
             down=True),
        # a transformer block's weights on their way into the packed form
        dict(name="prepare_block1280_w4", kind="prepare", C=1280, bits=4, sym=False, dtype="f16"),
    ]


def _log(rng, lo, hi, step):
    """A multiple of `step` between lo and hi, spread over the logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return int(min(max(round(v / step) * step, -(-lo // step) * step), hi // step * step))


def _bits_a8(rng):
    b = rng.choice((8, 8, 4, 4, 2))
    return b, b == 8 and rng.random() < 0.5


def draw(rng):
    most = max(work(c)["flops"] for c in listed())
    while True:
        kind = rng.choice(("linear", "linear", "kv", "kv_stacked", "block", "block", "ff", "resblock", "prepare"))
        if kind == "linear":
            act = rng.choice(("none", "dynamic", "static"))
            bits, sym = (rng.choice((2, 3, 4, 8, 16)), False) if act == "none" else _bits_a8(rng)
            c = dict(kind=kind, M=_log(rng, 1, 8192, 1), K=_log(rng, 320, 5120, 64), N=_log(rng, 320, 10240, 8), bits=bits, sym=sym,
                     act=act, dtype=rng.choice(("f16", "f16", "bf16")) if act == "none" else "f16")
        elif kind == "kv":
            bits, sym = _bits_a8(rng)
            c = dict(kind=kind, B=rng.randint(1, 16), N=rng.choice((320, 640, 1280)), bits=bits, sym=sym)
        elif kind == "kv_stacked":
            bits, sym = _bits_a8(rng)
            c = dict(kind=kind, B=rng.randint(1, 4), N=_log(rng, 2560, 166400, 640), bits=bits, sym=sym)
        elif kind == "block":
            act = rng.choice(("none", "none", "dynamic", "static"))
            if act == "none":
                bits, sym = " ".join(str(rng.choice((2, 3, 4, 8))) for _ in range(10)), False
            else:
                b, sym = _bits_a8(rng)
                bits = str(b)
            C = rng.choice((320, 640, 640, 1280, 1280))
            c = dict(kind=kind, B=rng.randint(1, 4), M=_log(rng, 256, 16384, rng.choice((1, 64))), C=C, act=act, bits=bits, sym=sym,
                     dtype=rng.choice(("f16", "f16", "bf16")) if act == "none" else "f16")
        elif kind == "ff":
            path = rng.choice(("a8_dynamic", "a8_static", "w_only", "w_only_a8"))
            bits, sym = (rng.choice((2, 3, 4, 8)), False) if path == "w_only" else (rng.choice((4, 8, 2)), False)
            c = dict(kind=kind, M=_log(rng, 256, 16384, rng.choice((1, 64))), C=rng.choice((320, 640, 1280)), path=path, bits=bits, sym=sym)
        elif kind == "resblock":
            act = rng.choice(("none", "dynamic", "static"))
            bits, sym = (rng.choice((2, 3, 4, 8)), False) if act == "none" else _bits_a8(rng)
            cout = rng.choice((320, 640, 1280))
            side = {320: 128, 640: 64, 1280: 32}[cout]
            c = dict(kind=kind, B=rng.randint(1, 4), H=rng.randint(side // 4, side), W=rng.randint(side // 4, side),
                     cin=rng.choice((320, 640, 960, 1280, 1920)), cout=cout, act=act, bits=bits, sym=sym, down=rng.random() < 0.3)
        else:
            bits = rng.choice((2, 3, 4, 8))
            c = dict(kind=kind, C=rng.choice((320, 640, 960, 1280)), bits=bits, sym=bits == 8 and rng.random() < 0.5,
                     dtype=rng.choice(("f16", "bf16")))
        if work(c)["flops"] <= most:
            return c


# ---------------------------------------------------------------------------------------------------------- inputs

class _Make:
    """Seeded tensors on the GPU."""

    def __init__(self, seed):
        self.dev = torch.device("cuda")
        self.gen = torch.Generator(device=self.dev)
        self.gen.manual_seed(seed)

    def normal(self, *shape, std=1.0, dtype=torch.float16):
        return (torch.randn(*shape, generator=self.gen, device=self.dev) * std).to(dtype)

    def acts(self, *shape, dtype=torch.float16):
        x = torch.randn(*shape, generator=self.gen, device=self.dev)
        x[torch.rand(*shape, generator=self.gen, device=self.dev) < 0.01] *= 10.0
        return x.to(dtype)

    def context(self, B):
        """Text context whose token 0 is the same for every prompt and carries 16 channels of large magnitude."""
        x = torch.randn(B, T, CTX, generator=self.gen, device=self.dev)
        bos = torch.randn(CTX, generator=self.gen, device=self.dev)
        ch = torch.randperm(CTX, generator=self.gen, device=self.dev)[:16]
        bos[ch] = torch.randn(16, generator=self.gen, device=self.dev) * 60.0
        x[:, 0] = bos
        return x.half()

    def packed(self, w, bits, sym=False):
        if bits == 16:
            return mq.keep_weights_16bit(w)
        codes, scale, zp = mq.quantize_weights(w, bits, sym)
        data, colsum = mq.pack_weights(codes, bits, mq.LAYOUT_KERNEL, codes_signed=sym)
        return mq.PackedWeight(data, scale, zp, colsum, w.shape[0], w.shape[1], bits, mq.LAYOUT_KERNEL, sym)

    def weight(self, N, K, bits, sym=False, dtype=torch.float16):
        return self.packed(self.normal(N, K, std=0.02, dtype=dtype), bits, sym)

    def bias(self, N, dtype=torch.float16):
        return self.normal(N, std=0.01, dtype=dtype)

    def params(self, lo, hi):
        """Calibrated 8-bit parameters of the range [lo, hi]."""
        s = (hi - lo) / 255.0
        return (torch.tensor([s], dtype=torch.float32, device=self.dev),
                torch.tensor([int(round(-lo / s))], dtype=torch.int32, device=self.dev))

    def empty(self, *shape, dtype=torch.float16):
        return torch.empty(*shape, dtype=dtype, device=self.dev)

    def workspace(self, nbytes):
        return torch.empty(max(int(nbytes), 256), dtype=torch.uint8, device=self.dev)


def _dtype(case):
    return torch.bfloat16 if case.get("dtype") == "bf16" else torch.float16


_A8 = {8: mq.qlinear_w8a8, 4: mq.qlinear_w4a8, 2: mq.qlinear_w2a8}


def _block_layers(c):
    """(output width, input width, bias) of a transformer block's linears on the image tokens."""
    C = c["C"]
    return [(C, C, False)] * 3 + [(C, C, True), (C, C, False), (C, C, True), (8 * C, C, True), (C, 4 * C, True)]


def prepare(case, seed):
    g = _Make(seed)
    return {"linear": _prepare_linear, "kv": _prepare_kv, "kv_stacked": _prepare_kv_stacked, "block": _prepare_block,
            "ff": _prepare_ff, "resblock": _prepare_resblock, "prepare": _prepare_weights}[case["kind"]](case, g)


def _calls(calls, outs):
    def go():
        for call in calls:
            call()
        return outs
    return go


def _prepare_linear(c, g):
    dt = _dtype(c)
    x, w, bias = g.acts(c["M"], c["K"], dtype=dt), g.weight(c["N"], c["K"], c["bits"], c["sym"], dt), g.bias(c["N"], dt)
    if c["act"] == "none":
        return lambda: mq.qlinear_w_only(x, w, bias)
    act = g.params(-40.0, 40.0) if c["act"] == "static" else None
    return lambda: _A8[c["bits"]](x, w, act=act, bias=bias)[0]


def _prepare_kv(c, g):
    B, N = c["B"], c["N"]
    ctx = g.context(B)
    ws = g.workspace(mq.bos_aware_kv_proj_workspace_bytes(B, T, CTX) + mq.split_workspace_bytes(B * T, N, CTX))
    calls, outs = [], []
    for _ in range(2):
        w16, y = g.normal(N, CTX, std=0.02), g.empty(B, T, N)
        calls.append(mq.plan_bos_aware_kv_proj(ctx, g.packed(w16, c["bits"], c["sym"]), y, ws, w_f16=w16))
        outs.append(y)
    return _calls(calls, outs)


def _prepare_kv_stacked(c, g):
    B, N = c["B"], c["N"]
    ctx, y = g.context(B), g.empty(B, T, N)
    parts, bos = [], []
    for n0 in range(0, N, 20480):  # (a layer at a time, as a model loader does)
        w16 = g.normal(min(20480, N - n0), CTX, std=0.02)
        parts.append(g.packed(w16, c["bits"], c["sym"]))
        bos.append((ctx[0, 0].float() @ w16.float().T).half())
        del w16
    ws = g.workspace(mq.bos_aware_kv_proj_workspace_bytes(B, T, CTX) + mq.split_workspace_bytes(B * T, N, CTX))
    return _calls([mq.plan_bos_aware_kv_proj(ctx, mq.stack_weights(parts), y, ws, bos_out=torch.cat(bos))], [y])


def _prepare_block(c, g):
    """Self-attention q, k, v, out; cross-attention q, out; feed-forward projection and output; cross-attention k, v."""
    M, C, dt = c["M"], c["C"], _dtype(c)
    layers, B = _block_layers(c), c["B"]
    bits = [int(b) for b in c["bits"].split()]
    bits = bits * 10 if len(bits) == 1 else bits
    x = {C: g.acts(M, C, dtype=dt), 4 * C: g.acts(M, 4 * C, dtype=dt)}  # (the attention outputs are further tensors like x)
    attn, ctx = g.acts(M, C, dtype=dt), g.context(B)
    act = g.params(-40.0, 40.0) if c["act"] == "static" else None
    quant = c["act"] != "none"
    need = max(mq.split_workspace_bytes(M, N, K) + (mq.qlinear_a8_workspace_bytes(M, K) if quant else 0) for N, K, _ in layers)
    kv_need = mq.split_workspace_bytes(B * T, C, CTX) + (mq.bos_aware_kv_proj_workspace_bytes(B, T, CTX) if quant else 0)
    ws = g.workspace(max(need, kv_need))
    calls, outs = [], []
    for i, (N, K, has_bias) in enumerate(layers):
        w, bias, y = g.weight(N, K, bits[i], c["sym"], dt), g.bias(N, dt) if has_bias else None, g.empty(M, N, dtype=dt)
        src, res = (attn, x[C]) if i in (3, 5) else (x[K], x[C] if K == 4 * C else None)
        if quant:
            calls.append(mq.plan_qlinear_a8(src, w, bias, y, ws, act=act, residual=res))
        else:
            calls.append(mq.plan_qlinear_w_only(src, w, bias, y, residual=res, ws=ws))
        outs.append(y)
    for i in (8, 9):
        w16, y = g.normal(C, CTX, std=0.02), g.empty(B, T, C, dtype=dt)
        if quant:
            calls.append(mq.plan_bos_aware_kv_proj(ctx, g.packed(w16, bits[i], c["sym"]), y, ws, w_f16=w16))
        else:
            calls.append(mq.plan_qlinear_w_only(ctx.to(dt).view(B * T, CTX), g.packed(w16.to(dt), bits[i]), None, y.view(B * T, C), ws=ws))
        outs.append(y)
    return _calls(calls, outs)


def _prepare_ff(c, g):
    M, C, path = c["M"], c["C"], c["path"]
    H = 4 * C
    x = g.acts(M, C)
    w1, b1, w2, b2 = g.weight(2 * H, C, c["bits"], c["sym"]), g.bias(2 * H), g.weight(C, H, c["bits"], c["sym"]), g.bias(C)
    y = g.empty(M, C)
    mid = g.params(-2.0, 6.0)
    if path == "w_only":
        h = g.empty(M, H)
        second = mq.plan_qlinear_w_only(h, w2, b2, y, residual=x, ws=g.workspace(mq.split_workspace_bytes(M, C, H)))

        def go():
            mq.qlinear_w_only_geglu(x, w1, b1, out=h)
            second()
            return [h, y]
        return go
    if path == "w_only_a8":
        def go():
            codes, _ = mq.qlinear_w_only_geglu_a8(x, w1, mid, bias=b1)
            mq.qlinear_a8_codes(codes, H, mid, w2, bias=b2, out=y, residual=x)
            return [y]
        return go
    codes = g.empty(M, mq.a8_row_bytes(H), dtype=torch.int8)
    if path == "a8_static":
        ws = g.workspace(mq.qlinear_a8_workspace_bytes(M, C))
        calls = [mq.plan_qlinear_a8_geglu(x, w1, mid, b1, codes, ws, act=g.params(-40.0, 40.0)),
                 mq.plan_qlinear_a8_codes(codes, H, mid, w2, b2, y, residual=x)]
        return _calls(calls, [codes, y])
    ws, h = g.workspace(mq.qlinear_a8_geglu_dynamic_workspace_bytes(M, C, H)), g.empty(M, H)
    found = (g.empty(1, dtype=torch.float32), g.empty(1, dtype=torch.int32))
    calls = [mq.plan_qlinear_a8_geglu_dynamic(x, w1, b1, h, codes, found, ws),
             mq.plan_qlinear_a8_codes(codes, H, found, w2, b2, y, residual=x)]
    return _calls(calls, [h, codes, found[0], y])


def _prepare_resblock(c, g):
    B, H, W, cin, cout = c["B"], c["H"], c["W"], c["cin"], c["cout"]
    quant = c["act"] != "none"
    act = g.params(-40.0, 40.0) if c["act"] == "static" else None
    # the second convolution's input is the first one's output after a normalisation and an activation: another tensor
    x1, x2 = g.acts(B, H, W, cin), g.acts(B, H, W, cout)
    skip = g.normal(B, H, W, cout)
    ws = g.workspace(max(mq.conv3x3_a8_workspace_bytes(B, H, W, k) for k in (cin, cout))) if quant else None

    def conv(x, k, res, stride):
        codes, scale, zp = mq.quantize_weights(g.normal(cout, 9 * k, std=0.02), c["bits"], c["sym"])
        data, colsum = mq.pack_weights(codes, c["bits"], mq.LAYOUT_KERNEL, codes_signed=c["sym"])
        w = mq.PackedWeight(data, scale, zp, colsum, cout, 9 * k, c["bits"], mq.LAYOUT_KERNEL, c["sym"])
        bias = g.bias(cout)
        y = g.empty(B, (H - 1) // stride + 1, (W - 1) // stride + 1, cout)
        if not quant:
            return lambda: mq.conv3x3_w_only(x, w, bias, out=y, residual=res, stride=stride)
        taps = mq.conv_tap_sums(codes, k, c["bits"], c["sym"])
        return lambda: mq.conv3x3_a8(x, w, taps, act=act, bias=bias, out=y, ws=ws, residual=res, stride=stride)[0]

    calls = [conv(x1, cin, None, 1), conv(x2, cout, skip, 1)] + ([conv(x2, cout, None, 2)] if c["down"] else [])
    return lambda: [call() for call in calls]


def _prepare_weights(c, g):
    ws = [g.normal(N, K, std=0.02, dtype=_dtype(c)) for N, K, _ in _block_layers(c)]

    def go():
        out = []
        for w in ws:
            codes, scale, zp = mq.quantize_weights(w, c["bits"], c["sym"])
            packed, colsum = mq.pack_weights(codes, c["bits"], mq.LAYOUT_KERNEL, codes_signed=c["sym"])
            out.append((packed, scale, zp, colsum))
        return out
    return go


def run(state):
    return state()


# ------------------------------------------------------------------------------------------------- work, tolerance

def _linear_work(M, N, K, bits, residual=False):
    return 2 * M * K + N * K * bits // 8 + 10 * N + 2 * M * N * (2 if residual else 1), 2.0 * M * N * K


def work(case):
    c, parts = case, []
    kind = c["kind"]
    if kind == "linear":
        parts.append(_linear_work(c["M"], c["N"], c["K"], c["bits"]))
    elif kind == "kv":
        M, N = c["B"] * T, c["N"]
        b, f = _linear_work(M, N, CTX, c["bits"])
        parts += [(b + 2 * N * CTX, f), (b + 2 * N * CTX - 2 * M * CTX, f)]  # (both read one context)
    elif kind == "kv_stacked":
        parts.append(_linear_work(c["B"] * T, c["N"], CTX, c["bits"]))
    elif kind == "block":
        bits = [int(b) for b in c["bits"].split()] * 10
        for i, (N, K, _) in enumerate(_block_layers(c)):
            parts.append(_linear_work(c["M"], N, K, bits[i], i in (3, 5, 7)))
        for i in (8, 9):
            b, f = _linear_work(c["B"] * T, c["C"], CTX, bits[i])
            parts.append((b + (2 * c["C"] * CTX if c["act"] != "none" else 0), f))
    elif kind == "ff":
        M, C, H = c["M"], c["C"], 4 * c["C"]
        b1, f1 = _linear_work(M, 2 * H, C, c["bits"])
        b2, f2 = _linear_work(M, C, H, c["bits"], True)
        inner = {"w_only": (2, 2), "a8_static": (1, 1), "w_only_a8": (1, 1), "a8_dynamic": (3, 1)}[c["path"]]
        parts += [(b1 - 4 * M * H + inner[0] * M * H, f1), (b2 - 2 * M * H + inner[1] * M * H, f2)]
    elif kind == "resblock":
        B, H, W, cin, cout = c["B"], c["H"], c["W"], c["cin"], c["cout"]
        convs = [(cin, 1, False), (cout, 1, True)] + ([(cout, 2, False)] if c["down"] else [])
        for k, s, res in convs:
            M = B * ((H - 1) // s + 1) * ((W - 1) // s + 1)
            parts.append((2 * B * H * W * k + cout * 9 * k * c["bits"] // 8 + 10 * cout + 2 * M * cout * (2 if res else 1),
                          2.0 * M * cout * 9 * k))
    else:
        for N, K, _ in _block_layers(c):
            parts.append((2 * N * K + N * K * c["bits"] // 8 + 12 * N, 5.0 * N * K))  # range, scale, round, clamp
    return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}


def tolerance(case):
    if case["kind"] == "prepare":
        return "exact"
    if case.get("dtype") == "bf16":
        return {"rel": 6.5e-3, "max": 1.6e-2}  # (four times the error against 64-bit sums: 1.65e-3 and 3.9e-3)
    # four times the error of the 16-bit outputs against 64-bit sums (2.1e-4 and 4.9e-4); 8-bit codes of the gated product
    # may differ where the product lies at a rounding boundary
    return {"rel": 8e-4, "max": 2e-3, "differ": 1e-3}
