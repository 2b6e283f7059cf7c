"""The operator calls this library's performance is judged on.

Each case is what an eager program does per step: inputs, weights and the output buffer are in device memory, the
split-reduction workspace is registered once for the stream, and the call goes through the binding's entry points with
the built-in choice of kernel (no tuning records).  Families:

  gemm       one tir_gemm_fused; "a" / "b" say whether the operand is stored row-major ("n") or as its transpose ("t")
  bmm        one tir_batch_matmul_fused on dense [batch, rows, columns] tensors
  conv       one tir_conv2d_fused, channels-last, square filter with "same"-style padding dil * (r - 1) / 2
  separable  a depth-wise 3x3 convolution followed by the 1x1 convolution that mixes its channels
  downup     a strided 3x3 convolution and the 4x4 stride-2 transposed convolution that undoes its striding
  attention  one tir_attention over `batch` heads
"""
import torch

from paper_2207_04296_amd import binding as B

_TORCH = {"f16": torch.float16, "bf16": torch.bfloat16, "i8": torch.int8, "f32": torch.float32, "i32": torch.int32}
_SIZE = {"f16": 2, "bf16": 2, "i8": 1, "f32": 4, "i32": 4}
_MAX_FLOPS = 2.0 * 4096 ** 3
_MAX_BYTES = 256e6
_workspaces = {}


def listed():
    return [
        # the smallest GEMM anybody launches: nothing but call and launch latency
        dict(name="gemm_small_f16", kind="gemm", m=128, n=128, k=128, a="n", b="n", dtype="f16", out="f32", fused=False),
        # sizes that come from data, not from hardware: no extent is a multiple of anything, dense row-major operands
        dict(name="gemm_odd_f16", kind="gemm", m=1001, n=1531, k=777, a="n", b="n", dtype="f16", out="f16", fused=True),
        # feed-forward layer of a BERT-base-shaped block, bias and ReLU fused
        dict(name="gemm_ffn_f16", kind="gemm", m=2048, n=3072, k=768, a="n", b="n", dtype="f16", out="f16", fused=True),
        # weight gradient of that layer, dW = X^T dY: the reduction runs over the tokens, X is read as its transpose
        dict(name="gemm_wgrad_bf16", kind="gemm", m=768, n=3072, k=2048, a="t", b="n", dtype="bf16", out="f32", fused=False),
        # a large square GEMM
        dict(name="gemm_large_bf16", kind="gemm", m=4096, n=4096, k=4096, a="n", b="n", dtype="bf16", out="f32", fused=False),
        # attention scores of 16 sequences x 12 heads as a batched matmul, K^T by strides
        dict(name="bmm_qk_f16", kind="bmm", batch=192, m=128, n=128, k=64, b="t", dtype="f16", out="f32", fused=False),
        # 3x3 convolution of a ResNet-50-shaped first stage
        dict(name="conv_3x3_f16", kind="conv", images=16, h=56, w=56, c=64, filters=64, r=3, stride=1, dil=1, groups=1,
             dtype="f16", out="f16", fused=False),
        # the stem of an image network: three channels, a large filter, a large image
        dict(name="conv_stem_f16", kind="conv", images=16, h=224, w=224, c=3, filters=64, r=7, stride=2, dil=1, groups=1,
             dtype="f16", out="f16", fused=True),
        # quantised inference: grouped, dilated int8 convolution, requantised to int8 codes
        dict(name="conv_grouped_i8", kind="conv", images=8, h=28, w=28, c=256, filters=256, r=3, stride=1, dil=2, groups=8,
             dtype="i8", out="i8", fused=True),
        # a MobileNet-style block: depth-wise, then point-wise
        dict(name="separable_f16", kind="separable", images=16, h=56, w=56, c=128, filters=128, stride=1, dtype="f16"),
        # one level of an encoder / decoder: strided convolution down, transposed convolution up
        dict(name="downup_f16", kind="downup", images=16, h=28, w=28, c=128, filters=256, dtype="f16"),
        # attention over long sequences
        dict(name="attention_long_bf16", kind="attention", batch=16, m=4096, n=4096, d=128, dtype="bf16", out="bf16"),
    ]


def _log(rng, lo, hi):
    """An extent spread over the logarithm of [lo, hi]."""
    return max(lo, min(hi, round(lo * (hi / lo) ** rng.random())))


def _round(v, to):
    return max(to, v // to * to)


def _types(rng):
    dtype = rng.choice(["f16", "f16", "bf16", "bf16", "i8"])
    out = rng.choice({"f16": ["f16", "f32"], "bf16": ["bf16", "f32"], "i8": ["i8", "i32"]}[dtype])
    return dtype, out


def _draw_once(rng):
    kind = rng.choice(["gemm", "gemm", "gemm", "bmm", "conv", "conv", "separable", "downup", "attention"])
    if kind in ("gemm", "bmm"):
        dtype, out = _types(rng)
        odd = rng.random() < 0.25            # extents from data; the rest are network widths
        fused = rng.random() < 0.5
        if kind == "gemm":
            m, n, k = _log(rng, 16, 4096), _log(rng, 64, 4096), _log(rng, 64, 4096)
            if not odd:
                n, k = _round(n, 32), _round(k, 32)
                m = _round(m, 16)
            return dict(kind=kind, m=m, n=n, k=k, a="t" if rng.random() < 0.2 else "n", b=rng.choice("nt"), dtype=dtype, out=out,
                        fused=fused)
        m, n, k = _log(rng, 32, 1024), _log(rng, 32, 1024), rng.choice([32, 64, 96, 128])
        if not odd:
            m, n = _round(m, 16), _round(n, 16)
        return dict(kind=kind, batch=_log(rng, 4, 256), m=m, n=n, k=k, b=rng.choice("nt"), dtype=dtype, out=out, fused=fused)
    if kind == "conv":
        dtype, out = _types(rng)
        if rng.random() < 0.25:              # a stem
            return dict(kind=kind, images=_log(rng, 1, 32), h=_log(rng, 32, 256), w=_log(rng, 32, 256), c=rng.choice([1, 3, 4]),
                        filters=_round(_log(rng, 16, 128), 16), r=rng.choice([3, 5, 7]), stride=rng.choice([1, 2]), dil=1, groups=1,
                        dtype=dtype, out=out, fused=rng.random() < 0.5)
        groups = rng.choice([1, 1, 1, 2, 4, 8])
        return dict(kind=kind, images=_log(rng, 1, 32), h=_log(rng, 7, 112), w=_log(rng, 7, 112),
                    c=_round(_log(rng, 16, 512), 16) * groups, filters=_round(_log(rng, 16, 512), 16) * groups, r=rng.choice([1, 3, 3, 5]),
                    stride=rng.choice([1, 1, 2]), dil=rng.choice([1, 1, 2]), groups=groups, dtype=dtype, out=out,
                    fused=rng.random() < 0.5)
    if kind == "separable":
        return dict(kind=kind, images=_log(rng, 1, 32), h=_log(rng, 7, 112), w=_log(rng, 7, 112), c=_round(_log(rng, 32, 512), 16),
                    filters=_round(_log(rng, 32, 512), 16), stride=rng.choice([1, 2]), dtype=rng.choice(["f16", "bf16"]))
    if kind == "downup":
        return dict(kind=kind, images=_log(rng, 1, 32), h=2 * _log(rng, 4, 56), w=2 * _log(rng, 4, 56), c=_round(_log(rng, 32, 256), 32),
                    filters=_round(_log(rng, 32, 512), 32), dtype=rng.choice(["f16", "bf16"]))
    dtype = rng.choice(["f16", "bf16"])
    m = _log(rng, 64, 4096)
    return dict(kind=kind, batch=_log(rng, 8, 256), m=m, n=m if rng.random() < 0.6 else _log(rng, 64, 4096), d=rng.choice([64, 128]),
                dtype=dtype, out=rng.choice([dtype, dtype, "f32"]))


def draw(rng):
    """A case of the listed families: extents over the ranges of image and language networks, a share of them odd."""
    while True:
        case = _draw_once(rng)
        w = work(case)
        if w["flops"] <= _MAX_FLOPS and w["bytes"] <= _MAX_BYTES:
            return case


# ---------------------------------------------------------------------------------------------------------------------
def _conv_out(c):
    pad = c["dil"] * (c["r"] - 1) // 2
    span = c["dil"] * (c["r"] - 1) + 1
    return pad, (c["h"] + 2 * pad - span) // c["stride"] + 1, (c["w"] + 2 * pad - span) // c["stride"] + 1


def _separable_out(c):
    return (c["h"] - 1) // c["stride"] + 1, (c["w"] - 1) // c["stride"] + 1


def work(c):
    kind = c["kind"]
    es = _SIZE[c["dtype"]]
    if kind in ("gemm", "bmm"):
        batch, m, n, k = c.get("batch", 1), c["m"], c["n"], c["k"]
        bias = 4 * n if c["fused"] else 0
        return {"bytes": batch * (es * (m * k + k * n) + _SIZE[c["out"]] * m * n) + bias, "flops": 2.0 * batch * m * n * k}
    if kind == "conv":
        _, p, q = _conv_out(c)
        taps = c["r"] ** 2 * (c["c"] // c["groups"])
        pixels = c["images"] * p * q
        nbytes = es * (c["images"] * c["h"] * c["w"] * c["c"] + c["filters"] * taps) + _SIZE[c["out"]] * pixels * c["filters"]
        return {"bytes": nbytes + (4 * c["filters"] if c["fused"] else 0), "flops": 2.0 * pixels * c["filters"] * taps}
    if kind == "separable":
        p, q = _separable_out(c)
        pixels = c["images"] * p * q
        nbytes = es * (c["images"] * c["h"] * c["w"] * c["c"] + 9 * c["c"] + pixels * c["c"]          # depth-wise in, filter, out
                       + pixels * c["c"] + c["c"] * c["filters"] + pixels * c["filters"]) + 4 * (c["c"] + c["filters"])
        return {"bytes": nbytes, "flops": 2.0 * pixels * c["c"] * (9 + c["filters"])}
    if kind == "downup":
        big, small = c["images"] * c["h"] * c["w"], c["images"] * (c["h"] // 2) * (c["w"] // 2)
        nbytes = es * (2 * big * c["c"] + 2 * small * c["filters"] + (9 + 16) * c["c"] * c["filters"]) + 4 * (c["c"] + c["filters"])
        # every output pixel of the transposed convolution receives 16 / 4 taps
        return {"bytes": nbytes, "flops": 2.0 * c["c"] * c["filters"] * (9 * small + 4 * big)}
    batch, m, n, d = c["batch"], c["m"], c["n"], c["d"]
    return {"bytes": batch * d * (es * (m + 2 * n) + _SIZE[c["out"]] * m), "flops": 4.0 * batch * m * n * d}


def tolerance(c):
    kind = c["kind"]
    if c["dtype"] == "i8":
        return "exact"
    if kind in ("separable", "downup", "attention"):       # a 16-bit rounding between two products as well
        return {"rel": 1e-2 if c["dtype"] == "bf16" else 2e-3}
    return {"rel": {"f32": 1e-5, "f16": 1e-3, "bf16": 1e-2}[c["out"]]}


# ---------------------------------------------------------------------------------------------------------------------
def _workspace():
    """The buffer for split reductions, registered for the current stream by the first call that runs there."""
    stream = torch.cuda.current_stream().cuda_stream
    if stream not in _workspaces:
        ws = torch.empty(B.tir_workspace_bytes(), dtype=torch.uint8, device="cuda")
        B.tir_set_workspace(ws, stream=stream)
        _workspaces[stream] = ws


def _values(gen, shape, dtype, dist):
    """U(-1, 1), N(0, 0.1^2) or uniform int8 codes in [-127, 127]."""
    if dtype == "i8":
        return torch.randint(-127, 128, shape, generator=gen, device="cuda", dtype=torch.int8)
    if dist == "u":
        return (torch.rand(shape, generator=gen, device="cuda") * 2 - 1).to(_TORCH[dtype])
    return (torch.randn(shape, generator=gen, device="cuda") * 0.1).to(_TORCH[dtype])


def _epilogue(gen, channels, dtype, out, fused, reduction, relu=True):
    """(Epilogue or None, the bias tensor it points to): bias and ReLU when fused; the scale int8 codes need."""
    bias = None
    if fused:
        bias = (torch.randint(-8128, 8129, (channels,), generator=gen, device="cuda", dtype=torch.int32) if dtype == "i8"
                else torch.randn(channels, generator=gen, device="cuda") * 0.1)
    scale = 40.0 / (5376.0 * reduction ** 0.5) if out == "i8" else 0.0        # codes with a spread of about 40
    return B.make_epilogue(bias, relu and fused, scale), bias


def _empty(shape, dtype):
    return torch.empty(shape, dtype=_TORCH[dtype], device="cuda")


def prepare(case, seed):
    c = dict(case)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    _workspace()
    kind, dtype = c["kind"], c["dtype"]
    if kind in ("gemm", "bmm"):
        lead = (c["batch"],) if kind == "bmm" else ()
        m, n, k = c["m"], c["n"], c["k"]
        c["A"] = _values(gen, lead + ((k, m) if c.get("a", "n") == "t" else (m, k)), dtype, "u")
        c["B"] = _values(gen, lead + ((n, k) if c["b"] == "t" else (k, n)), dtype, "u")
        c["ep"], c["bias"] = _epilogue(gen, n, dtype, c["out"], c["fused"], k)
        c["C"] = _empty(lead + (m, n), c["out"])
    elif kind == "conv":
        c["pad"], p, q = _conv_out(c)
        cg = c["c"] // c["groups"]
        c["X"] = _values(gen, (c["images"], c["h"], c["w"], c["c"]), dtype, "n")
        c["W"] = _values(gen, (c["filters"], c["r"], c["r"], cg), dtype, "n")
        c["ep"], c["bias"] = _epilogue(gen, c["filters"], dtype, c["out"], c["fused"], c["r"] ** 2 * cg)
        c["Y"] = _empty((c["images"], p, q, c["filters"]), c["out"])
    elif kind == "separable":
        p, q = _separable_out(c)
        c["X"] = _values(gen, (c["images"], c["h"], c["w"], c["c"]), dtype, "n")
        c["W1"] = _values(gen, (c["c"], 3, 3, 1), dtype, "n")
        c["W2"] = _values(gen, (c["filters"], 1, 1, c["c"]), dtype, "n")
        c["ep1"], c["bias1"] = _epilogue(gen, c["c"], dtype, dtype, True, 9)
        c["ep2"], c["bias2"] = _epilogue(gen, c["filters"], dtype, dtype, True, c["c"], relu=False)
        c["Y1"] = _empty((c["images"], p, q, c["c"]), dtype)
        c["Y2"] = _empty((c["images"], p, q, c["filters"]), dtype)
        c["p"], c["q"] = p, q
    elif kind == "downup":
        h, w = c["h"], c["w"]
        c["X"] = _values(gen, (c["images"], h, w, c["c"]), dtype, "n")
        c["W1"] = _values(gen, (c["filters"], 3, 3, c["c"]), dtype, "n")
        c["W2"] = _values(gen, (c["c"], 4, 4, c["filters"]), dtype, "n")
        c["ep1"], c["bias1"] = _epilogue(gen, c["filters"], dtype, dtype, True, 9 * c["c"])
        c["ep2"], c["bias2"] = _epilogue(gen, c["c"], dtype, dtype, True, 4 * c["filters"])
        c["Y1"] = _empty((c["images"], h // 2, w // 2, c["filters"]), dtype)
        c["Y2"] = _empty((c["images"], h, w, c["c"]), dtype)
    else:
        batch, m, n, d = c["batch"], c["m"], c["n"], c["d"]
        c["Q"], c["K"], c["V"] = (torch.randn((batch, r, d), generator=gen, device="cuda").to(_TORCH[dtype]) for r in (m, n, n))
        c["O"] = _empty((batch, m, d), c["out"])
    return c


def run(s):
    kind, dtype = s["kind"], s["dtype"]
    if kind == "gemm":
        m, n, k = s["m"], s["n"], s["k"]
        a_rs, a_cs = (1, m) if s["a"] == "t" else (k, 1)
        b_rs, b_cs = (1, k) if s["b"] == "t" else (n, 1)
        B.tir_gemm_fused(s["A"], s["B"], s["C"], m, n, k, a_rs, a_cs, b_rs, b_cs, n, 1, dtype, s["out"], s["ep"])
        return s["C"]
    if kind == "bmm":
        m, n, k = s["m"], s["n"], s["k"]
        b_rs, b_cs = (1, k) if s["b"] == "t" else (n, 1)
        B.tir_batch_matmul_fused(s["A"], s["B"], s["C"], s["batch"], m, n, k, m * k, k, 1, k * n, b_rs, b_cs, m * n, n, 1, dtype,
                                 s["out"], s["ep"])
        return s["C"]
    if kind == "conv":
        B.tir_conv2d_fused(s["X"], s["W"], s["Y"], s["images"], s["h"], s["w"], s["c"], s["filters"], s["r"], s["r"], s["stride"],
                           s["stride"], s["pad"], s["pad"], s["dil"], s["dil"], s["groups"], dtype, s["out"], s["ep"])
        return s["Y"]
    if kind == "separable":
        B.tir_conv2d_fused(s["X"], s["W1"], s["Y1"], s["images"], s["h"], s["w"], s["c"], s["c"], 3, 3, s["stride"], s["stride"], 1, 1,
                           1, 1, s["c"], dtype, dtype, s["ep1"])
        B.tir_conv2d_fused(s["Y1"], s["W2"], s["Y2"], s["images"], s["p"], s["q"], s["c"], s["filters"], 1, 1, 1, 1, 0, 0, 1, 1, 1,
                           dtype, dtype, s["ep2"])
        return s["Y1"], s["Y2"]
    if kind == "downup":
        B.tir_conv2d_fused(s["X"], s["W1"], s["Y1"], s["images"], s["h"], s["w"], s["c"], s["filters"], 3, 3, 2, 2, 1, 1, 1, 1, 1,
                           dtype, dtype, s["ep1"])
        B.tir_conv2d_transpose(s["Y1"], s["W2"], s["Y2"], s["images"], s["h"] // 2, s["w"] // 2, s["filters"], s["c"], 4, 4, (2, 2),
                               (1, 1), (1, 1), (0, 0), 1, dtype, dtype, s["ep2"])
        return s["Y1"], s["Y2"]
    B.tir_attention(s["Q"], s["K"], s["V"], s["O"], s["batch"], s["m"], s["n"], s["d"], s["d"] ** -0.5, dtype, s["out"])
    return s["O"]
