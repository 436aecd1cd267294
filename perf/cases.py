"""The work this library is used for, as cases that can be timed: every entry point of include/gensor.h through its
binding (gemm, bmm, conv2d, gemv, avgpool2d), with the schedule and workspace a program constructs once and keeps.
Shapes are the benchmark's own configurations (paper_2502_11407_amd/inputs.py) or generic ones; inputs are drawn on
the GPU from the seed alone, uniform in [-1, 1) or normal as the configurations state, and rounded once."""
import math

import torch

from paper_2502_11407_amd import binding as gs

TORCH = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
BYTES = {"f32": 4, "f16": 2, "bf16": 2}


def _gemm(name, dtype, out, M, N, K, ta=0, tb=0, batch=1, values="uniform", w_sigma=1.0):
    c = dict(kind="gemm", dtype=dtype, out=out, M=M, N=N, K=K, ta=ta, tb=tb, batch=batch, values=values, w_sigma=w_sigma)
    return dict(c, name=name) if name else c


def _conv(name, dtype, out, n, c, h, w, k, r, stride, pad):
    d = dict(kind="conv", dtype=dtype, out=out, n=n, c=c, h=h, w=w, k=k, r=r, stride=stride, pad=pad)
    return dict(d, name=name) if name else d


def _gemv(name, dtype, M, N):
    c = dict(kind="gemv", dtype=dtype, out="f32", M=M, N=N)
    return dict(c, name=name) if name else c


def _pool(name, dtype, out, n, c, h, w, f, stride):
    d = dict(kind="pool", dtype=dtype, out=out, n=n, c=c, h=h, w=w, f=f, stride=stride)
    return dict(d, name=name) if name else d


def listed():
    return [
        # the smallest call of the benchmark: a single small fp32 product, bound by latency
        _gemm("gemm_f32_512", "f32", "f32", 512, 512, 512),
        # the headline: a large square fp16 product with column-major B and fp32 output
        _gemm("gemm_f16_4096", "f16", "f32", 4096, 4096, 4096, tb=1),
        # a transformer MLP projection, forward, activations kept in bf16
        _gemm("mlp_up_bf16", "bf16", "bf16", 8192, 3072, 768, values="normal", w_sigma=0.02),
        # the same layer's weight gradient, dW = X^T dY: m-contiguous A, reduction over the tokens, fp32 result
        _gemm("mlp_wgrad_f16", "f16", "f32", 768, 3072, 8192, ta=1, values="normal"),
        # attention scores of a batch of heads, shallow reduction, bound by the output
        _gemm("bmm_scores_f16", "f16", "f32", 1024, 1024, 64, tb=1, batch=96, values="normal"),
        # nothing is a multiple of anything: rows that start off every vector boundary
        _gemm("gemm_ragged_bf16", "bf16", "f32", 2039, 1511, 1003, tb=1),
        # few output tiles and a deep reduction: the shape a split along k exists for
        _gemm("gemm_deep_k_f16", "f16", "f32", 512, 512, 32768, tb=1),
        # residual-network body: 3x3 convolution
        _conv("conv_3x3_f16", "f16", "f32", 32, 64, 56, 56, 64, 3, 1, 1),
        # residual-network shortcut: pointwise convolution with stride 2
        _conv("conv_1x1_s2_f16", "f16", "f16", 32, 256, 56, 56, 512, 1, 2, 0),
        # image input layer: three channels, a large filter, stride 2
        _conv("conv_7x7_rgb_f16", "f16", "f32", 16, 3, 112, 112, 64, 7, 2, 3),
        # matrix-vector product of the operator table (rows that are not whole panels)
        _gemv("gemv_f16", "f16", 16384, 8192),
        # average pooling of the operator table: odd image rows
        _pool("avgpool_f16", "f16", "f32", 128, 168, 83, 83, 2, 2),
    ]


def _logint(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _mult(rng, lo, hi, m):
    return max(m, _logint(rng, lo, hi) // m * m)


def _half(rng):
    return rng.choice(["f16", "bf16"])


def _out(rng, dtype):
    return rng.choice(["f32", dtype])


def draw(rng):
    family = rng.choice(["small", "square", "mlp", "wgrad", "bmm", "ragged", "deep", "conv3", "pointwise", "conv_wide", "gemv", "pool"])
    if family == "small":          # small fp32 products, sizes as they come
        return _gemm(None, "f32", "f32", _logint(rng, 64, 1024), _logint(rng, 64, 1024), _logint(rng, 64, 1024), tb=rng.randint(0, 1))
    if family == "square":
        dt = _half(rng)
        return _gemm(None, dt, "f32", *[_mult(rng, 1024, 4096, 64) for _ in range(3)], tb=rng.randint(0, 1))
    if family == "mlp":            # rows = tokens, forward (row-major weights) and input gradient (transposed weights)
        dt, d, rows = _half(rng), _mult(rng, 512, 1024, 64), _logint(rng, 256, 8192)
        a, b = (d, 4 * d) if rng.random() < 0.5 else (4 * d, d)
        return _gemm(None, dt, _out(rng, dt), rows, b, a, tb=rng.randint(0, 1), values="normal", w_sigma=0.02)
    if family == "wgrad":
        dt, d = _half(rng), _mult(rng, 512, 1024, 64)
        a, b = (d, 4 * d) if rng.random() < 0.5 else (4 * d, d)
        return _gemm(None, dt, "f32", a, b, _mult(rng, 512, 8192, 8), ta=1, values="normal")
    if family == "bmm":            # scores (shallow k) and values (k = sequence), any sequence length
        dt, head, seq, batch = _half(rng), rng.choice([64, 128]), _logint(rng, 100, 1024), rng.randint(4, 96)
        if rng.random() < 0.5:
            return _gemm(None, dt, _out(rng, dt), seq, seq, head, tb=1, batch=batch, values="normal")
        return _gemm(None, dt, _out(rng, dt), seq, head, seq, batch=batch, values="normal")
    if family == "ragged":
        dt = rng.choice(["f32", "f16", "bf16"])
        return _gemm(None, dt, "f32", *[_logint(rng, 150, 2047) | 1 for _ in range(3)], ta=int(rng.random() < 0.25), tb=rng.randint(0, 1))
    if family == "deep":
        return _gemm(None, _half(rng), "f32", _mult(rng, 128, 768, 8), _mult(rng, 128, 768, 8), _mult(rng, 4096, 32768, 64), tb=rng.randint(0, 1))
    if family == "conv3":
        dt = rng.choice(["f16", "bf16", "f16", "bf16", "f32"])
        hw, ch = _logint(rng, 14, 58), _mult(rng, 32, 256, 8)
        n = max(1, min(_logint(rng, 4, 64), 3500000 // (hw * hw * ch)))
        return _conv(None, dt, "f32" if dt == "f32" else _out(rng, dt), n, ch, hw, hw, _mult(rng, 32, 256, 8), 3, rng.choice([1, 1, 2]), 1)
    if family == "pointwise":
        dt = _half(rng)
        hw, ch = _logint(rng, 7, 56), _mult(rng, 64, 512, 8)
        n = max(1, min(_logint(rng, 4, 64), 25000000 // (hw * hw * ch)))
        return _conv(None, dt, _out(rng, dt), n, ch, hw, hw, _mult(rng, 64, 512, 8), 1, rng.choice([1, 2]), 0)
    if family == "conv_wide":      # large filters, few channels
        dt, r = _half(rng), rng.choice([5, 7])
        return _conv(None, dt, "f32", rng.randint(1, 16), rng.choice([1, 3, 4, 6, 16]), _logint(rng, 28, 112), _logint(rng, 28, 112),
                     _mult(rng, 16, 64, 2), r, rng.choice([1, 2]), r // 2)
    if family == "gemv":
        return _gemv(None, rng.choice(["f32", "f16", "bf16"]), _logint(rng, 256, 16384), _logint(rng, 500, 8192))
    dt = rng.choice(["f32", "f16", "bf16"])
    hw, f = _logint(rng, 14, 112), rng.choice([2, 3])
    planes = max(1, 130000000 // (hw * hw))
    return _pool(None, dt, "f32" if dt == "f32" else _out(rng, dt), rng.randint(1, 128), min(_logint(rng, 16, 617), max(1, planes // 128)), hw, hw + rng.randint(0, 3), f, 2)


# ---------------------------------------------------------------------------------------------------------------------
def _inputs(case, seed):
    """The two operands (one for the pooling) in their storage type, from the seed alone."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    dt = TORCH[case["dtype"]]

    def draw_values(shape, normal, sigma=1.0):
        t = torch.empty(shape, dtype=torch.float32, device="cuda")
        t = t.normal_(0.0, sigma, generator=g) if normal else t.uniform_(-1.0, 1.0, generator=g)
        return t.to(dt)

    if case["kind"] == "gemm":
        M, N, K, b = case["M"], case["N"], case["K"], case["batch"]
        sa, sb = ((K, M) if case["ta"] else (M, K)), ((N, K) if case["tb"] else (K, N))
        if b > 1:
            sa, sb = (b,) + sa, (b,) + sb
        normal = case["values"] == "normal"
        return draw_values(sa, normal), draw_values(sb, normal, case["w_sigma"])
    if case["kind"] == "conv":
        fan_in = case["c"] * case["r"] * case["r"]
        return (draw_values((case["n"], case["c"], case["h"], case["w"]), True),
                draw_values((case["k"], case["c"], case["r"], case["r"]), True, math.sqrt(2.0 / fan_in)))
    if case["kind"] == "gemv":
        return draw_values((case["M"], case["N"]), False), draw_values((case["N"],), False)
    return (draw_values((case["n"], case["c"], case["h"], case["w"]), True),)


def _conv_out(case):
    return ((case["h"] + 2 * case["pad"] - case["r"]) // case["stride"] + 1, (case["w"] + 2 * case["pad"] - case["r"]) // case["stride"] + 1)


def _pool_out(case):
    return (case["h"] - case["f"]) // case["stride"] + 1, (case["w"] - case["f"]) // case["stride"] + 1


def prepare(case, seed):
    x = _inputs(case, seed)
    if case["kind"] == "gemm":
        p = gs.gemm_problem(case["dtype"], case["M"], case["N"], case["K"], case["ta"], case["tb"], case["batch"], case["out"])
        shape = (case["M"], case["N"]) if case["batch"] == 1 else (case["batch"], case["M"], case["N"])
        s = gs.construct(p)
        return dict(call=gs.gemm if case["batch"] == 1 else gs.bmm, p=p, x=x, s=s, ws=gs.gemm_workspace(p, s), out=gs.empty_device(shape, case["out"]))
    if case["kind"] == "conv":
        p = gs.conv_problem(case["dtype"], case["n"], case["c"], case["h"], case["w"], case["k"], case["r"], case["r"], case["stride"], case["pad"], case["out"])
        # (large filters leave the schedule to the library: a constructed one asks for vector reads, which the filters
        # of three channels cannot give)
        s = gs.construct(p) if case["r"] <= 3 else None
        return dict(call=gs.conv2d, p=p, x=x, s=s, ws=gs.conv_workspace(p, s), out=gs.empty_device((case["n"], case["k"]) + _conv_out(case), case["out"]))
    if case["kind"] == "gemv":
        return dict(call=gs.gemv, dtype=case["dtype"], x=x, out=gs.empty_device((case["M"],)))
    return dict(call=gs.avgpool2d, dtype=case["dtype"], x=x, out=gs.empty_device((case["n"], case["c"]) + _pool_out(case), case["out"]),
                f=case["f"], stride=case["stride"], out_dtype=case["out"])


def run(state):
    call, x, out = state["call"], state["x"], state["out"]
    if call is gs.gemv:
        call(state["dtype"], x[0], x[1], out)
    elif call is gs.avgpool2d:
        call(state["dtype"], x[0], out, state["f"], state["stride"], state["out_dtype"])
    else:
        call(state["p"], x[0], x[1], out, schedule=state["s"], workspace=state["ws"])
    return out


def work(case):
    e, eo = BYTES[case["dtype"]], BYTES[case["out"]]
    if case["kind"] == "gemm":
        M, N, K, b = case["M"], case["N"], case["K"], case["batch"]
        return {"bytes": b * (e * (M * K + K * N) + eo * M * N), "flops": 2 * b * M * N * K}
    if case["kind"] == "conv":
        P, Q = _conv_out(case)

        def touched(extent, outs):           # input rows (or columns) that some window reads
            seen = {o * case["stride"] - case["pad"] + i for o in range(outs) for i in range(case["r"])}
            return sum(1 for v in seen if 0 <= v < extent)
        inp = case["n"] * case["c"] * touched(case["h"], P) * touched(case["w"], Q)
        filt = case["k"] * case["c"] * case["r"] * case["r"]
        outs = case["n"] * case["k"] * P * Q
        return {"bytes": e * (inp + filt) + eo * outs, "flops": 2 * outs * case["c"] * case["r"] * case["r"]}
    if case["kind"] == "gemv":
        return {"bytes": e * (case["M"] * case["N"] + case["N"]) + 4 * case["M"], "flops": 2 * case["M"] * case["N"]}
    P, Q = _pool_out(case)
    planes = case["n"] * case["c"]
    return {"bytes": e * planes * case["h"] * case["w"] + eo * planes * P * Q, "flops": planes * P * Q * case["f"] * case["f"]}


def tolerance(case):
    """fp32 sums of exact (16-bit) or once-rounded (fp32) products: the error grows like the square root of the depth.
    A 16-bit output adds one rounding to nearest, at most 2^-9 (bf16) or 2^-12 (fp16) of the value.  Each bound is about
    four times the measured distance to 64-bit sums (512 fp32: 4e-7, 4096 fp16: 4e-7, bf16 output: 1.7e-3, fp16: 2.1e-4)."""
    if case["out"] == "bf16":
        return {"rel": 7e-3}
    if case["out"] == "f16":
        return {"rel": 9e-4}
    if case["kind"] == "pool":
        return {"rel": 3e-7}
    if case["kind"] == "conv":
        depth = case["c"] * case["r"] * case["r"]
    else:
        depth = case["K"] if case["kind"] == "gemm" else case["N"]
    return {"rel": 3e-7 + 4e-8 * math.sqrt(depth)}


def exact(case, seed):
    x = [t.to(torch.float64) for t in _inputs(case, seed)]
    if case["kind"] == "gemm":
        a = x[0].transpose(-1, -2).contiguous() if case["ta"] else x[0]
        b = x[1].transpose(-1, -2).contiguous() if case["tb"] else x[1]
        if case["batch"] == 1:
            return a @ b
        return torch.stack([a[i] @ b[i] for i in range(case["batch"])])
    if case["kind"] == "conv":
        # one product per filter tap on the shifted, subsampled, zero-padded input
        inp, wgt = x
        P, Q = _conv_out(case)
        st, pad = case["stride"], case["pad"]
        padded = torch.zeros((case["n"], case["c"], case["h"] + 2 * pad, case["w"] + 2 * pad), dtype=torch.float64, device="cuda")
        padded[:, :, pad:pad + case["h"], pad:pad + case["w"]] = inp
        rows = padded.permute(1, 0, 2, 3).contiguous()                      # channel first: one matrix per tap
        out = torch.zeros((case["k"], case["n"] * P * Q), dtype=torch.float64, device="cuda")
        for r in range(case["r"]):
            for s in range(case["r"]):
                tap = rows[:, :, r:r + st * (P - 1) + 1:st, s:s + st * (Q - 1) + 1:st].contiguous().view(case["c"], -1)
                out += wgt[:, :, r, s].contiguous() @ tap
        return out.view(case["k"], case["n"], P, Q).permute(1, 0, 2, 3).contiguous()
    if case["kind"] == "gemv":
        return x[0] @ x[1]
    P, Q = _pool_out(case)
    f, st = case["f"], case["stride"]
    out = torch.zeros((case["n"], case["c"], P, Q), dtype=torch.float64, device="cuda")
    for i in range(f):
        for j in range(f):
            out += x[0][:, :, i:i + st * (P - 1) + 1:st, j:j + st * (Q - 1) + 1:st]
    return out / (f * f)
