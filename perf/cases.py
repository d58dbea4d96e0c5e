"""Timed cases: the work a program has this library do, one pass each.

Every case goes through the public entry points of the Python binding, with
the output buffers, plans and workspaces such a program keeps.  Sizes are
those of bench.py and the tests (bf16 and e4m3 8192^3, the 512^3 of the
bimodal queue, the decode and decode-layer shapes of width 5120, the
64-problem batch, the picker's training set) and generic ones between.

Kinds (what each stands for in use):
  gemm     one matrix product: square training-size products, small queue
           items, and contiguous tensors of any size (odd ones among them),
           B stored N x K (weights) or K x N, binary32 or bf16 output
  e4m3     quantised product, one scale per row of A and of B
  weight8  prefill with weight-only quantisation: bf16 activations times
           e4m3 weights with a scale per output column
  f32      binary32 product
  split    binary32 operands through bf16 planes (bf16x3, bf16x6)
  decode   M <= 16 rows times weights stored N x K, bf16 or e4m3
  layer    decode layer, fused: residual + rms_norm(x) . W^T
  norm_add prefill's element-wise part: rms_norm of the rows, then the
           residual add
  grouped  many uneven bf16 products in one launch (plan prepared once)
  picker   one training step of the tile picker's cost model: forward,
           backward, Adam
"""
import math

import torch

import paper_2606_15991_amd as tg

DEV = "cuda"
E4M3_MAX = 448.0
PICKER_IN, PICKER_HIDDEN, PICKER_DEPTH = tg.TG_PICKER_FEATURES, 64, 3


def listed():
    return [
        # the headline product of bench.py
        {"name": "gemm_bf16_8192", "kind": "gemm", "M": 8192, "N": 8192,
         "K": 8192, "nk": True, "out": "f32"},
        # the small item of the bimodal queue: latency
        {"name": "gemm_bf16_512", "kind": "gemm", "M": 512, "N": 512,
         "K": 512, "nk": True, "out": "f32"},
        # contiguous tensors whose rows are not 16-byte aligned
        {"name": "gemm_bf16_odd", "kind": "gemm", "M": 1111, "N": 1531,
         "K": 1003, "nk": False, "out": "bf16"},
        # the quantised headline
        {"name": "gemm_e4m3_8192", "kind": "e4m3", "M": 8192, "N": 8192,
         "K": 8192, "out": "f32"},
        # prefill of 512 tokens through weights quantised for decode
        {"name": "prefill_e4m3_weights", "kind": "weight8", "M": 512,
         "N": 5120, "K": 5120, "out": "bf16"},
        {"name": "gemm_f32_2048", "kind": "f32", "M": 2048, "N": 2048,
         "K": 2048, "nk": False},
        {"name": "gemm_bf16x6_4096", "kind": "split", "M": 4096, "N": 4096,
         "K": 4096, "nk": True, "precision": "bf16x6"},
        # the widest decode product of bench.py, eight rows in flight
        {"name": "decode_e4m3_8x51200", "kind": "decode", "M": 8, "N": 51200,
         "K": 5120, "w": "e4m3", "out": "bf16"},
        # one token through one decode layer
        {"name": "decode_layer_5120", "kind": "layer", "M": 1, "d": 5120,
         "w": "bf16"},
        {"name": "norm_add_4096x5120", "kind": "norm_add", "rows": 4096,
         "d": 5120, "dtype": "bf16"},
        # the mixed-shape batch of bench.py
        {"name": "grouped_64", "kind": "grouped", "n": 64, "shapes": 4,
         "nk": False, "out": "f32"},
        # one step over the samples that 2000 tuned shapes give
        {"name": "picker_step_20000", "kind": "picker", "batch": 20000},
    ]


def _log(rng, lo, hi, mult=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(mult, int(round(v / mult)) * mult)


def draw(rng):
    kind = rng.choice(["gemm", "gemm", "e4m3", "weight8", "f32", "split",
                       "decode", "decode", "layer", "norm_add", "grouped",
                       "picker"])
    c = {"kind": kind}
    if kind == "gemm":
        if rng.random() < 0.5:      # any size, contiguous
            hi, mult = 4096, 1
        else:
            hi, mult = 8192, 64
        c.update(M=_log(rng, 64, hi, mult), N=_log(rng, 64, hi, mult),
                 K=_log(rng, 64, hi, mult), nk=rng.random() < 0.5,
                 out=rng.choice(["f32", "bf16"]))
    elif kind == "e4m3":
        c.update(M=_log(rng, 128, 8192), N=_log(rng, 128, 8192),
                 K=_log(rng, 256, 8192, 16), out=rng.choice(["f32", "bf16"]))
    elif kind == "weight8":
        c.update(M=_log(rng, 17, 2048), N=_log(rng, 1024, 8192, 16),
                 K=_log(rng, 1024, 8192, 16), out=rng.choice(["f32", "bf16"]))
    elif kind == "f32":
        mult = rng.choice([1, 4, 64])
        c.update(M=_log(rng, 128, 4096, mult), N=_log(rng, 128, 4096, mult),
                 K=_log(rng, 128, 4096, mult), nk=rng.random() < 0.5)
    elif kind == "split":
        c.update(M=_log(rng, 256, 4096), N=_log(rng, 256, 4096, 8),
                 K=_log(rng, 256, 4096, 8), nk=rng.random() < 0.5,
                 precision=rng.choice(["bf16x3", "bf16x6"]))
    elif kind == "decode":
        N = _log(rng, 2048, 51200, 16)
        K = min(_log(rng, 1024, 25600, 16), 51200 * 5120 // N // 16 * 16)
        c.update(M=rng.choice([1, 1, 2, 4, 8, 16]), N=N, K=K,
                 w=rng.choice(["bf16", "e4m3"]),
                 out=rng.choice(["f32", "bf16"]))
    elif kind == "layer":
        c.update(M=rng.choice([1, 1, 2, 4, 8]), d=_log(rng, 1024, 8192, 16),
                 w=rng.choice(["bf16", "e4m3"]))
    elif kind == "norm_add":
        c.update(rows=_log(rng, 1, 8192), d=_log(rng, 1024, 8192, 8),
                 dtype=rng.choice(["bf16", "f32"]))
    elif kind == "grouped":
        c.update(n=rng.randint(4, 24), shapes=rng.randint(5, 1 << 20),
                 nk=rng.random() < 0.5, out=rng.choice(["f32", "bf16"]))
    else:
        c.update(batch=_log(rng, 500, 40000))
    return c


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _normal(shape, g, std=1.0, dtype=torch.bfloat16):
    return (torch.randn(shape, generator=g, device=DEV) * std).to(dtype)


def _quant_rows(w):
    """e4m3 codes and one scale per row (row maximum / 448)."""
    s = w.abs().amax(dim=1) / E4M3_MAX
    s = torch.where(s > 0, s, torch.ones_like(s))
    return (w / s[:, None]).clamp(-E4M3_MAX, E4M3_MAX).to(
        torch.float8_e4m3fn), s


def _out(shape, name):
    return torch.empty(shape, device=DEV,
                       dtype=torch.float32 if name == "f32"
                       else torch.bfloat16)


def _b_shape(c):
    return (c["N"], c["K"]) if c["nk"] else (c["K"], c["N"])


def _grouped_shapes(c):
    """M uniform in 1..2048, N and K multiples of 128 in 1024..8192."""
    g = torch.Generator().manual_seed(c["shapes"])
    m = torch.randint(1, 2049, (c["n"],), generator=g)
    n = torch.randint(8, 65, (c["n"],), generator=g) * 128
    k = torch.randint(8, 65, (c["n"],), generator=g) * 128
    return [(int(a), int(b), int(d)) for a, b, d in zip(m, n, k)]


def prepare(case, seed):
    c, g = case, _gen(seed)
    s = {"case": dict(c)}
    kind = c["kind"]
    if kind == "gemm":
        s["A"] = _normal((c["M"], c["K"]), g)
        s["B"] = _normal(_b_shape(c), g)
        s["C"] = _out((c["M"], c["N"]), c["out"])
    elif kind == "e4m3":
        s["A"], s["sa"] = _quant_rows(_normal((c["M"], c["K"]), g,
                                              dtype=torch.float32))
        s["B"], s["sb"] = _quant_rows(_normal((c["N"], c["K"]), g,
                                              dtype=torch.float32))
        s["C"] = _out((c["M"], c["N"]), c["out"])
    elif kind in ("weight8", "decode"):
        s["A"] = _normal((c["M"], c["K"]), g)
        w = _normal((c["N"], c["K"]), g, 0.02, torch.float32)
        if kind == "weight8" or c["w"] == "e4m3":
            s["B"], s["sb"] = _quant_rows(w)
        else:
            s["B"], s["sb"] = w.to(torch.bfloat16), None
        s["C"] = _out((c["M"], c["N"]), c["out"])
    elif kind in ("f32", "split"):
        s["A"] = _normal((c["M"], c["K"]), g, dtype=torch.float32)
        s["B"] = _normal(_b_shape(c), g, dtype=torch.float32)
        s["C"] = _out((c["M"], c["N"]), "f32")
        if kind == "split":
            s["ws"] = torch.empty(
                tg.tile_gemm_workspace_size(s["A"], s["B"], s["C"],
                                            b_trans=c["nk"],
                                            precision=c["precision"]),
                dtype=torch.uint8, device=DEV)
    elif kind == "layer":
        M, d = c["M"], c["d"]
        s["x"] = _normal((M, d), g)
        s["nw"] = (1 + _normal((d,), g, 0.1, torch.float32)).to(
            torch.bfloat16)
        w = _normal((d, d), g, 0.02, torch.float32)
        if c["w"] == "e4m3":
            s["W"], s["sw"] = _quant_rows(w)
        else:
            s["W"], s["sw"] = w.to(torch.bfloat16), None
        s["y"] = _out((M, d), "bf16")
    elif kind == "norm_add":
        dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
        s["x"] = _normal((c["rows"], c["d"]), g, 2.0, dt)
        s["r"] = _normal((c["rows"], c["d"]), g, 1.0, dt)
        s["nw"] = (1 + _normal((c["d"],), g, 0.1, torch.float32)).to(dt)
        s["y"] = torch.empty_like(s["x"])
        s["z"] = torch.empty_like(s["x"])
    elif kind == "grouped":
        sh = _grouped_shapes(c)
        As = [_normal((m, k), g) for m, n, k in sh]
        Bs = [_normal((n, k) if c["nk"] else (k, n), g) for m, n, k in sh]
        Cs = [_out((m, n), c["out"]) for m, n, k in sh]
        s["launch"] = tg.tile_gemm_grouped_prepare(As, Bs, Cs,
                                                   b_trans=c["nk"])
    else:
        B, n_in, hid, dep = (c["batch"], PICKER_IN, PICKER_HIDDEN,
                             PICKER_DEPTH)
        dims, parts = [n_in] + [hid] * dep + [1], []
        for i, o in zip(dims[:-1], dims[1:]):
            lim = math.sqrt(6.0 / i)
            parts.append((torch.rand(o * i, generator=g, device=DEV) * 2 - 1)
                         * lim)
            parts.append(torch.randn(o, generator=g, device=DEV) * 0.1)
        s["p"] = torch.cat(parts)
        s["X"] = _normal((B, n_in), g, dtype=torch.float32)
        s["y"] = _normal((B,), g, 0.5, torch.float32)
        # moments as they stand in the middle of a training run
        s["m"] = torch.randn(s["p"].numel(), generator=g, device=DEV) * 1e-2
        s["v"] = torch.rand(s["p"].numel(), generator=g, device=DEV) * 1e-3
        s["v"] += 1e-4
        s["t"] = 100
        s["grads"] = torch.empty_like(s["p"])
        s["loss"] = torch.empty(1, device=DEV)
        s["ws"] = torch.empty(tg.tile_mlp_workspace_bytes(n_in, hid, dep, B),
                              dtype=torch.uint8, device=DEV)
    return s


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind in ("gemm", "f32"):
        tg.tile_gemm(s["A"], s["B"], s["C"], b_trans=c["nk"])
        return s["C"]
    if kind == "split":
        tg.tile_gemm(s["A"], s["B"], s["C"], b_trans=c["nk"],
                     precision=c["precision"], workspace=s["ws"])
        return s["C"]
    if kind == "e4m3":
        tg.tile_gemm(s["A"], s["B"], s["C"], b_trans=True, scale_a=s["sa"],
                     scale_b=s["sb"])
        return s["C"]
    if kind in ("weight8", "decode"):
        tg.tile_gemm(s["A"], s["B"], s["C"], b_trans=True, scale_b=s["sb"])
        return s["C"]
    if kind == "layer":
        return tg.tile_rms_norm_matvec(s["x"], s["nw"], s["W"], s["y"],
                                       scale_w=s["sw"], residual=s["x"])
    if kind == "norm_add":
        tg.tile_rms_norm(s["x"], s["nw"], s["y"])
        tg.tile_add(s["y"], s["r"], s["z"])
        return s["y"], s["z"]
    if kind == "grouped":
        return list(tg.tile_gemm_grouped(s["launch"]))
    n_in, hid, dep = PICKER_IN, PICKER_HIDDEN, PICKER_DEPTH
    tg.tile_mlp_loss_grad(s["p"], s["X"], s["y"], n_in, hid, dep,
                          grads=s["grads"], loss=s["loss"], ws=s["ws"])
    tg.tile_mlp_adam(s["p"], s["grads"], s["m"], s["v"], s["t"], lr=3e-3)
    s["t"] += 1
    return {"loss": s["loss"], "grads": s["grads"], "p": s["p"],
            "m": s["m"], "v": s["v"]}


def work(case):
    c, kind = case, case["kind"]
    osz = 2 if c.get("out") == "bf16" else 4
    if kind in ("gemm", "e4m3", "weight8", "f32", "split", "decode"):
        M, N, K = c["M"], c["N"], c["K"]
        a = {"gemm": 2, "e4m3": 1, "weight8": 2, "f32": 4, "split": 4,
             "decode": 2}[kind]
        b = {"gemm": 2, "e4m3": 1, "weight8": 1, "f32": 4, "split": 4,
             "decode": 1 if c.get("w") == "e4m3" else 2}[kind]
        planes = {"bf16x3": 3, "bf16x6": 6}.get(c.get("precision"), 1)
        scales = {"e4m3": 4 * (M + N), "weight8": 4 * N,
                  "decode": 4 * N if c.get("w") == "e4m3" else 0}
        return {"bytes": M * K * a + N * K * b + M * N * osz +
                scales.get(kind, 0), "flops": 2 * M * N * K * planes}
    if kind == "layer":
        M, d = c["M"], c["d"]
        w = 1 if c["w"] == "e4m3" else 2
        return {"bytes": d * d * w + (4 * d if w == 1 else 0) + 2 * d +
                4 * M * d, "flops": 2 * M * d * d}
    if kind == "norm_add":
        es = 2 if c["dtype"] == "bf16" else 4
        n = c["rows"] * c["d"]
        # x and r read, y and z written
        return {"bytes": 4 * n * es + c["d"] * es, "flops": 5 * n}
    if kind == "grouped":
        sh = _grouped_shapes(c)
        return {"bytes": sum(2 * (m * k + k * n) + osz * m * n
                             for m, n, k in sh),
                "flops": sum(2 * m * n * k for m, n, k in sh)}
    B, n_in, hid, dep = c["batch"], PICKER_IN, PICKER_HIDDEN, PICKER_DEPTH
    w = n_in * hid + (dep - 1) * hid * hid + hid
    params = w + dep * hid + 1
    # forward, weight gradients, input gradients of all layers but the first
    return {"bytes": 4 * (B * (n_in + 1) + 8 * params),
            "flops": 2 * B * (3 * w - n_in * hid)}


def _f64(t):
    return (t.to(torch.float32) if t.dtype == torch.float8_e4m3fn
            else t).double()


def _mm(A, B, nk):
    b = _f64(B)
    return _f64(A) @ (b.t() if nk else b)


def exact(case, seed):
    c, kind = case, case["kind"]
    s = prepare(case, seed)
    if kind in ("gemm", "f32", "split"):
        return _mm(s["A"], s["B"], c["nk"])
    if kind == "e4m3":
        return (_mm(s["A"], s["B"], True) * s["sa"].double()[:, None] *
                s["sb"].double()[None, :])
    if kind in ("weight8", "decode"):
        R = _mm(s["A"], s["B"], True)
        return R if s["sb"] is None else R * s["sb"].double()[None, :]
    if kind == "layer":
        x = s["x"].double()
        # the weighted activations are held in bf16 (the library's
        # definition of the fused product); their product is exact in 64
        # bits
        h = (x * s["nw"].double()).to(torch.bfloat16).double()
        y = h @ _f64(s["W"]).t()
        y = y / torch.sqrt((x * x).mean(dim=1, keepdim=True) + 1e-6)
        if s["sw"] is not None:
            y = y * s["sw"].double()[None, :]
        return y + x
    if kind == "norm_add":
        x = s["x"].double()
        y = x * s["nw"].double() / torch.sqrt(
            (x * x).mean(dim=1, keepdim=True) + 1e-6)
        # the sum's own input is the stored y
        return y, y.to(s["x"].dtype).double() + s["r"].double()
    if kind == "grouped":
        L = s["launch"]
        return [_mm(a, b, c["nk"]) for a, b in zip(L.As, L.Bs)]
    n_in, hid, dep = PICKER_IN, PICKER_HIDDEN, PICKER_DEPTH
    p, X, y = s["p"].double(), s["X"].double(), s["y"].double()
    dims, layers, o0 = [n_in] + [hid] * dep + [1], [], 0
    for i, o in zip(dims[:-1], dims[1:]):
        layers.append((p[o0:o0 + o * i].view(o, i),
                       p[o0 + o * i:o0 + o * i + o]))
        o0 += o * i + o
    acts = [X]
    for n, (W, b) in enumerate(layers):
        z = acts[-1] @ W.t() + b
        acts.append(z.clamp(min=0) if n < dep else z)
    d = acts[-1][:, 0] - y
    dz, parts = (2 * d / X.shape[0])[:, None], []
    for n in range(dep, -1, -1):
        parts[:0] = [(dz.t() @ acts[n]).reshape(-1), dz.sum(dim=0)]
        if n:
            dz = (dz @ layers[n][0]) * (acts[n] > 0)
    gr = torch.cat(parts)
    m = 0.9 * s["m"].double() + 0.1 * gr
    v = 0.999 * s["v"].double() + 0.001 * gr * gr
    t = s["t"]
    p = p - 3e-3 * (m / (1 - 0.9 ** t)) / (
        torch.sqrt(v / (1 - 0.999 ** t)) + 1e-8)
    return {"loss": (d * d).mean().reshape(1), "grads": gr, "p": p, "m": m,
            "v": v}
