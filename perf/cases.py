"""Performance cases of the sparse linear library: the work its users run, through its public entry points.

A case is a dict of plain values.  Its "kind" says which calls one pass makes:

* ``linear``    one ``sparse_linear`` call, issued eagerly: the smallest unit of work, where launch and
                call overhead count;
* ``decode``    a token step of a few decoder layers at a small batch, replayed as one HIP graph (how a
                serving loop issues it): q|k|v as a group, o, gate|up as a group or as the fused gated half,
                down;
* ``decode_q``  the same step with quantized weights: per-token int8 activations, then int8 groups or 4-bit
                linears;
* ``prefill``   a prompt through one decoder layer, issued eagerly: q|k|v, o, the gated half, down;
* ``prefill_q`` the same in int8: activations quantized per token, then the seven int8 linears;
* ``train``     one masked training step of a layer's seven linears: forward, weight gradients, SGD on the
                stored values, input gradients;
* ``compress``  pruning, packing and unpacking a layer's seven matrices.

``hidden`` and ``ffn`` are the layer's widths: q, k, v, o are hidden x hidden, gate and up ffn x hidden, down
hidden x ffn.  Weights are N(0, 0.02^2) with the smallest magnitudes pruned, activations N(0, 1).
"""
from __future__ import annotations

import math

import torch

import paper_2405_03594_amd as spl

STD = 0.02
LR = 0.01
DTYPES = {"bf16": torch.bfloat16, "fp16": torch.float16}


def listed():
    return [
        # one projection at batch 1 (a call from eager code): the smallest call
        {"name": "linear_b1", "kind": "linear", "m": 1, "n": 4096, "k": 4096, "dtype": "fp16", "sparsity": 0.5},
        # single-user text generation: every weight streamed for one token
        {"name": "decode_b1", "kind": "decode", "m": 1, "hidden": 4096, "ffn": 11008, "layers": 4, "dtype": "bf16",
         "sparsity": 0.7, "gated": False},
        # a few users on a narrow model whose widths fit no tile, with the fused gated half
        {"name": "decode_ragged_b5", "kind": "decode", "m": 5, "hidden": 3000, "ffn": 8008, "layers": 4,
         "dtype": "fp16", "sparsity": 0.5, "gated": True},
        # batched serving
        {"name": "decode_b16", "kind": "decode", "m": 16, "hidden": 4096, "ffn": 11008, "layers": 4, "dtype": "bf16",
         "sparsity": 0.7, "gated": False},
        # continuous batching of many users: between the decode and the prefill shapes
        {"name": "decode_b64", "kind": "decode", "m": 64, "hidden": 4096, "ffn": 11008, "layers": 4, "dtype": "bf16",
         "sparsity": 0.7, "gated": True},
        # batched serving of the sparse-quantized model
        {"name": "decode_int8_b16", "kind": "decode_q", "m": 16, "hidden": 4096, "ffn": 11008, "layers": 4, "bits": 8,
         "dtype": "bf16", "sparsity": 0.7},
        # single-user generation with 4-bit payloads
        {"name": "decode_int4_b1", "kind": "decode_q", "m": 1, "hidden": 4096, "ffn": 11008, "layers": 4, "bits": 4,
         "dtype": "bf16", "sparsity": 0.7},
        # a short prompt of no particular length
        {"name": "prefill_397", "kind": "prefill", "m": 397, "hidden": 4096, "ffn": 11008, "dtype": "fp16",
         "sparsity": 0.5},
        # a long prompt
        {"name": "prefill_2048", "kind": "prefill", "m": 2048, "hidden": 4096, "ffn": 11008, "dtype": "bf16",
         "sparsity": 0.7},
        # a long prompt of the sparse-quantized model
        {"name": "prefill_int8_2048", "kind": "prefill_q", "m": 2048, "hidden": 4096, "ffn": 11008, "dtype": "bf16",
         "sparsity": 0.7},
        # sparse fine-tuning: one layer's step on 2048 tokens
        {"name": "train_2048", "kind": "train", "m": 2048, "hidden": 4096, "ffn": 11008, "dtype": "bf16",
         "sparsity": 0.7},
        # bringing a checkpoint's layer into the packed format, and back
        {"name": "compress_layer", "kind": "compress", "hidden": 4096, "ffn": 11008, "dtype": "bf16",
         "sparsity": 0.7},
    ]


def _log_int(rng, lo, hi, step=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return min(hi // step * step, max(-(-lo // step) * step, int(round(v / step)) * step))


def _widths(rng, step):
    """The named layer half of the time, else widths of no particular divisibility (multiples of `step`)."""
    if rng.random() < 0.5:
        return 4096, 11008
    hidden = _log_int(rng, 768, 4096, step)
    return hidden, min(11008 // step * step, int(hidden * rng.uniform(2.0, 4.0)) // step * step)


def draw(rng):
    kind = rng.choice(["linear", "decode", "decode", "decode_q", "prefill", "prefill", "prefill_q", "train",
                       "compress"])
    dtype = rng.choice(["bf16", "fp16"])
    sparsity = round(rng.uniform(0.5, 0.8), 2)
    if kind == "linear":
        return {"kind": kind, "m": _log_int(rng, 1, 2048), "n": _log_int(rng, 512, 11008),
                "k": _log_int(rng, 512, 11008, 8), "dtype": dtype, "sparsity": sparsity}
    hidden, ffn = _widths(rng, 16 if kind in ("decode_q", "prefill_q") else 8)
    case = {"kind": kind, "hidden": hidden, "ffn": ffn, "dtype": dtype, "sparsity": sparsity}
    if kind == "decode":
        case.update(m=_log_int(rng, 1, 128), layers=rng.randint(1, 4), gated=rng.random() < 0.5)
    elif kind == "decode_q":
        bits = rng.choice([8, 8, 4])
        case.update(m=_log_int(rng, 1, 64 if bits == 8 else 16), layers=rng.randint(1, 4), bits=bits)
    elif kind in ("prefill", "prefill_q"):
        case.update(m=_log_int(rng, 129, 2048))
    elif kind == "train":
        case.update(m=_log_int(rng, 256, 1600, 8))
    return case


# ------------------------------------------------------------------------------------------------ inputs


def _layer_shapes(case):
    """(name, N, K, input) of the seven linears; linears with one input share its activations."""
    h, f = case["hidden"], case["ffn"]
    return [("q", h, h, "x"), ("k", h, h, "x"), ("v", h, h, "x"), ("o", h, h, "a"), ("gate", f, h, "y"),
            ("up", f, h, "y"), ("down", h, f, "z")]


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _weight(gen, n, k, case):
    """A dense weight and its keep-mask: the share `sparsity` of smallest magnitude is pruned, counted exactly."""
    w = torch.randn((n, k), generator=gen, device="cuda").mul_(STD)
    mask = torch.ones(n * k, dtype=torch.bool, device="cuda")
    mask[w.abs().view(-1).argsort()[: int(case["sparsity"] * n * k)]] = False
    return w.to(DTYPES[case["dtype"]]), mask.view(n, k)


def _codes(gen, n, k, case, top):
    """int8 codes of a pruned weight, one scale per row: absmax -> `top`."""
    w, mask = _weight(gen, n, k, case)
    w = w.float().mul_(mask)
    s = w.abs().amax(dim=1).clamp_(min=1e-6) / top
    return (w / s[:, None]).round_().to(torch.int8), mask, s


def _acts(gen, m, k, case):
    return torch.randn((m, k), generator=gen, device="cuda").to(DTYPES[case["dtype"]])


def _fp_layers(case, seed):
    """Per layer ({name: (dense W, mask)}, {input: X}), from the seed alone."""
    gen = _gen(seed)
    for _ in range(case.get("layers", 1)):
        ws = {name: _weight(gen, n, k, case) for name, n, k, _ in _layer_shapes(case)}
        xs = {}
        for _, n, k, src in _layer_shapes(case):
            if src not in xs:
                xs[src] = _acts(gen, case["m"], k, case)
        yield ws, xs


def _q_layers(case, seed):
    """Per layer ({name: (int8 codes, mask, scales)}, {input: X})."""
    gen = _gen(seed)
    top = 7 if case.get("bits") == 4 else 127
    for _ in range(case.get("layers", 1)):
        ws = {name: _codes(gen, n, k, case, top) for name, n, k, _ in _layer_shapes(case)}
        xs = {}
        for _, n, k, src in _layer_shapes(case):
            if src not in xs:
                xs[src] = _acts(gen, case["m"], k, case)
        yield ws, xs


def _graph(step):
    """`step` as a HIP graph (run once eagerly first, on the capture's side stream)."""
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    return graph


# ------------------------------------------------------------------------------------------------ the passes


def _new(case, m, n, dtype=None):
    return torch.empty((m, n), dtype=dtype or DTYPES[case["dtype"]], device="cuda")


def _fp_step(case, layer):
    """The seven linears of one layer on packed weights, into the layer's own output buffers."""
    w, x, y = layer["w"], layer["x"], layer["y"]
    spl.sparse_linear_group([x["x"]] * 3, [w["q"], w["k"], w["v"]], [y["q"], y["k"], y["v"]])
    spl.sparse_linear(x["a"], w["o"], out=y["o"])
    if case.get("gated", True):
        spl.sparse_linear_silu_mul(x["y"], w["gate"], w["up"], out=y["act"])
    else:
        spl.sparse_linear_group([x["y"]] * 2, [w["gate"], w["up"]], [y["gate"], y["up"]])
    spl.sparse_linear(x["z"], w["down"], out=y["down"])


def _fp_state(case, seed):
    layers = []
    for ws, xs in _fp_layers(case, seed):
        packed = {name: spl.pack_sparse(w, mask) for name, (w, mask) in ws.items()}
        names = ["q", "k", "v", "o"] + (["act"] if case.get("gated", True) else ["gate", "up"]) + ["down"]
        y = {n: _new(case, case["m"], case["ffn"] if n in ("act", "gate", "up") else case["hidden"]) for n in names}
        layers.append({"w": packed, "x": xs, "y": y})
    return layers


def _q_step(case, layer):
    w, sw, x, y, q = layer["w"], layer["sw"], layer["x"], layer["y"], layer["q"]
    for src in x:
        spl.quantize_rows_i8(x[src], out=q[src][0], scales=q[src][1])
    for names, src in ((("q", "k", "v"), "x"), (("o",), "a"), (("gate", "up"), "y"), (("down",), "z")):
        xq, sx = q[src]
        if case.get("bits") == 4:
            for n in names:
                spl.sparse_linear_int4(xq, sx, w[n], sw[n], out=y[n])
        elif len(names) > 1:
            spl.sparse_linear_int8_group([xq] * len(names), [sx] * len(names), [w[n] for n in names],
                                         [sw[n] for n in names], outs=[y[n] for n in names])
        else:
            spl.sparse_linear_int8(xq, sx, w[names[0]], sw[names[0]], out=y[names[0]])


def _q_state(case, seed):
    layers = []
    for ws, xs in _q_layers(case, seed):
        packed, scales = {}, {}
        for name, (codes, mask, s) in ws.items():
            packed[name], scales[name] = spl.pack_sparse(codes, mask), s
            if case.get("bits") == 4:
                packed[name] = spl.pack_int4(packed[name])
        m = case["m"]
        y = {name: _new(case, m, n, torch.float16) for name, n, _, _ in _layer_shapes(case)}
        q = {src: (_new(case, m, x.shape[1], torch.int8), torch.empty(m, device="cuda")) for src, x in xs.items()}
        layers.append({"w": packed, "sw": scales, "x": xs, "y": y, "q": q})
    return layers


def _train_state(case, seed):
    (ws, xs), = _fp_layers(case, seed)
    gen = _gen(seed + (1 << 40))
    w = {name: spl.pack_sparse(a, mask) for name, (a, mask) in ws.items()}
    dy = {name: _acts(gen, case["m"], n, case) for name, n, _, _ in _layer_shapes(case)}
    # the update writes a second copy of the stored values, so that a pass can be repeated
    new = {name: spl.SparseMatrix(p.bitmask, p.values.clone(), None, p.tile_offsets, p.rows, p.cols, p.nnz, p.layout)
           for name, p in w.items()}
    return {"w": w, "x": xs, "dy": dy, "new": new}


def _train_step(state):
    w, x, dy, new = state["w"], state["x"], state["dy"], state["new"]
    out = {"y": {}, "grad": {}, "values": {}, "dx": {}}
    for names, src in ((("q", "k", "v"), "x"), (("o",), "a"), (("gate", "up"), "y"), (("down",), "z")):
        xs, mats = [x[src]] * len(names), [w[n] for n in names]
        ys = spl.sparse_linear_group(xs, mats)
        grads = spl.sparse_weight_grad_group([dy[n] for n in names], xs, mats)
        for n, yv, g in zip(names, ys, grads):
            nnz = w[n].nnz
            out["y"][n], out["grad"][n] = yv, g[:nnz]
            out["dx"][n] = spl.sparse_input_grad(dy[n], w[n])
            new[n].values.copy_(w[n].values)
            spl.sparse_sgd_update(new[n], g, LR)
            out["values"][n] = new[n].values[:nnz]
    return out


def _compress(state):
    out = {}
    for name, (w, prune) in state.items():
        mask = spl.magnitude_mask(w, prune)
        p = spl.pack_sparse(w, mask)
        out[name] = [mask, p.bitmask, p.values[: p.nnz], p.tile_offsets, spl.unpack(p)]
    return out


def prepare(case, seed):
    kind = case["kind"]
    if kind == "linear":
        gen = _gen(seed)
        w, mask = _weight(gen, case["n"], case["k"], case)
        return case, (_acts(gen, case["m"], case["k"], case), spl.pack_sparse(w, mask))
    if kind == "decode":
        layers = _fp_state(case, seed)
        return case, (layers, _graph(lambda: [_fp_step(case, layer) for layer in layers]))
    if kind == "decode_q":
        layers = _q_state(case, seed)
        return case, (layers, _graph(lambda: [_q_step(case, layer) for layer in layers]))
    if kind == "prefill":
        return case, _fp_state(case, seed)[0]
    if kind == "prefill_q":
        return case, _q_state(case, seed)[0]
    if kind == "train":
        return case, _train_state(case, seed)
    gen, state = _gen(seed), {}
    for name, n, k, _ in _layer_shapes(case):
        w = torch.randn((n, k), generator=gen, device="cuda").mul_(STD).to(DTYPES[case["dtype"]])
        state[name] = (w, int(case["sparsity"] * n * k))
    return case, state


def run(state):
    case, s = state
    kind = case["kind"]
    if kind == "linear":
        return spl.sparse_linear(*s)
    if kind in ("decode", "decode_q"):
        layers, graph = s
        graph.replay()
        return [layer["y"] for layer in layers]
    if kind == "prefill":
        _fp_step(case, s)
        return s["y"]
    if kind == "prefill_q":
        _q_step(case, s)
        return {"y": s["y"], "scales": {src: sx for src, (_, sx) in s["q"].items()}}
    return _train_step(s) if kind == "train" else _compress(s)


# ------------------------------------------------------------------------------------------------ what it takes


def work(case):
    """Bytes: each packed weight, activation and output once.  Operations: two per kept entry and batch row."""
    kind, keep = case["kind"], 1.0 - case["sparsity"]
    payload = 0.5 if case.get("bits") == 4 else 1.0 if kind in ("decode_q", "prefill_q") else 2.0

    def packed(n, k):
        tiles = -(-n // 16) * -(-k // 32)
        return keep * n * k * payload + tiles * 68

    if kind == "linear":
        m, n, k = case["m"], case["n"], case["k"]
        return {"bytes": packed(n, k) + 2 * m * (n + k), "flops": 2 * m * n * k * keep}
    shapes = _layer_shapes(case)
    if kind == "compress":   # the matrix and its mask, the packed form, the matrix again
        return {"bytes": sum(2 * n * k + n * k + 2 * packed(n, k) + 2 * n * k for _, n, k, _ in shapes), "flops": 0}
    m = case["m"]
    weights = sum(packed(n, k) for _, n, k, _ in shapes)
    kept = sum(n * k * keep for _, n, k, _ in shapes)
    ins = sum({src: 2 * m * k for _, _, k, src in shapes}.values())
    outs = sum(2 * m * n for _, n, _, _ in shapes)
    if kind == "train":      # forward, weight gradient and update, input gradient
        dx = sum(2 * m * k for _, _, k, _ in shapes)
        return {"bytes": weights + ins + 2 * outs + 4 * kept + dx, "flops": 3 * 2 * m * kept}
    if kind in ("decode", "prefill") and case.get("gated", True):
        outs -= 2 * m * case["ffn"]
    return {"bytes": case.get("layers", 1) * (weights + ins + outs), "flops": case.get("layers", 1) * 2 * m * kept}


def tolerance(case):
    """fp16 / bf16 results are fp32 sums rounded once: about four times what that rounding gives against 64-bit
    sums.  The quantized paths are exact integer sums with a fixed epilogue, and packing moves bits."""
    if case["kind"] in ("decode_q", "prefill_q", "compress"):
        return "exact"
    return {"rel": 7e-3, "max": 3e-2} if case["dtype"] == "bf16" else {"rel": 1e-3, "max": 4e-3}


def _dense(w, mask):
    return w.double().mul_(mask)


def _tile_order(dense, mask):
    """The kept entries of [N][K] in the packed order: 16 x 32 tiles row-major; inside one by 8-column group, then
    row, then column."""
    n, k = dense.shape
    b, s = -(-n // 16), -(-k // 32)

    def tiled(t):
        t = torch.nn.functional.pad(t, (0, 32 * s - k, 0, 16 * b - n))
        return t.view(b, 16, s, 4, 8).permute(0, 2, 3, 1, 4).reshape(-1)

    return tiled(dense)[tiled(mask.to(torch.uint8)).bool()]


def exact(case, seed):
    kind = case["kind"]
    if kind == "compress":
        return None
    if kind == "linear":
        gen = _gen(seed)
        w = _dense(*_weight(gen, case["n"], case["k"], case))
        return _acts(gen, case["m"], case["k"], case).double() @ w.t().contiguous()
    if kind in ("decode_q", "prefill_q"):
        outs = []
        for ws, xs in _q_layers(case, seed):
            quant = {}
            for src, x in xs.items():
                sx = (x.float().abs().amax(dim=1) / 127.0)
                sx = torch.where(sx == 0, torch.ones_like(sx), sx)
                quant[src] = ((x.float() / sx[:, None]).round().clamp(-127, 127).double(), sx.double())
            y = {}
            for name, _, _, src in _layer_shapes(case):
                codes, mask, sw = ws[name]
                xq, sx = quant[src]
                y[name] = (xq @ _dense(codes, mask).t().contiguous()) * sx[:, None] * sw.double()[None, :]
            outs.append((y, {src: q[1] for src, q in quant.items()}))
        return [y for y, _ in outs] if kind == "decode_q" else {"y": outs[0][0], "scales": outs[0][1]}
    if kind == "train":
        (ws, xs), = _fp_layers(case, seed)
        gen = _gen(seed + (1 << 40))
        out = {"y": {}, "grad": {}, "values": {}, "dx": {}}
        dys = {name: _acts(gen, case["m"], n, case) for name, n, _, _ in _layer_shapes(case)}
        for name, _, _, src in _layer_shapes(case):
            w, mask = ws[name]
            d, x, dy = _dense(w, mask), xs[src].double(), dys[name].double()
            out["y"][name] = x @ d.t().contiguous()
            out["dx"][name] = dy @ d
            grad = dy.t().contiguous() @ x
            out["grad"][name] = _tile_order(grad, mask)
            out["values"][name] = _tile_order(w.double() - LR * grad, mask)
        return out
    outs = []
    for ws, xs in _fp_layers(case, seed):
        y = {}
        for name, _, _, src in _layer_shapes(case):
            y[name] = xs[src].double() @ _dense(*ws[name]).t().contiguous()
        if case.get("gated", True):
            g = y.pop("gate")
            y["act"] = g * torch.sigmoid(g) * y.pop("up")
        outs.append(y)
    return outs if kind == "decode" else outs[0]
