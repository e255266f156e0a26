"""Performance cases: the calls a decode engine makes through paper_2609_16338_amd.

Four kinds of case:

* ``gemv``  -- one call of ``api.gemv`` on one packed matrix (any of the three formats).
* ``layer`` -- the launches of one decoder layer in the order its data flow forces:
  q/k/v in one batched launch, the output projection, gate/up in one batched launch,
  the down projection.  With int8 activations every stage first quantises its bf16
  activations (``api.quantize_activations``), as a decode loop does.
* ``set``   -- every GEMV of several layers in one batched launch per row length, the
  way the benchmark's step issues them; rows longer than a batch-1 tile are stored as
  column blocks whose partial outputs ``api.add_partials`` sums.
* ``pack``  -- packing a matrix on the GPU into a buffer of the caller
  (``api.bitcos_pack_device_noalloc``), as at model load.

Sizes are those of ``workloads.py`` (BitNet-2B-like, Qwen3-8B-like and Qwen3-32B-like
layers, the 256 x 1024 instance, the 8192 x 8192 sweep matrix).  Weights are ternary with
the layer sets' zero densities, scales fp16, activations N(0, 1) in bf16 (or int8 from
the quantiser, or uniform int8 for the 256 x 1024 instance).
"""

from __future__ import annotations

import math

import torch

from paper_2609_16338_amd import api

FORMATS = {"bitcos": api.FMT_BITCOS, "trit5": api.FMT_TRIT5, "bit2": api.FMT_BIT2}
KSPLIT_MAX = 16384  # rows longer than this are stored as column blocks in a ``set``
SPLIT_BLOCK = 5120  # ... of this many columns

# (hidden, k/v rows, FFN, scale group, zero density range, scale range) of workloads.py's layer sets
MODELS = {
    "bitnet2b": (2560, 640, 6912, 0, (0.42, 0.42), (0.01, 0.1)),
    "qwen3_8b": (4096, 1024, 12288, 128, (0.467, 0.467), (0.005, 0.05)),
    "qwen3_32b": (5120, 1024, 25600, 128, (0.30, 0.60), (0.005, 0.05)),
}


def _gemv(name, fmt, n, k, m, act, group, z=(0.42, 0.42), scales=(0.01, 0.1), raw=False):
    c = {"kind": "gemv", "fmt": fmt, "n": n, "k": k, "m": m, "act": act, "group": group,
         "z_lo": z[0], "z_hi": z[1], "s_lo": scales[0], "s_hi": scales[1], "raw": raw}
    return {"name": name, **c} if name else c


def _layers(name, kind, dims, layers, m, act):
    h, kv, ffn, group, z, s = dims
    c = {"kind": kind, "h": h, "kv": kv, "ffn": ffn, "group": group, "z_lo": z[0], "z_hi": z[1], "s_lo": s[0], "s_hi": s[1],
         "layers": layers, "m": m, "act": act}
    return {"name": name, **c} if name else c


def _pack(name, n, k, group, z):
    c = {"kind": "pack", "n": n, "k": k, "group": group, "z_lo": z[0], "z_hi": z[1], "s_lo": 0.005, "s_hi": 0.05}
    return {"name": name, **c} if name else c


def listed():
    return [
        # The smallest instance of workloads.py: one launch whose latency is all there is.
        _gemv("single_256x1024_i8", "bitcos", 256, 1024, 1, "int8", 128, (0.5, 0.5)),
        # One projection of a small model called on its own (tensor-scale weights).
        _gemv("bitnet2b_o_bf16", "bitcos", 2560, 2560, 1, "bf16", 0),
        # One decoder layer of a mid-size model at batch 1, int8 activations: four dependent stages.
        _layers("qwen3_8b_layer_i8", "layer", MODELS["qwen3_8b"], 1, 1, "int8"),
        # The same layer for four sequences decoded together, bf16 activations.
        _layers("qwen3_8b_layer_m4_bf16", "layer", MODELS["qwen3_8b"], 1, 4, "bf16"),
        # A down projection whose rows are longer than a batch-1 tile, called directly.
        _gemv("qwen3_32b_down_bf16", "bitcos", 5120, 25600, 1, "bf16", 128, (0.30, 0.60), (0.005, 0.05)),
        # Batch 16 on the widest matrix: the up projection of the largest layer set.
        _gemv("qwen3_32b_up_m16_bf16", "bitcos", 25600, 5120, 16, "bf16", 128, (0.30, 0.60), (0.005, 0.05)),
        # Benchmark-style steps: whole layer sets at batch 1, one launch per row length.
        _layers("bitnet2b_set_bf16", "set", MODELS["bitnet2b"], 12, 1, "bf16"),
        _layers("qwen3_8b_set_i8", "set", MODELS["qwen3_8b"], 8, 1, "int8"),
        _layers("qwen3_32b_set_bf16", "set", MODELS["qwen3_32b"], 4, 1, "bf16"),
        # The fixed-rate formats on the sweep matrix, one with each activation type.
        _gemv("trit5_8192_bf16", "trit5", 8192, 8192, 1, "bf16", 128),
        _gemv("bit2_8192_i8", "bit2", 8192, 8192, 1, "int8", 128),
        # Encode: packing a projection on the GPU at load time.
        _pack("pack_5120x5120", 5120, 5120, 128, (0.30, 0.60)),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["gemv", "gemv", "gemv", "rows", "rows", "layer", "set", "fixed", "pack"])
    z = round(rng.uniform(0.30, 0.60), 3)
    act = rng.choice(["bf16", "int8"])
    if kind in ("gemv", "rows"):
        group = rng.choice([128, 128, 0])
        k = 128 * _logint(rng, 4, 200) if group or kind == "rows" else 32 * _logint(rng, 16, 512)
        n = _logint(rng, 128, 25600)
        m = 1 if kind == "gemv" else rng.randint(2, 16)
        return _gemv(None, "bitcos", n, k, m, act, group, (z, z), raw=act == "int8" and rng.random() < 0.25)
    if kind == "fixed":
        return _gemv(None, rng.choice(["trit5", "bit2"]), _logint(rng, 512, 8192), 128 * _logint(rng, 8, 64), 1, act, 128,
                     (z, z))
    if kind in ("layer", "set"):
        h, ffn = 128 * _logint(rng, 8, 40), 128 * _logint(rng, 24, 200)
        if kind == "set" and ffn > KSPLIT_MAX:
            ffn = SPLIT_BLOCK * round(ffn / SPLIT_BLOCK)
        kv, group = 128 * rng.randint(2, 8), rng.choice([128, 128, 0])
        dims = (h, kv, ffn, group, (z, z), (0.005, 0.05))
        if kind == "layer":
            return _layers(None, "layer", dims, 1, rng.choice([1, 1, rng.randint(2, 16)]), act)
        most = max(2, min(20, 1_500_000_000 // (2 * h * h + 2 * kv * h + 3 * h * ffn)))
        return _layers(None, "set", dims, rng.randint(2, most), 1, act)
    return _pack(None, _logint(rng, 256, 8192), 128 * _logint(rng, 4, 64), rng.choice([128, 0]), (z, z))


# ---------------------------------------------------------------------------
# Inputs: plain torch, from the seed alone
# ---------------------------------------------------------------------------


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(0x5EED + 7919 * int(seed))
    return g


def _weights(g, n, k, z_lo, z_hi):
    """Ternary int8 [n][k] with a zero density per row drawn from [z_lo, z_hi], and balanced signs."""
    z = z_lo + (z_hi - z_lo) * torch.rand((n, 1), device="cuda", generator=g)
    u = torch.rand((n, k), device="cuda", generator=g)
    return (u >= z).to(torch.int8) - 2 * (u >= z + (1.0 - z) / 2).to(torch.int8)


def _scales(g, n, k, group, lo, hi):
    shape = (n, k // 128) if group == 128 else (1, 1)
    return (lo + (hi - lo) * torch.rand(shape, device="cuda", generator=g)).to(torch.float16)


def _acts(g, m, k):
    return torch.randn((m, k), device="cuda", generator=g).to(torch.bfloat16)


def _matrices(case):
    """The seven matrices of one layer: (name, n, k)."""
    h, kv, ffn = case["h"], case["kv"], case["ffn"]
    return [("q", h, h), ("k", kv, h), ("v", kv, h), ("o", h, h), ("gate", ffn, h), ("up", ffn, h), ("down", h, ffn)]


STAGES = [("q", "k", "v"), ("o",), ("gate", "up"), ("down",)]


def _layer_inputs(case, g):
    """Yields (layer, matrix name, W, scales, column block or None); draws in a fixed order."""
    for layer in range(case["layers"]):
        for name, n, k in _matrices(case):
            yield (layer, name, _weights(g, n, k, case["z_lo"], case["z_hi"]),
                   _scales(g, n, k, case["group"], case["s_lo"], case["s_hi"]))


def _layer_acts(case, g):
    """bf16 activations [m][k] of the four stages (shared by every layer of a ``set``)."""
    h, ffn = case["h"], case["ffn"]
    return [_acts(g, case["m"], h), _acts(g, case["m"], h), _acts(g, case["m"], h), _acts(g, case["m"], ffn)]


def _blocks(k):
    return [(0, k)] if k <= KSPLIT_MAX else [(k0, SPLIT_BLOCK) for k0 in range(0, k, SPLIT_BLOCK)]


# ---------------------------------------------------------------------------
# prepare / run
# ---------------------------------------------------------------------------


def prepare(case, seed):
    g = _generator(seed)
    if case["kind"] == "gemv":
        return _prepare_gemv(case, g)
    if case["kind"] == "pack":
        w = _weights(g, case["n"], case["k"], case["z_lo"], case["z_hi"])
        sc = _scales(g, case["n"], case["k"], case["group"], case["s_lo"], case["s_hi"])
        # Room for the blob at any density: both bit streams full, an offset per row, scales, padding.
        dst = torch.zeros(2 * (w.numel() // 8) + 4 * w.shape[0] + 2 * sc.numel() + 2048, dtype=torch.uint8, device="cuda")
        return {"kind": "pack", "w": w, "scales": sc.reshape(-1), "group": case["group"], "dst": dst}
    return _prepare_layer(case, g) if case["kind"] == "layer" else _prepare_set(case, g)


def _gemv_inputs(case, g):
    w = _weights(g, case["n"], case["k"], case["z_lo"], case["z_hi"])
    sc = _scales(g, case["n"], case["k"], case["group"], case["s_lo"], case["s_hi"])
    if case["act"] == "int8":
        x = torch.randint(-127, 128, (case["m"], case["k"]), device="cuda", generator=g, dtype=torch.int8)
    else:
        x = _acts(g, case["m"], case["k"])
    return w, sc, x


def _prepare_gemv(case, g):
    w, sc, x = _gemv_inputs(case, g)
    if case["fmt"] == "bitcos":
        layout, blob = api.bitcos_pack_device(w, sc.reshape(-1), case["group"])
    else:
        layout, host = api.plan_and_pack(FORMATS[case["fmt"]], w.cpu().numpy(), sc.reshape(-1).cpu().numpy(), case["group"])
        blob = torch.from_numpy(host).cuda()
    y = torch.empty((case["m"], case["n"]), dtype=torch.int32 if case["raw"] else torch.float32, device="cuda")
    return {"kind": "gemv", "layout": layout, "blob": blob, "x": x, "y": y,
            "mode": api.Y_I32_RAW if case["raw"] else api.Y_F32}


def _prepare_layer(case, g):
    m, group, act = case["m"], case["group"], case["act"]
    packed = {name: api.bitcos_pack_device(w, sc.reshape(-1), group) for _, name, w, sc in _layer_inputs(case, g)}
    shape = {name: n for name, n, _ in _matrices(case)}
    stages = []
    for x, names in zip(_layer_acts(case, g), STAGES):
        k = x.shape[1]
        q = a = None
        if act == "int8":
            q = torch.empty((m, k), dtype=torch.int8, device="cuda")
            a = torch.empty((m, k // 128), dtype=torch.float32, device="cuda")
        ys = [torch.empty((m, shape[nm]), dtype=torch.float32, device="cuda") for nm in names]
        batch = None
        if len(names) > 1:
            one = x if q is None else q
            batch = api.Batch([packed[nm][0] for nm in names], [packed[nm][1] for nm in names], [one] * len(names), ys,
                              None if a is None else [a] * len(names))
        stages.append({"x": x, "q": q, "a": a, "ys": ys, "batch": batch, "packed": packed[names[0]]})
    return {"kind": "layer", "stages": stages}


def _prepare_set(case, g):
    m, group, act = case["m"], case["group"], case["act"]
    shape = {name: (n, k) for name, n, k in _matrices(case)}
    names = [name for name, _, _ in _matrices(case)]
    ys = {}
    for name in names:  # one stacked output per matrix of the layer
        ys[name] = torch.empty((case["layers"], m, shape[name][0]), dtype=torch.float32, device="cuda")
    parts = {}
    for name in names:
        nb = len(_blocks(shape[name][1]))
        if nb > 1:
            parts[name] = torch.empty((nb - 1, *ys[name].shape), dtype=torch.float32, device="cuda")
    entries = []
    for layer, name, w, sc in _layer_inputs(case, g):
        for c, (k0, kb) in enumerate(_blocks(w.shape[1])):
            wb = w[:, k0:k0 + kb].contiguous()
            sb = sc[:, k0 // 128:(k0 + kb) // 128].contiguous() if group == 128 else sc
            layout, blob = api.bitcos_pack_device(wb, sb.reshape(-1), group)
            entries.append((name, c, k0, kb, layout, blob, ys[name][layer] if c == 0 else parts[name][c - 1, layer]))
        del w
    stage_of = {name: i for i, st in enumerate(STAGES) for name in st}
    xs = []
    for x in _layer_acts(case, g):
        if act == "int8":
            q = torch.empty(x.shape, dtype=torch.int8, device="cuda")
            a = torch.empty((m, x.shape[1] // 128), dtype=torch.float32, device="cuda")
            api.quantize_activations(x, q, a)
            xs.append((q, a))
        else:
            xs.append((x, None))
    cut = {}

    def x_of(name, k0, kb):
        i = stage_of[name]
        if (i, k0) not in cut:
            x, a = xs[i]
            cut[(i, k0)] = (x[:, k0:k0 + kb].contiguous(),
                            None if a is None else a[:, k0 // 128:(k0 + kb) // 128].contiguous())
        return cut[(i, k0)]

    batches = []
    for k in sorted({e[3] for e in entries}):
        es = [e for e in entries if e[3] == k]
        xa = [x_of(e[0], e[2], e[3]) for e in es]
        batches.append(api.Batch([e[4] for e in es], [e[5] for e in es], [x for x, _ in xa], [e[6] for e in es],
                                 None if act != "int8" else [a for _, a in xa]))
    torch.cuda.synchronize()
    return {"kind": "set", "batches": batches, "ys": [ys[nm] for nm in names],
            "sums": [(ys[nm], parts[nm]) for nm in names if nm in parts]}


def run(state):
    if state["kind"] == "gemv":
        return api.gemv(state["layout"], state["blob"], state["x"], state["y"], y_mode=state["mode"])
    if state["kind"] == "pack":
        layout = api.bitcos_pack_device_noalloc(state["w"], state["scales"], state["dst"], state["group"])
        return {"blob": state["dst"], "nnz": int(layout.nnz)}
    if state["kind"] == "layer":
        out = []
        for st in state["stages"]:
            if st["q"] is not None:
                api.quantize_activations(st["x"], st["q"], st["a"])
            if st["batch"] is not None:
                st["batch"].run()
            else:
                layout, blob = st["packed"]
                api.gemv(layout, blob, st["x"] if st["q"] is None else st["q"], st["ys"][0], xscale=st["a"])
            out += st["ys"]
        return out
    for b in state["batches"]:
        b.run()
    for y, parts in state["sums"]:
        api.add_partials(y, parts)
    return state["ys"]


# ---------------------------------------------------------------------------
# work / tolerance / exact
# ---------------------------------------------------------------------------


def _blob_bytes(fmt, n, k, group, z):
    bits = {"bitcos": 2.0 - z, "trit5": 26 * 8 / 128, "bit2": 2.0}[fmt]
    return n * k * bits / 8 + (2 * n * (k // 128) if group == 128 else 2)


def work(case):
    kind = case["kind"]
    if kind == "gemv":
        n, k, m = case["n"], case["k"], case["m"]
        z = (case["z_lo"] + case["z_hi"]) / 2
        return {"bytes": _blob_bytes(case["fmt"], n, k, case["group"], z) + m * k * (1 if case["act"] == "int8" else 2) + 4 * m * n,
                "flops": 2.0 * m * n * k}
    if kind == "pack":
        n, k = case["n"], case["k"]
        z = (case["z_lo"] + case["z_hi"]) / 2
        ns = n * (k // 128) if case["group"] == 128 else 1
        return {"bytes": n * k + 2 * ns + _blob_bytes("bitcos", n, k, case["group"], z) + 4 * n, "flops": 0.0}
    h, ffn, m = case["h"], case["ffn"], case["m"]
    by = fl = 0.0
    for _, n, k in _matrices(case):
        by += case["layers"] * (_blob_bytes("bitcos", n, k, case["group"], (case["z_lo"] + case["z_hi"]) / 2) + 4 * m * n)
        fl += case["layers"] * 2.0 * m * n * k
    x_elem = 2 if kind == "layer" or case["act"] == "bf16" else 1
    return {"bytes": by + m * (3 * h + ffn) * x_elem, "flops": fl}


def tolerance(case):
    if case["kind"] == "pack" or case.get("raw"):
        return "exact"
    # fp32 sums of exact products: 3e-8 to 2.6e-7 from 64 bits as measured (the longest rows the most).
    return {"rel": 1e-6, "max": 1e-5}


def _quantized(x):
    """The quantiser's rule in plain torch (on the host: IEEE fp32 division): float64 q and a."""
    m, k = x.shape
    v = x.float().cpu().reshape(m, k // 128, 128)
    amax = v.abs().amax(dim=2, keepdim=True)
    a = torch.where(amax == 0, torch.ones_like(amax), amax / 127.0)
    q = torch.clamp(torch.round(v / a), -127, 127)
    return q.reshape(m, k).double().cuda(), a.reshape(m, k // 128).double().cuda()


def _dense(w, sc, group, x, a=None):
    """y[m][n] = sum_g S[n, g] a[m, g] sum_k W[n, k] x[m, k] in float64, a few thousand rows at a time."""
    n, k = w.shape
    x = x.double()
    if a is not None:
        x = (x.reshape(x.shape[0], k // 128, 128) * a.unsqueeze(2)).reshape(x.shape[0], k)
    y = torch.empty((x.shape[0], n), dtype=torch.float64, device=w.device)
    for r in range(0, n, 2048):
        wr = w[r:r + 2048].double()
        s = sc[r:r + 2048].double() if group == 128 else sc.double()
        if group == 128:
            wr = (wr.reshape(wr.shape[0], k // 128, 128) * s.unsqueeze(2)).reshape(wr.shape[0], k)
        else:
            wr = wr * s
        y[:, r:r + 2048] = torch.stack([wr @ row for row in x])
    return y


def exact(case, seed):
    g = _generator(seed)
    if case["kind"] == "pack":
        return None
    if case["kind"] == "gemv":
        w, sc, x = _gemv_inputs(case, g)
        if case["raw"]:
            return _dense(w, torch.ones((1, 1), device="cuda"), 0, x)
        return _dense(w, sc, case["group"], x)
    names = [name for name, _, _ in _matrices(case)]
    acts_at = {name: i for i, st in enumerate(STAGES) for name in st}
    # The activations are drawn after every weight: a first pass over the weights finds them.
    for _ in _layer_inputs(case, g):
        pass
    acts = [_quantized(x) if case["act"] == "int8" else (x.double(), None) for x in _layer_acts(case, g)]
    out = {name: [] for name in names}
    for _, name, w, sc in _layer_inputs(case, _generator(seed)):
        x, a = acts[acts_at[name]]
        out[name].append(_dense(w, sc, case["group"], x, a))
    if case["kind"] == "layer":
        return [out[name][0] for name in names]
    return [torch.stack(out[name]) for name in names]
