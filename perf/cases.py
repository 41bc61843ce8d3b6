"""Performance cases: the work that a program built on this package has it do.

Six kinds of pass, each through the package's public calls on buffers that such a program keeps:

  one      a single linear layer: (rotate and) quantise the activation, multiply
  decode   the linear layers of consecutive decoder layers for M new tokens: q|k|v, o, gate|up and down per
           layer, every layer with weights of its own, the down input behind its online rotation
  kv       one new token of one sequence: append its key and value to the 4-bit cache, attend (per layer)
  kvbatch  one new token for each of several sequences of different lengths (per layer)
  prompt   the keys and values of a whole prompt appended to the 4-bit cache (per layer)
  export   the offline packing of a decoder layer's weight matrices

Shapes are those of the repository's configurations (LLaMA-3.2-1B-, LLaMA-2-7B- and LLaMA-3-8B-shaped layers), inputs
are synthetic with the distributions of rcp_synth.py, drawn on the GPU.
"""
import math

import torch

import paper_2502_15779_amd as rcp

DTYPES = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}
ACT_CLIP, KV_CLIP = 0.9, 0.95   # clipping ratios of the paper's quantisation table
# a stand-in for the 3-bit format's normal-float table: eight ascending values with one 0, ends at -1 and 1
GRID8 = (-1.0, -0.61, -0.29, 0.0, 0.18, 0.39, 0.64, 1.0)


# ---- the cases ------------------------------------------------------------------------------------
def listed():
    return [
        # the smallest call: one small matrix whose input is rotated, quantised and multiplied in one launch; latency only
        {"name": "one_256x512", "kind": "one", "n": 256, "k": 512, "m": 1, "fmt": "w2", "fused": True, "rot": "wht",
         "dtype": "f16"},
        # a small model's decode step (all 16 layers): short matrices, bf16 activations, Hadamard across the heads in
        # front of the out-projection, an 8192-point Hadamard in front of the down projection
        {"name": "decode_1b", "kind": "decode", "hidden": 2048, "kvdim": 512, "ffn": 8192, "wht": 8192, "heads": 32,
         "layers": 16, "m": 1, "fmt": "w2", "dtype": "bf16"},
        # the headline workload: one token through the 32 layers of the 7B shape
        {"name": "decode_7b", "kind": "decode", "hidden": 4096, "kvdim": 4096, "ffn": 11008, "wht": 64, "heads": 0,
         "layers": 32, "m": 1, "fmt": "w2", "dtype": "f16"},
        # the deployed weight setting (one look-up table per 128 input channels), grouped-query shapes
        {"name": "decode_8b_g128", "kind": "decode", "hidden": 4096, "kvdim": 1024, "ffn": 14336, "wht": 512, "heads": 0,
         "layers": 8, "m": 1, "fmt": "g128", "dtype": "bf16"},
        # 3-bit weights
        {"name": "decode_7b_w3", "kind": "decode", "hidden": 4096, "kvdim": 4096, "ffn": 11008, "wht": 64, "heads": 0,
         "layers": 8, "m": 1, "fmt": "w3", "dtype": "f16"},
        # weights only: 16-bit activations, no activation quantiser
        {"name": "decode_7b_w2a16", "kind": "decode", "hidden": 4096, "kvdim": 4096, "ffn": 11008, "wht": 64, "heads": 0,
         "layers": 8, "m": 1, "fmt": "w2a16", "dtype": "f16"},
        # a full small batch
        {"name": "batch16_7b", "kind": "decode", "hidden": 4096, "kvdim": 4096, "ffn": 11008, "wht": 64, "heads": 0,
         "layers": 8, "m": 16, "fmt": "w2", "dtype": "f16"},
        # a ragged small batch in the deployed weight setting
        {"name": "batch6_8b_g128", "kind": "decode", "hidden": 4096, "kvdim": 1024, "ffn": 14336, "wht": 512, "heads": 0,
         "layers": 8, "m": 6, "fmt": "g128", "dtype": "bf16"},
        # attention part of a decode step: 32 heads, a context just past 4000 tokens
        {"name": "kv_step_7b", "kind": "kv", "hq": 32, "hkv": 32, "s": 4001, "layers": 8, "dtype": "f16"},
        # the same for sixteen sequences of different lengths with grouped-query heads
        {"name": "kv_batch16_8b", "kind": "kvbatch", "b": 16, "hq": 32, "hkv": 8, "smin": 300, "smax": 6000, "layers": 4,
         "dtype": "bf16"},
        # a prompt enters the cache
        {"name": "kv_prompt_8b", "kind": "prompt", "n": 2000, "h": 8, "s": 4096, "layers": 8, "dtype": "bf16"},
        # export of one decoder layer
        {"name": "export_7b", "kind": "export", "hidden": 4096, "kvdim": 4096, "ffn": 11008, "fmt": "w2", "dtype": "f16"},
    ]


def _log(rng, lo, hi, step=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return min(hi, max(lo, int(round(v / step)) * step))


def draw(rng):
    kind = rng.choice(["one", "one", "decode", "decode", "decode", "kv", "kvbatch", "prompt", "export"])
    dtype = rng.choice(["f16", "bf16"])
    if kind == "one":
        fmt = rng.choice(["w2", "w2", "w2", "g128", "w3", "w2a16"])
        m = 1 if fmt in ("w3", "w2a16") or rng.random() < 0.5 else rng.randint(2, 16)
        k = _log(rng, 256, 16384, 128 if fmt == "g128" else 32)
        rot = "none"
        if fmt == "w2" and m == 1 and rng.random() < 0.3:
            k, rot = 1 << rng.randint(8, 11), "wht"
        n = _log(rng, 256, 131072, 4)
        while n * k > 131072 * 4096:
            n = _log(rng, 256, 131072, 4)
        return {"kind": "one", "n": n, "k": k, "m": m, "fmt": fmt, "fused": bool(rot == "wht" or rng.random() < 0.6),
                "rot": rot, "dtype": dtype}
    if kind in ("decode", "export"):
        fmt = rng.choice(["w2", "w2", "g128", "g128", "w3", "w2a16"] if kind == "decode" else ["w2", "g128", "w3"])
        hidden = 128 * rng.randint(8, 40)
        kvdim = hidden if rng.random() < 0.5 else 128 * max(1, hidden // 512)
        wht = rng.choice([64, 128, 512])
        ffn = wht * int(rng.uniform(2.5, 3.6) * hidden / wht)
        ffn = min(ffn, 16384)  # beyond that the fused calls want scratch
        while ffn % 128:
            ffn += wht
        if kind == "export":
            return {"kind": kind, "hidden": hidden, "kvdim": kvdim, "ffn": ffn, "fmt": fmt,
                    "dtype": rng.choice(list(DTYPES) if hidden <= 3072 else ["f16", "bf16"])}
        m = 1 if fmt in ("w3", "w2a16") or rng.random() < 0.5 else rng.randint(2, 16)
        heads = hidden // 128 if fmt == "w2" and hidden & (hidden - 1) == 0 and rng.random() < 0.5 else 0
        return {"kind": kind, "hidden": hidden, "kvdim": kvdim, "ffn": ffn, "wht": wht, "heads": heads,
                "layers": rng.randint(2, 8), "m": m, "fmt": fmt, "dtype": dtype}
    hkv = rng.choice([4, 8, 16, 32])
    hq = hkv * rng.choice([r for r in (1, 2, 4, 8) if 8 <= hkv * r <= 64])
    if kind == "kv":
        s = _log(rng, 100, 70000)
        while s * hq > 70000 * 32:
            s = _log(rng, 100, 70000)
        return {"kind": kind, "hq": hq, "hkv": hkv, "s": s, "layers": max(1, min(8, 600000 // (s * hkv))), "dtype": dtype}
    if kind == "kvbatch":
        b = rng.randint(2, 16)
        smax = _log(rng, 200, max(400, 2_500_000 // (b * hq)))
        return {"kind": kind, "b": b, "hq": hq, "hkv": hkv, "smin": _log(rng, 16, smax), "smax": smax,
                "layers": rng.randint(1, 4), "dtype": dtype}
    n = _log(rng, 16, 8192)
    return {"kind": kind, "n": n, "h": hkv, "s": n + rng.randint(0, 2000), "layers": rng.randint(1, 8), "dtype": dtype}


# ---- inputs ---------------------------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _act(g, shape, dtype):
    """Activations: N(0, 1), 1 % of the entries twenty times as large."""
    x = torch.randn(shape, generator=g, device="cuda")
    x = torch.where(torch.rand(shape, generator=g, device="cuda") < 0.01, 20 * x, x)
    return x.to(dtype)


def _raw_weights(g, n, k, fmt, dtype):
    """A weight matrix N(0, 0.02^2) and its learnt clip range and partition (per row or per row and group)."""
    w = (torch.randn((n, k), generator=g, device="cuda") * 0.02).to(dtype)
    unit = (n, k // rcp.GROUP) if fmt == "g128" else (n,)
    spread = 1 + 0.1 * torch.rand((2,) + unit, generator=g, device="cuda")
    lo, hi = (-0.0465 * spread[0]).contiguous(), (0.0465 * spread[1]).contiguous()
    if fmt == "w3":
        return w, lo, hi, torch.sigmoid(0.5 * torch.randn(unit, generator=g, device="cuda"))
    return w, lo, hi, torch.softmax(torch.randn(unit + (3,), generator=g, device="cuda"), dim=-1).contiguous()


def _pack(raw, fmt, packed=None, codebook=None):
    if fmt == "g128":
        return rcp.pack_weights_grouped(*raw, packed_out=packed, codebook_out=codebook)
    if fmt == "w3":
        return rcp.pack_weights_w3(*raw, GRID8, packed_out=packed, codebook_out=codebook)
    return rcp.pack_weights(*raw, packed_out=packed, codebook_out=codebook)


def _orthogonal(g, m):
    q, r = torch.linalg.qr(torch.randn((m, m), generator=g, device="cuda").double().cpu())
    return (q * torch.sign(torch.diagonal(r))).float().contiguous().cuda()


def _head_vectors(g, n, heads, dtype):
    """n x heads vectors of 128 with a spread and an offset per head."""
    sigma = torch.exp(0.4 * torch.randn((heads, 1), generator=g, device="cuda"))
    mu = 0.3 * sigma * torch.randn((heads, 1), generator=g, device="cuda")
    return (torch.randn((n, heads, 128), generator=g, device="cuda") * sigma + mu).to(dtype)


class Linear:
    """One linear layer as a program holds it: weights, input, output, and the scratch between quantiser and product."""

    def __init__(self, g, n, k, m, fmt, dtype, rot=None, fused=True, out=None):
        self.n, self.k, self.m, self.fmt, self.rot = n, k, m, fmt, rot
        self.packed, self.codebook = _pack(_raw_weights(g, n, k, fmt, torch.float16), fmt)
        self.x = _act(g, (m, k), dtype)
        self.out = out if out is not None else torch.empty((m, n), dtype=torch.float16, device="cuda")
        self.y = self.xq = self.scale = self.work = None
        self.fused = fused and m == 1
        # rotations that run inside the multiplying launch: across heads, and short Hadamard ones
        self.inside = rot is not None and self.fused and fmt == "w2" and (
            rot.kind == rcp.ROT_HEADS or (rot.kind == rcp.ROT_WHT and k <= 2048))
        if fmt == "w2a16" or self.fused:
            if rot is not None and not self.inside:
                self.y = torch.empty((m, k), dtype=torch.float32, device="cuda")
        else:
            self.xq = torch.empty((m, k // 2), dtype=torch.uint8, device="cuda")
            self.scale = torch.empty((m,), dtype=torch.float16, device="cuda")
            need = rcp.act_workspace_bytes(m, k, rot)
            self.work = torch.empty(need, dtype=torch.uint8, device="cuda") if need else None

    def __call__(self):
        p, c, n, k, x = self.packed, self.codebook, self.n, self.k, self.x
        if self.fmt == "w2a16" or self.fused:
            if self.inside:
                return rcp.rotate_quant_w2a4_gemv(p, c, n, k, x, self.rot, ACT_CLIP, out=self.out)
            if self.y is not None:
                x = rcp.rotate_act(x, self.rot, y_out=self.y)
            if self.fmt == "w2a16":
                return rcp.w2a16_gemv(p, c, n, k, x, out=self.out)
            if self.fmt == "g128":
                return rcp.quant_w2a4_gemv_grouped(p, c, n, k, x, ACT_CLIP, out=self.out)
            if self.fmt == "w3":
                return rcp.quant_w3a4_gemv(p, c, n, k, x, ACT_CLIP, out=self.out)
            return rcp.quant_w2a4_gemv(p, c, n, k, x, ACT_CLIP, out=self.out)
        rcp.rotate_quant_act(x, self.rot, ACT_CLIP, xq_out=self.xq, scale_out=self.scale, workspace=self.work)
        if self.fmt == "g128":
            return rcp.w2a4_gemm_grouped(p, c, n, k, self.xq, self.scale, self.m, out=self.out)
        if self.fmt == "w3":
            return rcp.w3a4_gemv(p, c, n, k, self.xq, self.scale, out=self.out)
        return rcp.w2a4_gemv(p, c, n, k, self.xq, self.scale, self.m, out=self.out)


def _shapes(c):
    """(N, K) of the four launches' matrices of a decoder layer."""
    return [(c["hidden"] + 2 * c["kvdim"], c["hidden"]), (c["hidden"], c["hidden"]), (2 * c["ffn"], c["hidden"]),
            (c["hidden"], c["ffn"])]


def prepare(case, seed):
    g, kind, dtype = _gen(seed), case["kind"], DTYPES[case["dtype"]]
    if kind == "one":
        rot = rcp.Rotation.wht(case["k"]) if case["rot"] == "wht" else None
        return [Linear(g, case["n"], case["k"], case["m"], case["fmt"], dtype, rot, case["fused"])]
    if kind == "decode":
        h, f, w, m = case["hidden"], case["ffn"], case["wht"], case["m"]
        down = rcp.Rotation.wht(f) if f == w else rcp.Rotation.kron(w, _orthogonal(g, f // w))
        heads = rcp.Rotation.heads(case["heads"], h // case["heads"]) if case["heads"] else None
        shapes, rots = _shapes(case), (None, heads, None, down)
        outs = [torch.empty((case["layers"], m, n), dtype=torch.float16, device="cuda") for n, _ in shapes]
        calls = [Linear(g, n, k, m, case["fmt"], dtype, r, out=o[i])
                 for i in range(case["layers"]) for (n, k), r, o in zip(shapes, rots, outs)]
        return {"calls": calls, "outs": outs}
    if kind == "export":
        raws = [_raw_weights(g, n, k, case["fmt"], dtype) for n, k in _shapes(case)]
        return {"fmt": case["fmt"], "raw": raws, "out": [_pack(r, case["fmt"]) for r in raws]}
    layers = case["layers"]
    if kind == "prompt":
        n, h, s = case["n"], case["h"], case["s"]
        kv = [[_head_vectors(g, n, h, dtype) for _ in range(2)] for _ in range(layers)]
        return {"kv": kv, "cache": [rcp.kv4_new_cache(h, s, "cuda") + rcp.kv4_new_cache(h, s, "cuda") for _ in range(layers)]}
    hq, hkv = case["hq"], case["hkv"]
    b = case.get("b", 1)
    if kind == "kv":
        lengths = [case["s"]]
    else:
        r = torch.rand(b, generator=torch.Generator().manual_seed(int(seed)))
        lengths = [case["smin"] + int(v * (case["smax"] - case["smin"])) for v in r.tolist()]
        lengths[0] = case["smax"]
    s_max = max(lengths) + 64
    state = {"lengths": lengths, "positions": [v - 1 for v in lengths], "layers": []}
    for _ in range(layers):
        caches = []
        for rotate in (True, False):
            codes, params = rcp.kv4_new_cache(b * hkv, s_max, "cuda")
            for i, n in enumerate(lengths):  # the tokens seen so far
                if n > 1:
                    rcp.kv4_append(_head_vectors(g, n - 1, hkv, dtype), 0, codes[i * hkv:(i + 1) * hkv],
                                   params[i * hkv:(i + 1) * hkv], KV_CLIP, rotate)
            caches += [codes, params]
        need = b * rcp.kv4_workspace_bytes(hq, max(lengths))
        q = torch.randn((b, hq, 128), generator=g, device="cuda").to(dtype)
        state["layers"].append({
            "cache": tuple(caches), "q": q if kind == "kvbatch" else q[0], "qrows": q.view(b * hq, 128),
            "y": torch.empty((b * hq, 128), dtype=torch.float32, device="cuda"), "k": _head_vectors(g, b, hkv, dtype),
            "v": _head_vectors(g, b, hkv, dtype),
            "out": torch.empty((b, hq, 128) if kind == "kvbatch" else (hq, 128), dtype=torch.float16, device="cuda"),
            "work": torch.empty(max(need, 16), dtype=torch.uint8, device="cuda")})
    state["batched"] = kind == "kvbatch"
    state["r3"] = rcp.Rotation.wht(128)
    return state


# ---- one pass -------------------------------------------------------------------------------------
SOFTMAX = 1.0 / math.sqrt(128.0)


def run(state):
    if isinstance(state, list):
        return [call() for call in state]
    if "calls" in state:
        for call in state["calls"]:
            call()
        return state["outs"]
    if "raw" in state:
        for raw, (packed, codebook) in zip(state["raw"], state["out"]):
            _pack(raw, state["fmt"], packed, codebook)
        return state["out"]
    if "kv" in state:
        for (k, v), (kc, kp, vc, vp) in zip(state["kv"], state["cache"]):
            rcp.kv4_append_kv(k, v, 0, kc, kp, vc, vp, KV_CLIP, rotate_k=True)
        return state["cache"]
    for d in state["layers"]:
        kc, kp, vc, vp = d["cache"]
        if state["batched"]:
            rcp.kv4_append_batched(d["k"], state["positions"], kc, kp, KV_CLIP, rotate=True)
            rcp.kv4_append_batched(d["v"], state["positions"], vc, vp, KV_CLIP)
            y = rcp.rotate_act(d["qrows"], state["r3"], y_out=d["y"]).view(d["q"].shape)
            rcp.kv4_attn_decode_batched(y, state["lengths"], kc, kp, vc, vp, SOFTMAX, out=d["out"], workspace=d["work"])
        else:
            rcp.kv4_append_kv(d["k"], d["v"], state["positions"][0], kc, kp, vc, vp, KV_CLIP, rotate_k=True)
            rcp.kv4_rotate_attn_decode(d["q"], state["lengths"][0], kc, kp, vc, vp, SOFTMAX, out=d["out"], workspace=d["work"])
    return [(d["out"],) + d["cache"] for d in state["layers"]]


# ---- what a pass cannot do without ------------------------------------------------------------------
def _linear_work(n, k, m, fmt, itemsize, rot_m=0):
    weights = {"w2": n * k // 4 + 8 * n, "w2a16": n * k // 4 + 8 * n, "g128": n * k // 4 + n * k // 128 * 8,
               "w3": 3 * n * k // 8 + 16 * n}[fmt]
    return weights + m * k * itemsize + 2 * m * n + 4 * rot_m * rot_m, 2 * m * n * k + 2 * m * k * rot_m


def work(case):
    kind, size = case["kind"], DTYPES[case["dtype"]].itemsize
    nbytes = flops = 0
    if kind == "one":
        nbytes, flops = _linear_work(case["n"], case["k"], case["m"], case["fmt"], size)
    elif kind == "decode":
        for i, (n, k) in enumerate(_shapes(case)):
            rot_m = case["ffn"] // case["wht"] if i == 3 and case["ffn"] != case["wht"] else 0
            b, f = _linear_work(n, k, case["m"], case["fmt"], size, rot_m)
            nbytes, flops = nbytes + b * case["layers"], flops + f * case["layers"]
    elif kind == "export":
        for n, k in _shapes(case):
            nbytes += n * k * size + _linear_work(n, k, 0, case["fmt"], 0)[0] + 20 * (n * k // 128 if case["fmt"] == "g128" else n)
    elif kind == "prompt":
        nbytes = 2 * case["layers"] * case["n"] * case["h"] * (128 * size + 68)
    else:
        b = case.get("b", 1)
        tokens = case["s"] if kind == "kv" else case["smax"] + (b - 1) * (case["smin"] + case["smax"]) // 2
        nbytes = 2 * tokens * case["hkv"] * 68 + b * (case["hq"] * 128 * (size + 2) + 2 * case["hkv"] * (128 * size + 68))
        flops = 4 * tokens * case["hq"] * 128
        nbytes, flops = nbytes * case["layers"], flops * case["layers"]
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Packed bytes, tables, codes and zero points are exact.  16-bit outputs of binary32 sums: one rounding each.  Where
    an online Kronecker rotation precedes the quantiser, its binary32 summation order is free, and a value on a rounding
    boundary may take the neighbouring int4 code: about 1 / sqrt(K) of one layer's output for each such value."""
    if case["kind"] in ("export", "prompt"):
        return "exact"
    if case["kind"] == "decode" and case["ffn"] != case["wht"]:
        return {"rel": 5e-3}
    return {"rel": 1e-3}
