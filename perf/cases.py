"""The work whose speed is watched: calls of the library as a model's program makes them.

Seven kinds of pass, each through the public entry points of the package:

  rowsum   a data-movement chain read by the fp32 add + row-sum consumer (vt_elementwise)
  attn     one decode step's attention over a KV cache (vt_decode_attn): the contiguous cache with
           the new token's row still in the QKV buffer, or pages picked through a block table
  segment  one decode step: the merged QKV projection writes Q and the new K/V rows where they
           live (vt_gemm_store), attention then reads the caches (vt_decode_attn)
  qkv      the same projection over a chunk of new tokens per sequence (prefill)
  oproj    the attention output's head transpose read by the output projection (vt_gemm)
  ln       window partition -> LayerNorm -> linear (vt_gemm with the LayerNorm prologue)
  moe      token dispatch to experts (grouped vt_gemm over gathered rows) and the combine step that
           reads the expert rows back in token order (vt_weighted_sum)

`listed` holds the cases that are timed by name, `draw` makes more of the same ranges.  Descriptors,
weights, workspaces and output buffers belong to a program's set-up and are made in `prepare`.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2604_09558_amd as vt
from paper_2604_09558_amd import binding

DEV = "cuda:0"
DT = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}


# ------------------------------------------------------------------------------------------
# the cases
# ------------------------------------------------------------------------------------------
def listed():
    return [
        # the smallest call there is: a chain over a few hundred elements; launch and host cost
        {"name": "rowsum_tiny", "kind": "rowsum", "form": "slice", "a": 4, "b": 6, "c": 8, "lo": 4, "hi": 20, "ny": 5},
        # a bandwidth-bound reduction behind permute -> reshape -> concat, 335 MB
        {"name": "rowsum_335mb", "kind": "rowsum", "form": "heads", "a": 32, "b": 8192, "c": 128, "ny": 1024},
        # one decode step of two short conversations: projection + attention, latency matters
        {"name": "segment_b2_1k", "kind": "segment", "dtype": "f16", "B": 2, "hidden": 4096, "Hkv": 8, "G": 4, "D": 128,
         "cap": 1280, "S": 1001},
        # decode attention of a batch at 4096 keys, the new row still in the QKV buffer
        {"name": "attn_b8_4k", "kind": "attn", "form": "append", "dtype": "bf16", "B": 8, "Hkv": 8, "G": 4, "D": 128, "S": 4096},
        # serving from a paged cache, 64-wide heads, a larger batch of mid-length contexts
        {"name": "attn_paged_d64", "kind": "attn", "form": "paged", "dtype": "bf16", "B": 16, "Hkv": 8, "G": 4, "D": 64,
         "page": 64, "pages": 37},
        # chunked prefill: 100 new tokens of each of 4 sequences stored into Q buffer and caches
        {"name": "qkv_chunk_400", "kind": "qkv", "dtype": "bf16", "B": 4, "T": 100, "hidden": 4096, "Hkv": 8, "G": 4, "D": 128,
         "cap": 1024, "pos": 517},
        # the output projection of a long prefill batch, 275 GFLOP
        {"name": "oproj_8192", "kind": "oproj", "dtype": "bf16", "B": 16, "H": 32, "S": 512, "D": 128, "N": 4096},
        # the same for one short prompt of ragged length
        {"name": "oproj_333", "kind": "oproj", "dtype": "f16", "B": 1, "H": 32, "S": 333, "D": 128, "N": 4096},
        # first stage of a window-attention backbone, 100k tokens
        {"name": "ln_c128", "kind": "ln", "dtype": "f16", "B": 32, "R": 56, "win": 7, "C": 128, "N": 384},
        # its second stage: twice the channels, a quarter of the tokens
        {"name": "ln_c256", "kind": "ln", "dtype": "bf16", "B": 32, "R": 28, "win": 7, "C": 256, "N": 768},
        # experts' first product and combine for a decode batch: few rows per expert, weights dominate
        {"name": "moe_200", "kind": "moe", "dtype": "bf16", "T": 200, "Hd": 4096, "E": 8, "N": 14336},
        # the same for a prefill batch, 3.8 TFLOP
        {"name": "moe_16384", "kind": "moe", "dtype": "bf16", "T": 16384, "Hd": 4096, "E": 8, "N": 14336},
    ]


def _log(rng, lo, hi):
    """An integer of [lo, hi], uniform over the logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["rowsum", "segment", "attn", "attn", "qkv", "oproj", "ln", "moe"])
    dtype = rng.choice(["bf16", "bf16", "f16"])
    if kind == "rowsum":
        if rng.random() < 0.4:      # small chains whose runs are single elements
            a, b, c = _log(rng, 2, 24), _log(rng, 2, 24), _log(rng, 4, 256)
            lo = rng.randrange(0, a * b // 2)
            return {"kind": kind, "form": "slice", "a": a, "b": b, "c": c, "lo": lo, "hi": rng.randrange(lo + 1, a * b + 1),
                    "ny": _log(rng, 1, 40)}
        return {"kind": kind, "form": "heads", "a": _log(rng, 2, 32), "b": _log(rng, 16, 8192), "c": rng.choice([32, 64, 96, 128]),
                "ny": rng.choice([64, 256, 1000, 1024])}
    heads = {"Hkv": rng.choice([1, 2, 4, 8]), "G": rng.choice([1, 2, 4, 7, 8])}
    if kind == "segment":
        S = _log(rng, 32, 8192)
        return {"kind": kind, "dtype": dtype, "B": _log(rng, 1, 16), "hidden": rng.choice([1024, 2048, 3072, 4096]), "D": 128,
                "cap": (S + 127) // 128 * 128, "S": S, **heads}
    if kind == "attn":
        c = {"kind": kind, "dtype": dtype, "B": _log(rng, 1, 32), "D": rng.choice([64, 128, 128]), **heads}
        if rng.random() < 0.5:
            return {**c, "form": "append", "S": _log(rng, 32, 8192)}
        page = rng.choice([32, 64, 128])
        return {**c, "form": "paged", "page": page, "pages": _log(rng, 1, 8192 // page)}
    if kind == "qkv":
        T, D = _log(rng, 1, 256), rng.choice([64, 128])
        pos = rng.randrange(0, 1024)
        return {"kind": kind, "dtype": dtype, "B": _log(rng, 1, 8), "T": T, "hidden": rng.choice([768, 1024, 2048, 4096]), "D": D,
                "cap": 1280, "pos": pos, "Hkv": rng.choice([2, 4, 8]), "G": rng.choice([1, 2, 4])}
    if kind == "oproj":
        H, D = rng.choice([8, 12, 16, 32]), rng.choice([64, 128])
        return {"kind": kind, "dtype": dtype, "B": _log(rng, 1, 16), "H": H, "S": _log(rng, 16, 512), "D": D,
                "N": rng.choice([H * D, 1000, 2048, 3072, 4096])}
    if kind == "ln":
        C = rng.choice([64, 96, 128, 192, 256, 384, 512])
        R, win = rng.choice([(56, 7), (28, 7), (14, 7), (64, 8), (32, 8), (40, 5)])
        return {"kind": kind, "dtype": dtype, "B": _log(rng, 1, 32 if C <= 128 or R < 50 else 8), "R": R, "win": win, "C": C,
                "N": rng.choice([C, 3 * C, 4 * C, 200])}
    return {"kind": kind, "dtype": dtype, "T": _log(rng, 16, 8192), "Hd": rng.choice([1024, 2048, 4096]), "E": rng.choice([4, 8]),
            "N": rng.choice([1000, 1408, 3584, 8192, 14336])}


# ------------------------------------------------------------------------------------------
# inputs: everything a case's values depend on, from (case, seed) alone
# ------------------------------------------------------------------------------------------
class _Gen:
    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(seed)

    def normal(self, shape, dtype, std=1.0):
        """N(0, std), drawn in fp32 and rounded once."""
        out = torch.empty(shape, dtype=DT[dtype], device=DEV)
        flat = out.view(-1)
        step = 1 << 26
        for i in range(0, flat.numel(), step):
            n = min(step, flat.numel() - i)
            flat[i:i + n] = torch.randn(n, generator=self.g, device=DEV, dtype=torch.float32) * std
        return out

    def uniform(self, shape):
        return torch.rand(shape, generator=self.g, device=DEV, dtype=torch.float32) * 2.0 - 1.0


def _attn_shape(c):
    Hq = c["Hkv"] * c["G"]
    S = c["pages"] * c["page"] if c.get("form") == "paged" else c["S"]
    return c["B"], c["Hkv"], c["G"], Hq, S, c["D"]


def _inputs(c, seed):
    g = _Gen(seed)
    kind = c["kind"]
    t = {}
    if kind == "rowsum":
        if c["form"] == "slice":
            t["X"], t["Y"] = g.uniform((c["a"], c["b"], c["c"])), g.uniform((c["c"], c["ny"]))
            t["Z"] = g.uniform((c["c"], c["hi"] - c["lo"] + c["ny"]))
        else:
            t["X"], t["Y"] = g.normal((c["a"], c["b"], c["c"]), "f32"), g.normal((c["b"], c["ny"]), "f32")
            t["Z"] = g.normal((c["b"], c["a"] * c["c"] + c["ny"]), "f32")
        return t
    dt = c["dtype"]
    if kind == "attn":
        B, Hkv, G, Hq, S, D = _attn_shape(c)
        if c["form"] == "append":
            t["QKV"] = g.normal((B, 1, (Hq + 2 * Hkv) * D), dt)
            t["Kcache"], t["Vcache"] = g.normal((B, Hkv, S, D), dt), g.normal((B, Hkv, S, D), dt)
        else:
            pool = B * c["pages"] + 3
            t["Qs"] = g.normal((B, 1, Hq * D), dt)
            t["Kpool"], t["Vpool"] = g.normal((pool, Hkv, c["page"], D), dt), g.normal((pool, Hkv, c["page"], D), dt)
            order = np.random.default_rng(seed).permutation(pool)[:B * c["pages"]].astype(np.int32)
            t["bt"] = torch.from_numpy(order).to(DEV)
            t["bt_host"] = order
    elif kind in ("segment", "qkv"):
        B, Hkv, D, cap = c["B"], c["Hkv"], c["D"], c["cap"]
        Hq, T = Hkv * c["G"], c.get("T", 1)
        t["X"], t["W"] = g.normal((B * T, c["hidden"]), dt), g.normal((c["hidden"], (Hq + 2 * Hkv) * D), dt, 0.02)
        t["Qbuf"] = g.normal((B, T, Hq * D), dt)
        t["Kcache"], t["Vcache"] = g.normal((B, Hkv, cap, D), dt), g.normal((B, Hkv, cap, D), dt)
    elif kind == "oproj":
        t["O"] = g.normal((c["B"], c["H"], c["S"], c["D"]), dt)
        t["W"] = g.normal((c["H"] * c["D"], c["N"]), dt, 0.02)
    elif kind == "ln":
        t["X"], t["W"] = g.normal((c["B"], c["R"], c["R"], c["C"]), dt), g.normal((c["C"], c["N"]), dt, 0.02)
    else:
        T, E = c["T"], c["E"]
        t["tokens"], t["W"] = g.normal((T, c["Hd"]), dt), g.normal((E, c["Hd"], c["N"]), dt, 0.02)
        r = np.random.default_rng(seed)
        first = r.integers(0, E, size=T)
        second = (first + 1 + r.integers(0, E - 1, size=T)) % E          # two distinct experts, uniform
        lists = [np.nonzero((first == e) | (second == e))[0].astype(np.int32) for e in range(E)]
        pos = np.zeros((2, T), dtype=np.int32)                           # where a token's two rows are
        seen, row = np.zeros(T, dtype=np.int64), 0
        for tok in lists:
            pos[seen[tok], tok] = row + np.arange(tok.size)
            seen[tok] += 1
            row += tok.size
        logits = r.standard_normal(size=(T, 2)).astype(np.float32)
        ex = np.exp(logits - logits.max(axis=1, keepdims=True))
        t["lists"], t["pos"] = lists, pos
        t["weights"] = torch.from_numpy((ex / ex.sum(axis=1, keepdims=True)).astype(np.float32)).to(DEV)
    return t


# ------------------------------------------------------------------------------------------
# set-up and pass
# ------------------------------------------------------------------------------------------
def _desc(chain, t, dtype, result, tables=None):
    """Descriptor of `result`; `tables` maps an index name to (host array, device tensor)."""
    src = {k: (tuple(v.shape), dtype, v.data_ptr()) for k, v in t.items() if isinstance(v, torch.Tensor) and v.dtype == DT[dtype]}
    tables = tables or {}
    return vt.build_chain(chain, src, result, {k: h for k, (h, _) in tables.items()}, {k: d.data_ptr() for k, (_, d) in tables.items()})


def _cache_store_chain(c):
    """Columns of the merged projection seen where they are stored: Q buffer, K rows, V rows."""
    B, Hkv, D, T = c["B"], c["Hkv"], c["D"], c.get("T", 1)
    pos = c["pos"] if c["kind"] == "qkv" else c["S"] - 1
    chain = [("q2", "reshape", ("Qbuf",), {"shape": (B * T, Hkv * c["G"] * D)})]
    for n, cache in (("k", "Kcache"), ("v", "Vcache")):
        chain += [(n + "s", "slice", (cache,), {"dim": 2, "start": pos, "stop": pos + T}),
                  (n + "p", "permute", (n + "s",), {"perm": (0, 2, 1, 3)}),
                  (n + "2", "reshape", (n + "p",), {"shape": (B * T, Hkv * D)})]
    return chain + [("Cout", "concat", ("q2", "k2", "v2"), {"dim": 1})]


def _attn_chain(c):
    B, Hkv, G, Hq, S, D = _attn_shape(c)
    chain = []
    form = c.get("form", "segment")
    if form == "append":
        sizes = (Hq * D, Hkv * D, Hkv * D)
        chain += [("q0", "split", ("QKV",), {"dim": 2, "sizes": sizes, "output": 0})]
    q = {"append": "q0", "paged": "Qs", "segment": "Qbuf"}[form]
    chain += [("q1", "reshape", (q,), {"shape": (B, 1, Hq, D)}), ("Q", "permute", ("q1",), {"perm": (0, 2, 1, 3)})]
    for n, cache, out in (("k", "K", 1), ("v", "V", 2)):
        if form == "append":
            chain += [(n + "0", "split", ("QKV",), {"dim": 2, "sizes": sizes, "output": out}),
                      (n + "1", "reshape", (n + "0",), {"shape": (B, 1, Hkv, D)}),
                      (n + "n", "permute", (n + "1",), {"perm": (0, 2, 1, 3)}),
                      (n + "p", "slice", (cache + "cache",), {"dim": 2, "start": 0, "stop": S - 1}),
                      (n + "f", "concat", (n + "p", n + "n"), {"dim": 2})]
        elif form == "paged":
            chain += [(n + "g", "index_select", (cache + "pool",), {"dim": 0, "index": "bt"}),
                      (n + "r", "reshape", (n + "g",), {"shape": (B, c["pages"], Hkv, c["page"], D)}),
                      (n + "t", "permute", (n + "r",), {"perm": (0, 2, 1, 3, 4)}),
                      (n + "f", "reshape", (n + "t",), {"shape": (B, Hkv, S, D)})]
        else:
            chain += [(n + "f", "slice", (cache + "cache",), {"dim": 2, "start": 0, "stop": S})]
        chain += [(n + "u", "unsqueeze", (n + "f",), {"dim": 2}),
                  (n + "x", "expand", (n + "u",), {"shape": (B, Hkv, G, S, D)}),
                  (cache, "reshape", (n + "x",), {"shape": (B, Hq, S, D)})]
    return chain


def _prepare_store(c, t, s):
    M, K, N = t["X"].shape[0], t["W"].shape[0], t["W"].shape[1]
    s["A"], s["W"] = _desc([], t, c["dtype"], "X"), _desc([], t, c["dtype"], "W")
    s["Cout"] = _desc(_cache_store_chain(c), t, c["dtype"], "Cout")
    s["store_ws_bytes"] = binding.vt_gemm_store_workspace(M, N, K)
    s["store_ws"] = torch.empty(s["store_ws_bytes"], dtype=torch.uint8, device=DEV)
    binding.vt_gemm_store_workspace_init(s["store_ws"], s["store_ws_bytes"])


def _prepare_attn(c, t, s):
    B, Hkv, G, Hq, S, D = _attn_shape(c)
    tables = {"bt": (t["bt_host"], t["bt"])} if "bt" in t else None
    chain = _attn_chain(c)
    s["Q"], s["K"], s["V"] = (_desc(chain, t, c["dtype"], n, tables) for n in ("Q", "K", "V"))
    s["ws_bytes"] = vt.vt_decode_attn_workspace(B, Hq, D, S)
    s["ws"] = torch.empty(s["ws_bytes"], dtype=torch.uint8, device=DEV)
    vt.vt_decode_attn_workspace_init(s["ws"], s["ws_bytes"])
    s["out"] = torch.empty((B, Hq, D), dtype=DT[c["dtype"]], device=DEV)
    s["lse"] = torch.empty((B, Hq), dtype=torch.float32, device=DEV)
    s["scale"] = 1.0 / math.sqrt(D)


def prepare(case, seed):
    c, t = case, _inputs(case, seed)
    s = {"case": c, "t": t}
    kind = c["kind"]
    if kind == "rowsum":
        if c["form"] == "slice":
            chain = [("t1", "permute", ("X",), {"perm": (2, 0, 1)}),
                     ("t2", "reshape", ("t1",), {"shape": (c["c"], c["a"] * c["b"])}),
                     ("t3", "slice", ("t2",), {"dim": 1, "start": c["lo"], "stop": c["hi"]}),
                     ("V", "concat", ("t3", "Y"), {"dim": 1})]
        else:
            chain = [("t1", "permute", ("X",), {"perm": (1, 0, 2)}),
                     ("t2", "reshape", ("t1",), {"shape": (c["b"], c["a"] * c["c"])}),
                     ("V", "concat", ("t2", "Y"), {"dim": 1})]
        s["x"], s["y"] = _desc(chain, t, "f32", "V"), _desc([], t, "f32", "Z")
        s["out"] = torch.empty(t["Z"].shape[0], dtype=torch.float32, device=DEV)
        return s
    dt = c["dtype"]
    if kind == "attn":
        _prepare_attn(c, t, s)
    elif kind == "segment":
        _prepare_store(c, t, s)
        _prepare_attn(c, t, s)
    elif kind == "qkv":
        _prepare_store(c, t, s)
    elif kind == "oproj":
        M, K = c["B"] * c["S"], c["H"] * c["D"]
        s["A"] = [_desc([("o1", "permute", ("O",), {"perm": (0, 2, 1, 3)}), ("A", "reshape", ("o1",), {"shape": (M, K)})], t, dt, "A")]
        s["W"] = [_desc([], t, dt, "W")]
        s["out"] = torch.empty((M, c["N"]), dtype=DT[dt], device=DEV)
    elif kind == "ln":
        B, R, win, C = c["B"], c["R"], c["win"], c["C"]
        nw = R // win
        s["A"] = [_desc([("x1", "reshape", ("X",), {"shape": (B, nw, win, nw, win, C)}),
                         ("x2", "permute", ("x1",), {"perm": (0, 1, 3, 2, 4, 5)}),
                         ("T", "reshape", ("x2",), {"shape": (B * nw * nw, win * win, C)})], t, dt, "T")]
        s["W"] = [_desc([], t, dt, "W")]
        s["out"] = torch.empty((B * R * R, c["N"]), dtype=DT[dt], device=DEV)
    else:
        T, E, Hd, N = c["T"], c["E"], c["Hd"], c["N"]
        s["Y"] = torch.empty((2 * T, N), dtype=DT[dt], device=DEV)
        s["out"] = torch.empty((T, N), dtype=DT[dt], device=DEV)
        s["A"], s["W"], s["C"], s["index"], row = [], [], [], [], 0
        for e, tok in enumerate(t["lists"]):
            if tok.size == 0:
                continue
            dev = torch.from_numpy(tok).to(DEV)
            s["index"].append(dev)
            s["A"].append(_desc([("A", "index_select", ("tokens",), {"dim": 0, "index": "tok"})], t, dt, "A", {"tok": (tok, dev)}))
            s["W"].append(_desc([("w", "slice", ("W",), {"dim": 0, "start": e, "stop": e + 1}),
                                 ("B", "reshape", ("w",), {"shape": (Hd, N)})], t, dt, "B"))
            s["C"].append(s["Y"].data_ptr() + row * N * 2)
            row += tok.size
        for k, name in enumerate(("x", "y")):
            dev = torch.from_numpy(t["pos"][k]).to(DEV)
            s["index"].append(dev)
            s[name] = _desc([(name, "index_select", ("Y",), {"dim": 0, "index": "pos"})], {"Y": s["Y"]}, dt, name,
                            {"pos": (t["pos"][k], dev)})
    return s


def run(state):
    s, c = state, state["case"]
    kind, t = c["kind"], s["t"]
    if kind == "rowsum":
        vt.vt_elementwise(vt.EW_ADD_ROWSUM, s["x"], s["y"], 0.0, s["out"])
        return s["out"]
    if kind in ("segment", "qkv"):
        binding.vt_gemm_store(s["A"], s["W"], s["Cout"], s["store_ws"], s["store_ws_bytes"])
        if kind == "qkv":
            return t["Qbuf"], t["Kcache"], t["Vcache"]
    if kind in ("segment", "attn"):
        vt.vt_decode_attn(s["Q"], s["K"], s["V"], s["scale"], s["out"], s["ws"], s["ws_bytes"], lse=s["lse"])
        return (s["out"], s["lse"]) if kind == "attn" else (s["out"], s["lse"], t["Qbuf"], t["Kcache"], t["Vcache"])
    if kind == "moe":
        vt.vt_gemm(s["A"], s["W"], s["C"], c["dtype"])
        binding.vt_weighted_sum(s["x"], s["y"], t["weights"], s["out"])
        return s["Y"], s["out"]
    if kind == "ln":
        vt.vt_gemm(s["A"], s["W"], [s["out"]], c["dtype"], vt.GEMM_LAYERNORM, 1e-5)
    else:
        vt.vt_gemm(s["A"], s["W"], [s["out"]], c["dtype"])
    return s["out"]


# ------------------------------------------------------------------------------------------
# what a pass cannot do without
# ------------------------------------------------------------------------------------------
def _work_store(c):
    M, K = c["B"] * c.get("T", 1), c["hidden"]
    N = (c["G"] + 2) * c["Hkv"] * c["D"]
    return {"bytes": 2 * (M * K + K * N + M * N), "flops": 2 * M * N * K}


def _work_attn(c):
    B, Hkv, G, Hq, S, D = _attn_shape(c)
    return {"bytes": 2 * B * D * (2 * Hkv * S + 2 * Hq) + 4 * B * Hq, "flops": 4 * B * Hq * S * D}


def work(case):
    c, kind = case, case["kind"]
    if kind == "rowsum":
        if c["form"] == "slice":
            R, C = c["c"], c["hi"] - c["lo"] + c["ny"]
        else:
            R, C = c["b"], c["a"] * c["c"] + c["ny"]
        return {"bytes": 8 * R * C + 4 * R, "flops": 2 * R * C}
    if kind == "attn":
        return _work_attn(c)
    if kind == "qkv":
        return _work_store(c)
    if kind == "segment":
        p, a = _work_store(c), _work_attn(c)
        return {k: p[k] + a[k] for k in p}
    if kind == "moe":
        T, E, Hd, N = c["T"], c["E"], c["Hd"], c["N"]
        # tokens once, every expert's weight once, the expert rows written and read back, the result
        return {"bytes": 2 * (T * Hd + E * Hd * N + 4 * T * N + T * N) + 16 * T, "flops": 4 * T * Hd * N + 6 * T * N}
    M, K, N = (c["B"] * c["S"], c["H"] * c["D"], c["N"]) if kind == "oproj" else (c["B"] * c["R"] * c["R"], c["C"], c["N"])
    return {"bytes": 2 * (M * K + K * N + M * N), "flops": 2 * M * N * K + (8 * M * K if kind == "ln" else 0)}


def tolerance(case):
    """About four times the distance from the 64-bit result measured for each kind: one rounding of
    the result to its type, and in attention, the segment and the LayerNorm product a second one
    of the weights or of the normalised row."""
    kind = case["kind"]
    if kind == "rowsum":
        return {"rel": 1e-6}
    return {"rel": 1e-2 if case["dtype"] == "bf16" else 1.5e-3}


# ------------------------------------------------------------------------------------------
# the same in 64 bits, plain torch
# ------------------------------------------------------------------------------------------
def _exact_attn(c, t):
    """Batch by batch: scores, softmax and the weighted sum of V's rows."""
    B, Hkv, G, Hq, S, D = _attn_shape(c)
    out = torch.empty((B, Hq, D), dtype=torch.float64, device=DEV)
    lse = torch.empty((B, Hq), dtype=torch.float64, device=DEV)
    for b in range(B):
        if c.get("form") == "append":
            row = t["QKV"][b, 0].double()
            q = row[:Hq * D].view(Hkv, G, D)
            k, v = t["Kcache"][b].double(), t["Vcache"][b].double()
            k[:, S - 1] = row[Hq * D:(Hq + Hkv) * D].view(Hkv, D)
            v[:, S - 1] = row[(Hq + Hkv) * D:].view(Hkv, D)
        elif c.get("form") == "paged":
            pages = t["bt"][b * c["pages"]:(b + 1) * c["pages"]].long()
            q = t["Qs"][b, 0].double().view(Hkv, G, D)
            k, v = (t[p][pages].double().permute(1, 0, 2, 3).reshape(Hkv, S, D) for p in ("Kpool", "Vpool"))
        else:
            q = t["Qbuf"][b, 0].double().view(Hkv, G, D)
            k, v = t["Kcache"][b, :, :S].double(), t["Vcache"][b, :, :S].double()
        for h in range(Hkv):
            x = torch.mm(q[h], k[h].t().contiguous()) / math.sqrt(D)
            l = torch.logsumexp(x, dim=1, keepdim=True)
            lse[b, h * G:(h + 1) * G] = l[:, 0]
            out[b, h * G:(h + 1) * G] = torch.mm(torch.exp(x - l), v[h])
    return out, lse


def _exact_store(c, t):
    """Q buffer and caches after the projection, in 64 bits."""
    B, Hkv, D, T = c["B"], c["Hkv"], c["D"], c.get("T", 1)
    Hq, pos = Hkv * c["G"], c["pos"] if c["kind"] == "qkv" else c["S"] - 1
    p = torch.mm(t["X"].double(), t["W"].double()).view(B, T, -1)
    k, v = t["Kcache"].double(), t["Vcache"].double()
    k[:, :, pos:pos + T] = p[:, :, Hq * D:(Hq + Hkv) * D].reshape(B, T, Hkv, D).permute(0, 2, 1, 3)
    v[:, :, pos:pos + T] = p[:, :, (Hq + Hkv) * D:].reshape(B, T, Hkv, D).permute(0, 2, 1, 3)
    return p[:, :, :Hq * D].contiguous(), k, v


def exact(case, seed):
    c, t = case, _inputs(case, seed)
    kind = c["kind"]
    if kind == "rowsum":
        if c["form"] == "slice":
            x = t["X"].double().permute(2, 0, 1).reshape(c["c"], c["a"] * c["b"])[:, c["lo"]:c["hi"]]
        else:
            x = t["X"].double().permute(1, 0, 2).reshape(c["b"], c["a"] * c["c"])
        return x.sum(1) + t["Y"].double().sum(1) + t["Z"].double().sum(1)
    if kind == "attn":
        return _exact_attn(c, t)
    if kind in ("segment", "qkv"):
        q, k, v = _exact_store(c, t)
        if kind == "qkv":
            return q, k, v
        out, lse = _exact_attn(c, {"Qbuf": q, "Kcache": k, "Vcache": v})
        return out, lse, q, k, v
    if kind == "oproj":
        a = t["O"].double().permute(0, 2, 1, 3).reshape(c["B"] * c["S"], c["H"] * c["D"])
        return torch.mm(a, t["W"].double())
    if kind == "ln":
        B, R, win, C = c["B"], c["R"], c["win"], c["C"]
        nw = R // win
        x = t["X"].double().view(B, nw, win, nw, win, C).permute(0, 1, 3, 2, 4, 5).reshape(-1, C)
        x = x - x.mean(1, keepdim=True)
        return torch.mm(x / torch.sqrt((x * x).mean(1, keepdim=True) + 1e-5), t["W"].double())
    T, N = c["T"], c["N"]
    y = torch.empty((2 * T, N), dtype=torch.float64, device=DEV)
    row = 0
    for e, tok in enumerate(t["lists"]):
        if tok.size:
            y[row:row + tok.size] = torch.mm(t["tokens"][torch.from_numpy(tok).long().to(DEV)].double(), t["W"][e].double())
        row += tok.size
    w = t["weights"].double()
    pos = torch.from_numpy(t["pos"]).long().to(DEV)
    return y, w[:, :1] * y[pos[0]] + w[:, 1:] * y[pos[1]]
