"""Timed cases of the framework's public entry points.

Each case is one call path that a program built on the package makes: the
chunked attention walk (forward and backward, with the offload modes), the
forward alone, the allocation-free backward of one chunk, the MLP and the
LayerNorm of a layer through the layer building blocks, and the whole layer.
Sizes are those of the package's own benchmark and tests (32 heads x 128,
chunks of 4096 to 16384 tokens, GQA 32/8, a layer of width 4096; the fp32
configuration of 1024 tokens) or generic ones between them.
"""
import math

import torch

from paper_2503_10377_amd import sppo as L
from paper_2503_10377_amd.chunked import ChunkedAttention
from paper_2503_10377_amd.chunked_layer import ChunkedLayer

BF, F32, F64 = torch.bfloat16, torch.float32, torch.float64


# ------------------------------------------------------------------- the cases
def _walk(name, S, N, Hq, Hkv, D, dtype="bf16", B=1, ragged=False, offload="none"):
    c = {"kind": "walk", "B": B, "S": S, "N": N, "Hq": Hq, "Hkv": Hkv, "D": D, "dtype": dtype, "ragged": ragged,
         "offload": offload}
    return dict(c, name=name) if name else c


def listed():
    return [
        # The fp32 configuration: a small walk held to fp32 accuracy, for checking a model against a reference.
        _walk("walk_f32_1k", 1024, 4, 1, 1, 64, dtype="f32"),
        # The smallest bf16 training step: latency and launches.
        _walk("walk_2k", 2048, 4, 4, 4, 128),
        # Batched, grouped-query, head size 64, chunk boundaries off every tile grid, offloaded.
        _walk("walk_5k_ragged_gqa_d64", 5001, 3, 8, 2, 64, B=2, ragged=True, offload="qol"),
        # Prefill: the forward alone over chunks of 4096.
        {"name": "forward_16k_gqa", "kind": "forward", "S": 16384, "N": 4, "Hq": 32, "Hkv": 8, "D": 128},
        # The backward of one chunk by a caller that cannot allocate.
        {"name": "bwd_chunk_2k_of_16k_gqa", "kind": "bwd_chunk", "S": 16384, "rows": 2048, "Hq": 32, "Hkv": 8,
         "D": 128},
        # The benchmark's 32K configuration.
        _walk("walk_32k", 32768, 8, 32, 32, 128),
        # Grouped-query heads and 16384-token chunks of the 512K configuration, with K/V eviction.
        _walk("walk_64k_gqa_evict", 65536, 4, 32, 8, 128, offload="qkvol_evict"),
        # The benchmark's headline configuration: 128K tokens, 16 chunks, offload.
        _walk("walk_128k_offload", 131072, 16, 32, 32, 128, offload="qkvol"),
        # The MLP of a small layer on a ragged number of tokens, forward and backward.
        {"name": "mlp_1k_ragged", "kind": "mlp", "rows": 1000, "N": 1, "H": 1024},
        # The MLP of the layer configuration over two chunks of 8192, forward and backward.
        {"name": "mlp_16k", "kind": "mlp", "rows": 16384, "N": 2, "H": 4096},
        # LayerNorm of one chunk of the layer configuration, forward and backward.
        {"name": "norm_8k", "kind": "norm", "rows": 8192, "H": 4096},
        # A whole layer of the layer configuration over two chunks of 8192, activations offloaded.
        {"name": "layer_16k", "kind": "layer", "S": 16384, "N": 2, "Hq": 32, "Hkv": 32, "D": 128, "offload": "qol"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


HEADS = ((4, 4), (8, 2), (8, 8), (16, 4), (16, 16), (32, 8), (32, 32))


def draw(rng):
    kind = rng.choice(("walk", "walk", "walk", "walk_f32", "forward", "bwd_chunk", "mlp", "mlp", "norm", "layer"))
    D = rng.choice((64, 128, 128))
    if kind == "walk_f32":
        S = _log(rng, 256, 4096)
        Hq, Hkv = rng.choice(((1, 1), (2, 1), (4, 4), (8, 2)))
        return _walk(None, S, rng.randint(1, 4), Hq, Hkv, D, dtype="f32", ragged=True)
    Hq, Hkv = rng.choice(HEADS)
    if kind == "walk":
        S = _log(rng, 512, 49152)
        B = rng.randint(1, 3) if S <= 4096 else 1
        N = rng.randint(1, max(1, min(16, S // 256)))
        return _walk(None, S, N, Hq, Hkv, D, B=B, ragged=True,
                     offload=rng.choice(("none", "none", "qol", "qkvol", "qkvol_evict")))
    if kind == "forward":
        S = _log(rng, 512, 49152)
        return {"kind": "forward", "S": S, "N": rng.randint(1, max(1, min(12, S // 512))), "Hq": Hq, "Hkv": Hkv,
                "D": D}
    if kind == "bwd_chunk":
        S = _log(rng, 1024, 32768)
        return {"kind": "bwd_chunk", "S": S, "rows": _log(rng, 64, min(S, 8192)), "Hq": Hq, "Hkv": Hkv, "D": D}
    if kind == "mlp":
        rows = _log(rng, 128, 20000)
        return {"kind": "mlp", "rows": rows, "N": rng.randint(1, 2) if rows > 2000 else 1,
                "H": 256 * rng.randint(2, 16)}
    if kind == "norm":
        return {"kind": "norm", "rows": _log(rng, 16, 30000), "H": 8 * _log(rng, 32, 1024)}
    Hq, Hkv = rng.choice(((8, 4), (16, 4), (16, 16), (32, 8)))
    S = _log(rng, 512, 12000)
    return {"kind": "layer", "S": S, "N": rng.randint(1, 3), "Hq": Hq, "Hkv": Hkv, "D": D,
            "offload": rng.choice(("none", "qol", "qkvol"))}


def _offsets(S, N, ragged):
    """Equal chunks, or chunk boundaries moved off every power of two."""
    if not ragged and S % N == 0:
        return [S // N * i for i in range(N + 1)]
    off = [S * i // N for i in range(N + 1)]
    shift = max(1, min(29, S // (4 * N)))
    return [c + (shift if 0 < i < N and i % 2 else -shift if 0 < i < N else 0) for i, c in enumerate(off)]


# ------------------------------------------------------------------- inputs
class _Draws:
    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda").manual_seed(int(seed))

    def __call__(self, *shape, dt=BF, std=1.0, mean=0.0):
        x = torch.randn(shape, generator=self.gen, device="cuda", dtype=F32)
        return (x if std == 1.0 and mean == 0.0 else x * std + mean).to(dt)


def _attn_inputs(B, S, Hq, Hkv, D, dt, seed, do=True):
    """Q, K, V (and dO) after a projection of normalised activations: N(0, 1)."""
    d = _Draws(seed)
    inp = {"q": d(B, S, Hq, D, dt=dt), "k": d(B, S, Hkv, D, dt=dt), "v": d(B, S, Hkv, D, dt=dt)}
    if do:
        inp["do"] = d(B, S, Hq, D, dt=dt)
    return inp


def _mlp_inputs(case, seed):
    d, n, H = _Draws(seed), case["rows"], case["H"]
    return {"z": d(n, H), "h": d(n, H), "dy": d(n, H), "w1": d(H, 4 * H, std=H ** -0.5),
            "w2": d(4 * H, H, std=(4 * H) ** -0.5)}


def _norm_inputs(case, seed):
    d, n, H = _Draws(seed), case["rows"], case["H"]
    return {"x": d(n, H, std=2.0, mean=0.5), "dy": d(n, H), "dres": d(n, H), "g": d(H, dt=F32, std=0.1, mean=1.0),
            "b": d(H, dt=F32, std=0.1)}


def _layer_inputs(case, seed):
    d, S, Hq, Hkv, D = _Draws(seed), case["S"], case["Hq"], case["Hkv"], case["D"]
    H, wt = Hq * D, (Hq + 2 * Hkv) * D
    inp = {"x": d(S, H), "dy": d(S, H)}
    p = {"w_qkv": d(H, wt, std=H ** -0.5), "w_o": d(H, H, std=H ** -0.5), "w_1": d(H, 4 * H, std=H ** -0.5),
         "w_2": d(4 * H, H, std=(4 * H) ** -0.5)}
    for k in ("1", "2"):
        p["g" + k] = d(H, dt=F32, std=0.1, mean=1.0)
        p["b" + k] = d(H, dt=F32, std=0.1)
    return inp, p


def _chunk_forward(q, k, v, c0):
    """O and LSE of the query rows [c0, c0 + n) in fp32 (the saved activations that a chunk's backward gets)."""
    n, Hq, D = q.shape
    G = Hq // k.shape[1]
    o, lse = torch.empty_like(q), torch.empty(Hq, n, device="cuda", dtype=F32)
    for h in range(Hq):
        s = (q[:, h].float() @ k[:c0 + n, h // G].float().t()) / math.sqrt(D)
        rows = torch.arange(c0, c0 + n, device="cuda")[:, None]
        s.masked_fill_(torch.arange(c0 + n, device="cuda")[None, :] > rows, -math.inf)
        lse[h] = torch.logsumexp(s, dim=1)
        o[:, h] = (torch.exp(s - lse[h][:, None]) @ v[:c0 + n, h // G].float()).to(o.dtype)
    return o, lse


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("walk", "forward"):
        B, S, N, Hq, Hkv, D = case.get("B", 1), case["S"], case["N"], case["Hq"], case["Hkv"], case["D"]
        dtype = case.get("dtype", "bf16")
        inp = _attn_inputs(B, S, Hq, Hkv, D, BF if dtype == "bf16" else F32, seed, do=kind == "walk")
        ca = ChunkedAttention(B, S, N, Hq, Hkv, D, dtype=dtype, offsets=_offsets(S, N, case.get("ragged", False)),
                              offload=case.get("offload", "none"))
        return {"kind": kind, "ca": ca, "inp": inp, "out": ca.alloc_outputs()}
    if kind == "bwd_chunk":
        S, n, Hq, Hkv, D = case["S"], case["rows"], case["Hq"], case["Hkv"], case["D"]
        inp = _attn_inputs(1, S, Hq, Hkv, D, BF, seed)
        q, do = inp["q"][0, S - n:].clone(), inp["do"][0, S - n:].clone()
        o, lse = _chunk_forward(q, inp["k"][0], inp["v"][0], S - n)
        return {"kind": kind, "case": case, "q": q, "k": inp["k"], "v": inp["v"], "do": do, "o": o, "lse": lse,
                "dq": torch.empty_like(q), "dk": torch.empty(S, Hkv, D, device="cuda", dtype=F32),
                "dv": torch.empty(S, Hkv, D, device="cuda", dtype=F32)}
    e = lambda *shape, dt=BF: torch.empty(shape, device="cuda", dtype=dt)  # noqa: E731
    if kind == "mlp":
        t, n, H = _mlp_inputs(case, seed), case["rows"], case["H"]
        return {"kind": kind, "case": case, **t, "w1T": t["w1"].t().contiguous(), "w2T": t["w2"].t().contiguous(),
                "a": e(n, 4 * H), "g": e(n, 4 * H), "y": e(n, H), "da": e(n, 4 * H), "dz": e(n, H),
                "dw1": e(H, 4 * H, dt=F32), "dw2": e(4 * H, H, dt=F32)}
    if kind == "norm":
        n, H = case["rows"], case["H"]
        wsb = L.sppo_layernorm_bwd_workspace(n, H)
        return {"kind": kind, "case": case, **_norm_inputs(case, seed), "y": e(n, H), "mean": e(n, dt=F32),
                "rstd": e(n, dt=F32), "dx": e(n, H), "dg": e(H, dt=F32), "db": e(H, dt=F32), "ws": e(wsb // 4, dt=F32),
                "wsb": wsb}
    inp, p = _layer_inputs(case, seed)
    lay = ChunkedLayer(case["S"], case["N"], case["Hq"], case["Hkv"], case["D"],
                       offsets=_offsets(case["S"], case["N"], False), offload=case["offload"])
    return {"kind": kind, "layer": lay, "inp": inp, "p": p, "out": lay.alloc_outputs()}


# ------------------------------------------------------------------- one pass
def run(st):
    kind = st["kind"]
    if kind == "walk":
        out = st["out"]
        st["ca"].step(st["inp"], out)
        return {k: out[k] for k in ("o", "lse", "dq", "dk", "dv")}
    if kind == "forward":
        st["ca"].forward_only(st["inp"], st["out"])
        return {k: st["out"][k] for k in ("o", "lse")}
    if kind == "bwd_chunk":
        c = st["case"]
        L.sppo_attn_bwd_chunk_noalloc(1, c["S"], c["S"] - c["rows"], c["S"], c["Hq"], c["Hkv"], c["D"], "bf16", 0.0, 0,
                                      st["q"], st["k"], st["v"], st["o"], st["lse"], st["do"], st["dq"], st["dk"],
                                      st["dv"])
        return {k: st[k] for k in ("dq", "dk", "dv")}
    if kind == "mlp":
        return _run_mlp(st)
    if kind == "norm":
        n, H = st["case"]["rows"], st["case"]["H"]
        L.sppo_layernorm_fwd(n, H, st["x"], H, st["g"], st["b"], 1e-5, st["y"], H, st["mean"], st["rstd"])
        L.sppo_layernorm_bwd(n, H, st["x"], H, st["g"], st["mean"], st["rstd"], st["dy"], H, st["dres"], H, st["dx"], H,
                             st["dg"], st["db"], st["ws"], st["wsb"], accumulate=0)
        return {k: st[k] for k in ("y", "mean", "rstd", "dx", "dg", "db")}
    st["layer"].step(st["inp"], st["p"], st["out"])
    return st["out"]


def _run_mlp(st):
    """y = h + gelu(z W1) W2 chunk by chunk, then the reverse walk: dz, and dW1, dW2 summed over the chunks."""
    n, N, H = st["case"]["rows"], st["case"]["N"], st["case"]["H"]
    F = 4 * H
    off = _offsets(n, N, False)
    rows = [slice(off[i], off[i + 1]) for i in range(N)]
    for r in rows:
        m = r.stop - r.start
        a, g = st["a"][r], st["g"][r]
        L.sppo_gemm_bf16("nt", m, F, H, st["z"][r], H, st["w1T"], H, g, F, "gelu", a, F)
        L.sppo_gemm_bf16("nt", m, H, F, g, F, st["w2T"], F, st["y"][r], H, "add_bf16", st["h"][r], H)
    for i, r in enumerate(reversed(rows)):
        m, acc = r.stop - r.start, "f32" if i == 0 else "acc_f32"
        a, g, da, dy = st["a"][r], st["g"][r], st["da"][r], st["dy"][r]
        L.sppo_gemm_bf16("nt", m, F, H, dy, H, st["w2"], H, da, F, "dgelu", a, F)
        L.sppo_gemm_bf16("tn", F, H, m, g, F, dy, H, st["dw2"], H, acc)
        L.sppo_gemm_bf16("nt", m, H, F, da, F, st["w1"], F, st["dz"][r], H)
        L.sppo_gemm_bf16("tn", H, F, m, st["z"][r], H, da, F, st["dw1"], F, acc)
    return {k: st[k] for k in ("a", "y", "dz", "dw1", "dw2")}


# ------------------------------------------------------------------- the work
def _pairs(c0, c1):
    return (c1 - c0) * c0 + (c1 - c0) * (c1 - c0 + 1) // 2


def work(case):
    kind = case["kind"]
    if kind in ("walk", "forward", "bwd_chunk"):
        B, S, Hq, Hkv, D = case.get("B", 1), case["S"], case["Hq"], case["Hkv"], case["D"]
        e = 4 if case.get("dtype") == "f32" else 2
        q, kv = B * S * Hq * D, B * S * Hkv * D
        if kind == "walk":
            # reads q, k, v, dO; writes o, lse, dq, fp32 dk, dv
            return {"bytes": e * (4 * q + 2 * kv) + 4 * B * S * Hq + 8 * kv, "flops": 14 * B * Hq * D * _pairs(0, S)}
        if kind == "forward":
            return {"bytes": e * (2 * q + 2 * kv) + 4 * B * S * Hq, "flops": 4 * B * Hq * D * _pairs(0, S)}
        n = case["rows"]
        return {"bytes": 2 * (4 * n * Hq * D + 2 * kv) + 4 * n * Hq + 8 * kv,
                "flops": 10 * Hq * D * _pairs(S - n, S)}
    if kind == "mlp":
        n, H = case["rows"], case["H"]
        # reads z, h, dy, W1, W2; writes a, y, dz, fp32 dW1, dW2
        return {"bytes": 2 * (9 * n * H + 8 * H * H) + 4 * 8 * H * H, "flops": 6 * 2 * n * 4 * H * H}
    if kind == "norm":
        n, H = case["rows"], case["H"]
        return {"bytes": 2 * 5 * n * H + 8 * n + 16 * H, "flops": 20 * n * H}
    S, Hq, Hkv, D = case["S"], case["Hq"], case["Hkv"], case["D"]
    H, w = Hq * D, Hq * D * ((Hq + 2 * Hkv) * D + Hq * D + 8 * Hq * D)
    return {"bytes": 2 * 4 * S * H + 2 * w + 4 * w, "flops": 6 * S * w + 14 * Hq * D * _pairs(0, S)}


def tolerance(case):
    """About four times the distance from `exact` measured on every output of the listed cases."""
    kind = case["kind"]
    if case.get("dtype") == "f32":
        return {"rel": 4e-6, "max": 2e-4}
    if kind == "norm":
        return {"rel": 7e-3, "max": 0.03}
    return {"rel": 2e-2 if kind in ("mlp", "layer") else 1e-2, "max": 0.3}


# ------------------------------------------------------------------- 64 bits
def _attention64(q, k, v, do, c0=0, block=1024):
    """Causal attention of rows [c0, c0 + n) of one batch entry in 64 bits: o, lse and, with do, dq, dk, dv."""
    n, Hq, D = q.shape
    S, Hkv = k.shape[0], k.shape[1]
    G, scale = Hq // Hkv, 1 / math.sqrt(D)
    z = lambda *s: torch.zeros(s, device=q.device, dtype=F64)  # noqa: E731
    o, lse, dq, dk, dv = z(n, Hq, D), z(Hq, n), z(n, Hq, D), z(S, Hkv, D), z(S, Hkv, D)
    for h in range(Hq):
        kh, vh = k[:, h // G].to(F64), v[:, h // G].to(F64)
        for r0 in range(0, n, block):
            r1 = min(n, r0 + block)
            kend = c0 + r1
            qb = q[r0:r1, h].to(F64)
            s = qb @ kh[:kend].t() * scale
            rows = torch.arange(c0 + r0, c0 + r1, device=q.device)[:, None]
            s.masked_fill_(torch.arange(kend, device=q.device)[None, :] > rows, -math.inf)
            le = torch.logsumexp(s, dim=1)
            p = torch.exp(s - le[:, None])
            ob = p @ vh[:kend]
            o[r0:r1, h], lse[h, r0:r1] = ob, le
            if do is None:
                continue
            db = do[r0:r1, h].to(F64)
            ds = p * (db @ vh[:kend].t() - (ob * db).sum(1, keepdim=True))
            dq[r0:r1, h] = ds @ kh[:kend] * scale
            dk[:kend, h // G] += ds.t() @ qb * scale
            dv[:kend, h // G] += p.t() @ db
    return o, lse, dq, dk, dv


def _gelu64(a):
    return 0.5 * a * (1 + torch.tanh(math.sqrt(2 / math.pi) * (a + 0.044715 * a ** 3)))


def _gelu64_grad(a):
    t = torch.tanh(math.sqrt(2 / math.pi) * (a + 0.044715 * a ** 3))
    return 0.5 * (1 + t) + 0.5 * a * (1 - t * t) * math.sqrt(2 / math.pi) * (1 + 3 * 0.044715 * a * a)


def _ln64(x, g, b):
    mean = x.mean(1, keepdim=True)
    rstd = 1 / torch.sqrt(((x - mean) ** 2).mean(1, keepdim=True) + 1e-5)
    xh = (x - mean) * rstd
    return xh * g + b, xh, mean, rstd


def _ln64_bwd(dy, xh, rstd, g):
    gg = dy * g
    dx = rstd * (gg - gg.mean(1, keepdim=True) - xh * (gg * xh).mean(1, keepdim=True))
    return dx, (dy * xh).sum(0), dy.sum(0)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("walk", "forward", "bwd_chunk") and work(case)["flops"] > 1.3e14:
        return None
    if kind in ("walk", "forward"):
        B, S, N, Hq, Hkv, D = case.get("B", 1), case["S"], case["N"], case["Hq"], case["Hkv"], case["D"]
        inp = _attn_inputs(B, S, Hq, Hkv, D, F32 if case.get("dtype") == "f32" else BF, seed, do=kind == "walk")
        got = [_attention64(inp["q"][b], inp["k"][b], inp["v"][b], inp["do"][b] if kind == "walk" else None)
               for b in range(B)]
        o, lse, dq, dk, dv = (torch.stack([g[i] for g in got]) for i in range(5))
        off = _offsets(S, N, case.get("ragged", False))
        res = {"o": o, "lse": [lse[:, :, off[i]:off[i + 1]].contiguous() for i in range(N)]}
        return dict(res, dq=dq, dk=dk, dv=dv) if kind == "walk" else res
    if kind == "bwd_chunk":
        S, n = case["S"], case["rows"]
        inp = _attn_inputs(1, S, case["Hq"], case["Hkv"], case["D"], BF, seed)
        _, _, dq, dk, dv = _attention64(inp["q"][0, S - n:], inp["k"][0], inp["v"][0], inp["do"][0, S - n:], S - n)
        return {"dq": dq, "dk": dk, "dv": dv}
    if kind == "mlp":
        t = {k: v.to(F64) for k, v in _mlp_inputs(case, seed).items()}
        a = t["z"] @ t["w1"]
        g = _gelu64(a)
        y = t["h"] + g @ t["w2"]
        da = (t["dy"] @ t["w2"].t()) * _gelu64_grad(a)
        return {"a": a, "y": y, "dz": da @ t["w1"].t(), "dw1": t["z"].t() @ da, "dw2": g.t() @ t["dy"]}
    if kind == "norm":
        t = {k: v.to(F64) for k, v in _norm_inputs(case, seed).items()}
        y, xh, mean, rstd = _ln64(t["x"], t["g"], t["b"])
        dx, dg, db = _ln64_bwd(t["dy"], xh, rstd, t["g"])
        return {"y": y, "mean": mean[:, 0], "rstd": rstd[:, 0], "dx": dx + t["dres"], "dg": dg, "db": db}
    return _layer64(case, seed)


def _layer64(case, seed):
    S, Hq, Hkv, D = case["S"], case["Hq"], case["Hkv"], case["D"]
    inp, p = _layer_inputs(case, seed)
    x, dy = inp["x"].to(F64), inp["dy"].to(F64)
    p = {k: v.to(F64) for k, v in p.items()}
    nq, nkv = Hq * D, Hkv * D
    u, xh1, _, r1 = _ln64(x, p["g1"], p["b1"])
    qkv = u @ p["w_qkv"]
    q, k, v = qkv[:, :nq].reshape(S, Hq, D), qkv[:, nq:nq + nkv].reshape(S, Hkv, D), qkv[:, nq + nkv:].reshape(S, Hkv, D)
    o = _attention64(q, k, v, None)[0].reshape(S, nq)
    h = x + o @ p["w_o"]
    z, xh2, _, r2 = _ln64(h, p["g2"], p["b2"])
    a = z @ p["w_1"]
    g = _gelu64(a)
    y = h + g @ p["w_2"]
    da = (dy @ p["w_2"].t()) * _gelu64_grad(a)
    dw_2, dw_1 = g.t() @ dy, z.t() @ da
    dz, dg2, db2 = _ln64_bwd(da @ p["w_1"].t(), xh2, r2, p["g2"])
    del a, g, z, da
    dh = dy + dz
    dO, dw_o = dh @ p["w_o"].t(), o.t() @ dh
    _, _, dq, dk, dv = _attention64(q, k, v, dO.reshape(S, Hq, D))
    dqkv = torch.cat([dq.reshape(S, nq), dk.reshape(S, nkv), dv.reshape(S, nkv)], dim=1)
    dw_qkv = u.t() @ dqkv
    dx, dg1, db1 = _ln64_bwd(dqkv @ p["w_qkv"].t(), xh1, r1, p["g1"])
    return {"y": y, "dx": dx + dh, "dw_qkv": dw_qkv, "dw_o": dw_o, "dw_1": dw_1, "dw_2": dw_2, "dg1": dg1, "db1": db1,
            "dg2": dg2, "db2": db2}
