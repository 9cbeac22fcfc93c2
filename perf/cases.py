"""What is measured: the calls a RAG server makes, over the sizes it makes them at.

A request selects the cache slots to recompute (from a [Q_a, T] attention block, or straight from
the auxiliary model's batched attention tensors), assembles every layer's cache from the per-chunk
caches, and recomputes the selected rows layer by layer.  A case is one of these calls at one size
(`kind` select, blocks, assemble, layer) or a whole small request (`kind` request).  Layer shapes
are those of `workloads/configs.py` and a d = 2048 layer with head dim 64.
"""
from __future__ import annotations

import random

import torch

import paper_2510_10129_amd as cc

DEV = "cuda:0"

#        d, H_q, H_kv, d_h, f, rope_base, rms_eps, qkv_bias
MODELS = {
    "d256": (256, 4, 2, 64, 1024, 1.0e4, 1e-5, False),
    "d2048": (2048, 32, 8, 64, 8192, 5.0e5, 1e-5, False),
    "d3584": (3584, 28, 4, 128, 18944, 1.0e6, 1e-6, True),
    "d4096": (4096, 32, 8, 128, 14336, 5.0e5, 1e-5, False),
    "d8192": (8192, 64, 8, 128, 28672, 5.0e5, 1e-5, False),
}


def listed():
    return [
        # a whole request on the smallest model: selection with its one host wait, two layers'
        # caches assembled, two layers recomputed; launches and latency are all there is
        dict(name="request_1k", kind="request", model="d256", layers=2, P=16, chunks=4, chunk_len=256, ragged=False,
             Q=32, bp=2000, window=8),
        # selection of a 16k-context request, the row count awaited on the host (what a server does
        # before it sizes the layer launches)
        dict(name="select_16k", kind="select", T=16384, Q_a=128, P=64, Q=128, bp=2000, window=16, noalloc=False),
        # selection at 64k context for callers that enqueue only (no context, no host wait)
        dict(name="select_64k", kind="select", T=65536, Q_a=256, P=64, Q=256, bp=2000, window=32, noalloc=True),
        # selection straight from a 14-head auxiliary model's batched attention tensors, 16 chunks
        dict(name="blocks_16k", kind="blocks", heads=14, P=64, chunks=16, chunk_len=1024, ragged=False, Q=128, bp=2000,
             window=16),
        # cache assembly of one layer, 32 ragged chunks, few kv heads
        dict(name="assemble_29k", kind="assemble", model="d3584", P=64, chunks=32, chunk_len=896, ragged=True, Q=128),
        # cache assembly of one layer at 64k context
        dict(name="assemble_64k", kind="assemble", model="d8192", P=64, chunks=64, chunk_len=1024, ragged=False, Q=256),
        # nothing recomputed but the user's query (recompute ratio 0, plain concatenation): few rows
        # against a whole layer's weights
        dict(name="layer_4k_tail", kind="layer", model="d4096", P=64, chunks=8, chunk_len=512, ragged=False, Q=64,
             bp=0, window=16, gather=False),
        # short context, one layer at the usual ratio, first layer (rows gathered by index)
        dict(name="layer_4k_20", kind="layer", model="d4096", P=64, chunks=8, chunk_len=512, ragged=False, Q=64,
             bp=2000, window=16, gather=True),
        # the benchmark's layer: 16k context at 20 %
        dict(name="layer_16k_20", kind="layer", model="d4096", P=64, chunks=16, chunk_len=1024, ragged=False, Q=128,
             bp=2000, window=16, gather=False),
        # every slot of the same cache recomputed: full prefill on the same call
        dict(name="layer_16k_dense", kind="layer", model="d4096", P=64, chunks=16, chunk_len=1024, ragged=False, Q=128,
             bp=10000, window=16, gather=True),
        # long ragged context, few rows, groups of seven query heads, QKV bias
        dict(name="layer_29k_5", kind="layer", model="d3584", P=64, chunks=32, chunk_len=896, ragged=True, Q=128,
             bp=500, window=16, gather=False),
        # one wide layer at 64k context: the largest call
        dict(name="layer_64k_20", kind="layer", model="d8192", P=64, chunks=64, chunk_len=1024, ragged=False, Q=256,
             bp=2000, window=32, gather=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    """A call of the same kinds: contexts of 256 to 65k tokens, ratios from none to all, any window."""
    most = max(work(c)["flops"] for c in listed())
    while True:
        kind = rng.choices(("request", "select", "blocks", "assemble", "layer"), (1, 2, 1, 1, 6))[0]
        window = rng.choice((4, 8, 16, 32))
        P, Q = rng.choice((0, 16, 64)), _log_int(rng, 16, 256)
        bp = rng.choice((0, 10000, _log_int(rng, 200, 10000), _log_int(rng, 200, 10000), _log_int(rng, 200, 10000)))
        T = _log_int(rng, 256, 65536)
        chunk_len = min(T, _log_int(rng, 128, 1536))
        lay = dict(P=P, chunks=max(1, T // chunk_len), chunk_len=chunk_len, ragged=rng.random() < 0.5, Q=Q)
        if kind == "select":
            return dict(kind=kind, T=T, Q_a=_log_int(rng, 16, 256), P=P, Q=Q, bp=rng.randint(300, 6000), window=window,
                        noalloc=rng.random() < 0.5)
        if kind == "blocks":
            c = dict(kind=kind, heads=rng.choice((4, 12, 14, 16)), bp=rng.randint(300, 6000), window=window, **lay)
            if work(c)["bytes"] < 4e8:
                return c
        elif kind == "assemble":
            return dict(kind=kind, model=rng.choice(sorted(MODELS)), **lay)
        elif kind == "request":
            c = dict(kind=kind, model=rng.choice(("d256", "d2048")), layers=rng.randint(1, 3), bp=rng.randint(300, 6000),
                     window=window, **lay)
            if _tokens(c) <= 4096:
                return c
        else:
            c = dict(kind=kind, model=rng.choice(sorted(MODELS)), bp=bp, window=window, gather=rng.random() < 0.5, **lay)
            if work(c)["flops"] < 0.5 * most:
                return c


# ---- sizes ----

def _chunk_lens(c):
    n, L = c["chunks"], c["chunk_len"]
    if not c["ragged"]:
        return [L] * n
    r = random.Random(n * 100003 + L)
    return [max(1, r.randint(L // 2, L + L // 2)) for _ in range(n)]


def _tokens(c):
    return c["T"] if c["kind"] == "select" else sum(_chunk_lens(c))


def _rows(c):
    """Rows that a layer case recomputes: the ratio's share of the chunk tokens and the query (all
    slots when the ratio is 100 %)."""
    T = _tokens(c)
    return c["P"] + T + c["Q"] if c["bp"] >= 10000 else T * c["bp"] // 10000 + c["Q"]


def _layer_idx(c, seed):
    """A selected set: runs of `window` tokens at random places, exactly the ratio's share, then the query."""
    T, P, Q, w = _tokens(c), c["P"], c["Q"], c["window"]
    if c["bp"] >= 10000:
        return list(range(P + T + Q))
    k = T * c["bp"] // 10000
    r = random.Random(seed * 1000003 + T)
    slots = sorted(r.sample(range(-(-T // w)), min(-(-T // w), -(-k // w) + 1)))
    sel = [t for s in slots for t in range(s * w, min(T, s * w + w))]
    drop = len(sel) - k
    sel = sel[drop // 2:len(sel) - (drop - drop // 2)]
    return [P + t for t in sel] + list(range(P + T, P + T + Q))


def _layer_work(m, M, N, keys, cache_rows_read):
    d, Hq, Hkv, dh, f = m[:5]
    nqkv = (Hq + 2 * Hkv) * dh
    weights = d * nqkv + Hq * dh * d + 3 * d * f
    flops = 2 * M * weights + 4 * dh * Hq * keys
    nbytes = 2 * weights + 2 * M * d * 2 + 2 * 2 * Hkv * dh * (cache_rows_read + M)
    return nbytes, flops


def work(case):
    c = case
    kind, T = c["kind"], _tokens(c)
    k = T * c.get("bp", 0) // 10000
    if kind == "select":
        return {"bytes": 4 * c["Q_a"] * T + 4 * (k + c["Q"]), "flops": c["Q_a"] * T}
    if kind == "blocks":
        return {"bytes": 4 * c["heads"] * c["Q"] * T + 4 * (k + c["Q"]), "flops": c["heads"] * c["Q"] * T}
    m = MODELS[c["model"]]
    row = m[2] * m[3] * 2
    N = c["P"] + T + c["Q"]
    if kind == "assemble":
        return {"bytes": 2 * row * (c["P"] + T + N), "flops": 3 * m[2] * m[3] * T}
    M = _rows(c)
    if c["bp"] >= 10000:
        keys = N * (N + 1) // 2
    else:      # the selected rows lie evenly over the chunks, the query rows at the end
        keys = int((M - c["Q"]) * (c["P"] + T / 2.0) + c["Q"] * (N - c["Q"] / 2.0))
    b, f = _layer_work(m, M, N, keys, N - M)
    if kind == "layer":
        return {"bytes": b, "flops": f}
    L = c["layers"]      # request: selection from the block, then the layers on caches it assembles
    return {"bytes": 4 * c["Q"] * T + L * (b + 2 * row * (c["P"] + T + N)), "flops": L * f}


# ---- inputs ----

class _Draw:
    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(seed)

    def normal(self, shape, std=1.0, mean=0.0, dtype=torch.bfloat16):
        x = torch.empty(shape, dtype=dtype, device=DEV)
        return x.normal_(mean, std, generator=self.g)


def _weights(r, m, layers):
    d, Hq, Hkv, dh, f, _, _, bias = m
    si = min(0.02, (2.0 / (5.0 * d)) ** 0.5)
    so = si / layers ** 0.5
    nqkv = (Hq + 2 * Hkv) * dh
    return cc.LayerWeights(
        w_in_norm=r.normal((d,), 0.1, 1.0), w_qkv=r.normal((nqkv, d), si), b_qkv=r.normal((nqkv,), 0.1) if bias else None,
        w_o=r.normal((d, Hq * dh), so), w_post_norm=r.normal((d,), 0.1, 1.0), w_gate=r.normal((f, d), si),
        w_up=r.normal((f, d), si), w_down=r.normal((d, f), so))


def _context(m, N, M, T):
    d, Hq, Hkv, dh, f, base, eps, _ = m
    return cc.Context(d, Hq, Hkv, dh, f, base, eps, N_cap=N, M_cap=M, T_cap=T)


def _attention(r, rows, cols, seed):
    """fp32 row softmax of 2 N(0,1) logits with bumps of +4 over runs of 4 to 24 columns (about a
    fifth of the columns) that all rows share: an attention map whose mass sits in runs of tokens."""
    z = r.normal((rows, cols), 2.0, dtype=torch.float32)
    p = random.Random(seed)
    bump = torch.zeros(cols)
    for _ in range(max(1, cols // 64)):
        s = p.randrange(cols)
        bump[s:s + p.randint(4, 24)] += 4.0
    return torch.softmax(z + bump.to(DEV), dim=1)


def _cache(r, m, N):
    return cc.KVLayer(r.normal((N, m[2], m[3]), 0.6), r.normal((N, m[2], m[3]), 0.6))


def _chunk_caches(r, m, c):
    rows = [c["P"] + L for L in _chunk_lens(c)]
    return [r.normal((n, m[2], m[3]), 0.6) for n in rows], [r.normal((n, m[2], m[3]), 0.6) for n in rows]


def prepare(case, seed):
    c, r = dict(case), _Draw(seed)
    T, P, Q = _tokens(c), c["P"], c["Q"]
    s = {"c": c, "T": T}
    N = P + T + Q
    if c["kind"] in ("select", "blocks"):
        s["idx"] = torch.zeros(T + Q, dtype=torch.int32, device=DEV)
        s["n"] = torch.zeros(1, dtype=torch.int32, device=DEV)
        if c["kind"] == "select":
            s["attn"] = _attention(r, c["Q_a"], T, seed)
        else:
            s["blocks"] = [(_attention(r, c["heads"] * Q, P + L + Q, seed + i).view(c["heads"], Q, P + L + Q), P, L)
                           for i, L in enumerate(_chunk_lens(c))]
        if not c.get("noalloc"):
            s["ctx"] = _context(MODELS["d256"], 64, 64, T)
        return s
    m = MODELS[c["model"]]
    if c["kind"] == "assemble":
        s["ctx"] = _context(m, N, 64, 64)
        s["cK"], s["cV"] = _chunk_caches(r, m, c)
        s["dst"] = cc.KVLayer(torch.zeros((N, m[2], m[3]), dtype=torch.bfloat16, device=DEV),
                              torch.zeros((N, m[2], m[3]), dtype=torch.bfloat16, device=DEV))
        return s
    if c["kind"] == "layer":
        idx = _layer_idx(c, seed)
        M = len(idx)
        s["M"] = M
        s["idx"] = torch.tensor(idx, dtype=torch.int32, device=DEV)
        s["ctx"] = _context(m, N, M, 64)
        s["w"] = _weights(r, m, 1)
        s["hidden"] = r.normal((N if c["gather"] else M, m[0]))
        s["kv"] = _cache(r, m, N)
        s["out"] = torch.zeros((M, m[0]), dtype=torch.bfloat16, device=DEV)
        return s
    L = c["layers"]
    s["ctx"] = _context(m, N, T + Q, T)
    s["attn"] = _attention(r, Q, T, seed)
    s["w"] = [_weights(r, m, L) for _ in range(L)]
    s["hidden"] = r.normal((N, m[0]))
    s["chunks"] = [_chunk_caches(r, m, c) for _ in range(L)]
    s["kv"] = [cc.KVLayer(torch.zeros((N, m[2], m[3]), dtype=torch.bfloat16, device=DEV),
                          torch.zeros((N, m[2], m[3]), dtype=torch.bfloat16, device=DEV)) for _ in range(L)]
    s["x"] = [torch.zeros((T + Q, m[0]), dtype=torch.bfloat16, device=DEV) for _ in range(2)]
    s["idx"] = torch.zeros(T + Q, dtype=torch.int32, device=DEV)
    s["n"] = torch.zeros(1, dtype=torch.int32, device=DEV)
    return s


# ---- one pass; index and row buffers come back whole, what lies past a request's rows stays zero ----

def run(s):
    c = s["c"]
    kind, P, Q = c["kind"], c["P"], c["Q"]
    if kind == "select" and c["noalloc"]:
        cc.select_noalloc(s["attn"], c["bp"], c["window"], 0, 0, P, Q, s["idx"], s["n"])
        return s["idx"], s["n"]
    if kind == "select":
        idx, _ = s["ctx"].select(s["attn"], c["bp"], c["window"], 0, 0, P, Q, s["idx"], s["n"])
        return idx, s["n"]
    if kind == "blocks":
        idx, _ = s["ctx"].select_blocks(s["blocks"], c["bp"], c["window"], 0, 0, P, Q, s["idx"], s["n"])
        return idx, s["n"]
    if kind == "assemble":
        s["ctx"].assemble_cache(s["cK"], s["cV"], P, Q, s["dst"])
        return s["dst"].K, s["dst"].V
    if kind == "layer":
        s["ctx"].recompute_layer(s["hidden"], s["idx"] if c["gather"] else None, s["kv"], s["idx"], s["M"], s["w"], s["out"])
        return s["out"], s["kv"].K, s["kv"].V
    ctx = s["ctx"]
    idx, M = ctx.select(s["attn"], c["bp"], c["window"], 0, 0, P, Q, s["idx"], s["n"])
    x = s["hidden"]
    for i, (w, kv, (cK, cV)) in enumerate(zip(s["w"], s["kv"], s["chunks"])):
        ctx.assemble_cache(cK, cV, P, Q, kv)
        ctx.recompute_layer(x, idx if i == 0 else None, kv, idx, M, w, s["x"][i % 2])
        x = s["x"][i % 2]
    return [idx, x] + [t for kv in s["kv"] for t in (kv.K, kv.V)]


def tolerance(case):
    kind = case["kind"]
    if kind in ("select", "blocks"):
        return "exact"
    if kind == "assemble":
        # one fp32 rotation rounded to bf16: a value on the edge of two codes may take either
        return {"rel": 1e-3, "max": 1e-2}
    # bf16 operands, fp32 sums, bf16 at every stage boundary: against the layer in 64 bits the
    # output differs by rel 1.9e-3 and K, V by 1.1e-3, single values by 1.2e-2; with the sums in
    # another order by 1.0e-3 and 1.2e-2
    return {"rel": 7e-3, "max": 4.5e-2}
