"""Performance cases of the merged-retrieval library.

What programs have the library do, through its public entry points, from the
smallest window (32 requests over 4,096 chunks) to the largest single-GPU
workloads (4M x 1024 bf16, 20M x 768 fp8).  Four kinds of program:

  window   one merge window: hs_dedup -> representative rows -> score + top-k
           -> delivery (MergedRetrieval.run), for each corpus type and layout;
  reuse    successive windows of one traffic stream over a result store that
           starts empty (MergedRetrieval.run_cached);
  chunks   chunk-id dedup and the gather of the distinct embedding rows;
  ingest   a scheduler's intake: node texts -> signatures -> dedup ->
           priorities and ready-queue order.

listed() names the cases, draw(rng) draws further ones from the same ranges,
prepare(case, seed) makes a state on the GPU, run(state) is one pass,
work(case) the bytes and operations a pass cannot do without, tolerance(case)
what another correct implementation may differ by and exact(case, seed) the
results in 64 bits from plain torch and hashlib.
"""
import hashlib
import math
import struct

import numpy as np
import torch

import paper_2607_22578_amd as hs

DEVICE = "cuda"
CODES = {"f32": hs.HS_F32, "bf16": hs.HS_BF16, "fp8": hs.HS_FP8_E4M3}
ROW_BYTES = {"f32": 4, "bf16": 2, "fp8": 1}
WEIGHTS = 2.0, 0.75, 5.0, 0.25   # alpha, gamma, delta, eps of the priority function
SHA_OPS_PER_BLOCK = 2296   # 32-bit operations of one SHA-256 block (FIPS 180-4)


def _window(name, dtype, layout, requests, pool, zipf, dim, corpus, k):
    return {"name": name, "kind": "window", "dtype": dtype, "layout": layout,
            "requests": requests, "pool": pool, "zipf": zipf, "dim": dim, "corpus": corpus,
            "k": k}


def listed():
    return [
        # A handful of workflows over a small fp32 collection: launches and latency.
        _window("tiny_f32", "f32", "rows", 32, 24, 0.5, 384, 4_096, 10),
        # An unquantised fp32 store (the type pgvector keeps) under ordinary traffic.
        _window("store_f32", "f32", "rows", 512, 256, 1.1, 768, 200_000, 10),
        # Few concurrent requests over the 1M-chunk index: the corpus is streamed once.
        _window("few_1m_bf16", "bf16", "tiled", 24, 512, 1.1, 768, 1_000_000, 10),
        # The ordinary window: 64 workflows x 32 queries over the 1M-chunk index.
        _window("window_1m_bf16", "bf16", "tiled", 2_048, 512, 1.1, 768, 1_000_000, 10),
        # A row-major bf16 corpus that is appended to (not tiled), odd sizes throughout.
        _window("rows_ragged_bf16", "bf16", "rows", 777, 1_000, 0.9, 1_000, 333_333, 20),
        # The largest bf16 window: 512 workflows x 64 queries over 4M chunks.
        _window("window_4m_bf16", "bf16", "tiled", 32_768, 16_384, 0.8, 1_024, 4_000_000, 32),
        # A mid-size quantised index, odd row count, deep result lists for a reranker.
        _window("mid_fp8", "fp8", "tiled", 3_000, 2_000, 0.9, 400, 500_009, 50),
        # The largest index of one GPU: 20M fp8 rows, k = 100.
        _window("window_20m_fp8", "fp8", "tiled", 16_384, 4_096, 1.1, 768, 20_000_000, 100),
        # Three successive windows of one stream over a store that starts empty: the first is
        # all misses, the later ones score only what has not been seen.
        {"name": "reuse_3_windows", "kind": "reuse", "dtype": "bf16", "layout": "tiled",
         "requests": 2_048, "pool": 512, "zipf": 1.1, "dim": 768, "corpus": 1_000_000, "k": 10,
         "windows": 3, "store": 4_096},
        # 1,024 workflows x 256 chunk ids: each distinct chunk's embedding is fetched once.
        {"name": "chunks_256k", "kind": "chunks", "requests": 262_144, "pool": 200_000,
         "zipf": 1.0, "dim": 1_024},
        # A scheduler's intake of one ordinary window.
        {"name": "ingest_2k", "kind": "ingest", "requests": 2_048, "pool": 512, "zipf": 1.1,
         "chars": 70, "k": 10},
        # The intake of a whole burst: 200,000 nodes, most of them distinct texts.
        {"name": "ingest_200k", "kind": "ingest", "requests": 200_000, "pool": 150_000,
         "zipf": 0.6, "chars": 70, "k": 10},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges: sizes over their logarithm, odd ones among them."""
    kind = rng.choice(["window"] * 7 + ["reuse", "chunks", "ingest", "ingest"])
    zipf = round(rng.uniform(0.5, 1.2), 2)
    if kind == "chunks":
        return {"kind": kind, "requests": _log(rng, 500, 262_144), "pool": _log(rng, 300, 200_000),
                "zipf": zipf, "dim": 8 * rng.randint(16, 128)}
    if kind == "ingest":
        return {"kind": kind, "requests": _log(rng, 500, 200_000), "pool": _log(rng, 200, 150_000),
                "zipf": zipf, "chars": _log(rng, 40, 300), "k": _log(rng, 5, 100)}
    dtype = "bf16" if kind == "reuse" else rng.choice(["f32", "bf16", "bf16", "fp8", "fp8"])
    step = {"f32": 4, "bf16": 8, "fp8": 16}[dtype]
    case = {"kind": kind, "dtype": dtype,
            "layout": "rows" if dtype == "f32" else rng.choice(["rows", "tiled", "tiled"]),
            "requests": _log(rng, 16, 8_192), "pool": _log(rng, 16, 8_192), "zipf": zipf,
            "dim": step * rng.randint(128 // step, 1_024 // step),
            "corpus": _log(rng, 2_000, {"f32": 300_000, "bf16": 2_000_000, "fp8": 6_000_000}[dtype]),
            "k": _log(rng, 8, 100 if dtype == "fp8" else 40)}
    if kind == "reuse":
        case.update(windows=3, store=1 << rng.randint(8, 14))
    # no drawn case costs more than the largest listed one
    most = {"f32": 4e11, "bf16": 1e13, "fp8": 1e13}[dtype]
    flops = 2.0 * _distinct(case) * case["corpus"] * case["dim"]
    if flops > most:
        case["corpus"] = max(2_000, int(case["corpus"] * most / flops))
    return case


# ------------------------------------------------------------------ inputs

def _shares(case):
    """Zipf law over the templates: each one's share of the requests."""
    w = np.arange(1, case["pool"] + 1, dtype=np.float64) ** (-case["zipf"])
    return w / w.sum()


def _distinct(case):
    """Expected number of distinct templates among a window's requests."""
    return float((1.0 - (1.0 - _shares(case)) ** case["requests"]).sum())


def _rng(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    return g


def _templates(case, g, windows=1):
    """Template ids of `windows` windows' requests: Zipf ranks through one permutation."""
    cdf = torch.from_numpy(np.cumsum(_shares(case))).to(DEVICE)
    perm = torch.randperm(case["pool"], device=DEVICE, generator=g)
    u = torch.rand(windows, case["requests"], dtype=torch.float64, device=DEVICE, generator=g)
    return perm[torch.searchsorted(cdf, u).clamp_(max=case["pool"] - 1)]


def _keys(case, g):
    """A 64-bit signature per template, over the whole signed range."""
    return torch.randint(-(1 << 63), (1 << 63) - 1, (case["pool"],), device=DEVICE, generator=g)


def _unit_rows(n, dim, g):
    x = torch.randn(n, dim, device=DEVICE, generator=g)
    return x.div_(x.norm(dim=1, keepdim=True))


def _corpus(case, g):
    """(rows, scale): unit-norm Gaussian rows in the corpus type, fp8 with a scale per row."""
    n, dim, dtype = case["corpus"], case["dim"], case["dtype"]
    kind = {"f32": torch.float32, "bf16": torch.bfloat16, "fp8": torch.uint8}[dtype]
    rows = torch.empty(n, dim, dtype=kind, device=DEVICE)
    scale = torch.empty(n, dtype=torch.float32, device=DEVICE) if dtype == "fp8" else None
    step = max(1, (1 << 28) // dim)
    for a in range(0, n, step):
        x = _unit_rows(min(step, n - a), dim, g)
        if scale is not None:
            s = x.abs().amax(dim=1) / 448.0
            scale[a:a + step] = s
            x = x.div_(s[:, None]).to(torch.float8_e4m3fn).view(torch.uint8)
        rows[a:a + step] = x
    return rows, scale


def _retrieval_inputs(case, seed):
    g = _rng(seed)
    ids = _templates(case, g, case.get("windows", 1))
    keys = _keys(case, g)
    q = _unit_rows(case["pool"], case["dim"], g)
    if case["dtype"] != "f32":
        q = q.bfloat16()
    windows = [(keys[t], q[t]) for t in ids]
    return windows, *_corpus(case, g)


def _node_texts(case, g):
    """Query texts: a pool of templates of lower-case words; a node renders its template with
    its own case flips, tabs for blanks and leading blanks.  (bytes, offsets, template ids)"""
    n, pool = case["requests"], case["pool"]
    ids = _templates(case, g)[0]
    size = torch.randint(max(8, case["chars"] // 3), case["chars"] * 5 // 3 + 1, (pool,),
                         device=DEVICE, generator=g)
    start = size.cumsum(0) - size
    letters = torch.randint(97, 123, (int(size.sum()),), device=DEVICE, generator=g)
    blank = torch.rand(letters.shape, device=DEVICE, generator=g) < 1 / 6
    letters = torch.where(blank, 32, letters)
    lead = torch.randint(-6, 4, (n,), device=DEVICE, generator=g).clamp_(min=0)
    lens = lead + size[ids]
    off = torch.zeros(n + 1, dtype=torch.int64, device=DEVICE)
    off[1:] = lens.cumsum(0)
    node = torch.repeat_interleave(torch.arange(n, device=DEVICE), lens)
    at = torch.arange(node.numel(), device=DEVICE) - off[node] - lead[node]
    c = torch.where(at < 0, 32, letters[(start[ids[node]] + at).clamp_(min=0)])
    flip = torch.rand(c.shape, device=DEVICE, generator=g) < 0.15
    c = torch.where(flip & (c != 32), c - 32, torch.where(flip, 9, c))
    return c.to(torch.uint8), off, ids


def _node_inputs(case, seed):
    g = _rng(seed)
    n = case["requests"]
    text, off, _ = _node_texts(case, g)
    some = torch.tensor([0.5, 1.0, 2.0, 4.0], device=DEVICE)
    phi = torch.where(torch.rand(n, device=DEVICE, generator=g) < 0.5,
                      some[torch.randint(0, 4, (n,), device=DEVICE, generator=g)],
                      torch.rand(n, device=DEVICE, generator=g) * 50)
    flows = torch.arange(n, device=DEVICE) // 32          # 32 nodes per workflow
    m = n // 32 + 1
    s_hat = (0.1 + 19.9 * torch.rand(m, device=DEVICE, generator=g))[flows]
    heavy = (torch.rand(m, device=DEVICE, generator=g) < 0.15).to(torch.uint8)[flows]
    return {"text": text, "text_off": off, "phi": phi, "s_hat": s_hat, "heavy": heavy,
            "op": torch.full((n,), 2, dtype=torch.int32, device=DEVICE),
            "params": torch.from_numpy(np.full(n, case["k"], "<u4").view(np.uint8)).to(DEVICE),
            "param_off": torch.arange(0, 4 * (n + 1), 4, dtype=torch.int64, device=DEVICE)}


def _chunk_inputs(case, seed):
    g = _rng(seed)
    ids = _templates(case, g)[0]
    return ids, _unit_rows(case["pool"], case["dim"], g).bfloat16()


# ------------------------------------------------------------------ the cases' programs

# The number of groups stays on the device, so per-group outputs are returned whole: buffers of
# one entry per request that start as zeros and of which a pass writes the first n_u entries.

def prepare(case, seed):
    if case["kind"] == "chunks":
        ids, table = _chunk_inputs(case, seed)
        n = case["requests"]
        plan = hs.hs_merge_plan(n, case["dim"], case["pool"], 1, hs.HS_BF16, hs.HS_BF16)
        new = lambda dtype, *shape: torch.zeros(shape, dtype=dtype, device=DEVICE)  # noqa: E731
        return {"kind": "chunks", "case": case, "plan": plan, "ids": ids, "table": table,
                "ws": new(torch.uint8, max(plan.workspace_bytes, 256)),
                "unique": new(torch.int64, n), "first": new(torch.int32, n),
                "counts": new(torch.int32, n), "inverse": new(torch.int32, n),
                "n_unique": torch.zeros(1, dtype=torch.int64, device=DEVICE),
                "rows": new(torch.bfloat16, n, case["dim"])}
    if case["kind"] == "ingest":
        state = _node_inputs(case, seed)
        n = case["requests"]
        state.update(kind="ingest", n=n,
                     digest=torch.empty((n, 32), dtype=torch.uint8, device=DEVICE),
                     keys=torch.empty(n, dtype=torch.int64, device=DEVICE),
                     engine=hs.MergedRetrieval(n, 8, 1, 1, hs.HS_BF16, hs.HS_BF16))
        m = state["engine"]
        m.first_index.zero_()
        m.counts.zero_()
        state.update({name: torch.zeros(n, dtype=dtype, device=DEVICE) for name, dtype in
                      (("phi_fused", torch.float64), ("pi", torch.float64),
                       ("order", torch.int32))})
        return state
    tiled = case["layout"] == "tiled"
    windows, rows, scale = _retrieval_inputs(case, seed)
    engine = hs.MergedRetrieval(case["requests"], case["dim"], case["corpus"], case["k"],
                                hs.HS_F32 if case["dtype"] == "f32" else hs.HS_BF16,
                                CODES[case["dtype"]], tiled_corpus=tiled)
    corpus = engine.tile_corpus(rows) if tiled else rows
    state = {"kind": case["kind"], "engine": engine, "windows": windows, "corpus": corpus,
             "scale": scale}
    if case["kind"] == "reuse":
        engine.enable_cache(case["store"])
        # each window's results in buffers of its own
        state["results"] = [(torch.empty_like(engine.out_score),
                             torch.empty_like(engine.out_index)) for _ in windows]
    return state


def run(s):
    if s["kind"] == "window":
        m = s["engine"]
        keys, q = s["windows"][0]
        m.run(keys, q, s["corpus"], s["scale"])
        return {"score": m.out_score, "index": m.out_index, "inverse": m.inverse}
    if s["kind"] == "reuse":
        m = s["engine"]
        hs.hs_cache_reset(m.plan, m.cache, m.cache_capacity)
        for (keys, q), (m.out_score, m.out_index) in zip(s["windows"], s["results"]):
            m.run_cached(keys, q, s["corpus"], s["scale"])
        return {"score": [r[0] for r in s["results"]], "index": [r[1] for r in s["results"]],
                "inverse": m.inverse}
    if s["kind"] == "chunks":
        c = s["case"]
        hs.hs_dedup(s["plan"], s["ids"], s["unique"], s["first"], s["counts"], s["inverse"],
                    s["n_unique"], None, s["ws"])
        hs.hs_scatter(s["table"], c["pool"], c["dim"] * 2, s["unique"], 1, c["requests"],
                      s["n_unique"], s["rows"])
        return {name: s[name] for name in ("unique", "first", "counts", "inverse", "n_unique",
                                           "rows")}
    m, n = s["engine"], s["n"]
    hs.hs_signature(s["op"], n, 0, n, s["digest"], s["keys"], params=s["params"],
                    param_off=s["param_off"], text=s["text"], text_off=s["text_off"],
                    flags=hs.HS_SIG_NORMALIZE_TEXT)
    m.dedup(s["keys"])
    hs.hs_priority(m.plan, m.inverse, m.first_index, -1, m.n_unique, s["phi"], s["s_hat"],
                   s["heavy"], *WEIGHTS, s["phi_fused"], s["pi"], s["order"], m.ws)
    return {"digest": s["digest"], "keys": s["keys"], "first": m.first_index,
            "counts": m.counts, "inverse": m.inverse, "n_unique": m.n_unique,
            "phi_fused": s["phi_fused"], "pi": s["pi"], "order": s["order"]}


# ------------------------------------------------------------------ what a pass cannot do without

def work(case):
    n, u = case["requests"], _distinct(case)
    if case["kind"] == "chunks":
        return {"bytes": 12 * n + u * (16 + 4 * case["dim"]), "flops": 0}
    if case["kind"] == "ingest":
        blocks = max(1.0, (case["chars"] + 20 + 9) / 64)
        return {"bytes": n * (case["chars"] + 16 + 4 + 4 + 40 + 4 + 9) + u * (8 + 16 + 4),
                "flops": n * blocks * SHA_OPS_PER_BLOCK}
    dim, rows, k = case["dim"], case["corpus"], case["k"]
    corpus = rows * (dim * ROW_BYTES[case["dtype"]] + (4 if case["dtype"] == "fp8" else 0))
    q = dim * (4 if case["dtype"] == "f32" else 2)
    passes, scored = 1, u
    if case["kind"] == "reuse":   # every template is scored once, the corpus read per window
        passes = case["windows"]
        scored = _distinct(dict(case, requests=passes * n))
    return {"bytes": passes * (corpus + 12 * n + 8 * n * k) + scored * q,
            "flops": 2.0 * scored * rows * dim}


def tolerance(case):
    """Scores are sums of up to 1,024 products in 32 bits: other orders of summation differ by
    a few 1e-7 (measured against 64 bits: 4.4e-7 for fp32 rows, 1.8e-7 for bf16, 0.9e-7 for
    fp8; largest 1.7e-6); neighbours in a result list whose scores differ by less than that
    may change places (measured: 0.12 % of the rows).  Everything else is whole numbers, copies or exactly rounded."""
    if case["kind"] in ("window", "reuse"):
        return {"rel": 2e-6, "max": 1e-5, "differ": 0.01}
    return "exact"


# ------------------------------------------------------------------ results in 64 bits

def _best(q, rows, scale, k):
    """(score, row) of the k best rows per query, exact inner products in 64 bits."""
    n, corpus = q.shape[0], rows.shape[0]
    best = torch.full((n, k), -math.inf, dtype=torch.float64, device=DEVICE)
    at = torch.full((n, k), -1, dtype=torch.int64, device=DEVICE)
    q = q.double()
    step = max(64, (1 << 27) // max(n, rows.shape[1]) // 64 * 64)
    for a in range(0, corpus, step):
        c = rows[a:a + step]
        c = (c.view(torch.float8_e4m3fn).float() if scale is not None else c).double()
        if scale is not None:
            c *= scale[a:a + step, None].double()
        s = q @ c.T
        row = torch.arange(a, a + c.shape[0], device=DEVICE).expand(n, -1)
        if s.shape[1] % 64 == 0 and s.shape[1] // 64 > k:
            # the k best lie in the k blocks of 64 with the largest maxima
            block = s.view(n, -1, 64).amax(2).topk(k, dim=1).indices
            pick = (block[:, :, None] * 64 + torch.arange(64, device=DEVICE)).view(n, -1)
            s, row = s.gather(1, pick), row.gather(1, pick)
        s, row = torch.cat([best, s], 1), torch.cat([at, row], 1)
        best, pick = s.topk(k, dim=1)
        at = row.gather(1, pick)
    return best, at


def _groups(keys, n):
    """(unique, first, counts, inverse, n_u) of n keys; the per-group ones padded with zeros."""
    unique, inverse, counts = torch.unique(keys, return_inverse=True, return_counts=True)
    first = torch.full_like(unique, n).scatter_reduce_(
        0, inverse, torch.arange(n, device=DEVICE), "amin")
    return unique, first, counts, inverse, unique.numel()


def _padded(x, n):
    out = torch.zeros((n,) + x.shape[1:], dtype=x.dtype, device=x.device)
    out[:x.shape[0]] = x
    return out


def _exact_window(keys, q, rows, scale, k):
    _, first, _, inverse, _ = _groups(keys, keys.numel())
    score, row = _best(q[first], rows, scale, k)
    return score[inverse], row[inverse].int(), inverse.int()


def exact(case, seed):
    if case["kind"] in ("window", "reuse"):
        windows, rows, scale = _retrieval_inputs(case, seed)
        got = [_exact_window(keys, q, rows, scale, case["k"]) for keys, q in windows]
        if case["kind"] == "window":
            return {"score": got[0][0], "index": got[0][1], "inverse": got[0][2]}
        return {"score": [g[0] for g in got], "index": [g[1] for g in got],
                "inverse": got[-1][2]}
    if case["kind"] == "chunks":
        ids, table = _chunk_inputs(case, seed)
        n = case["requests"]
        unique, first, counts, inverse, n_u = _groups(ids, n)
        return {"unique": _padded(unique, n), "first": _padded(first.int(), n),
                "counts": _padded(counts.int(), n), "inverse": inverse.int(),
                "n_unique": torch.tensor([n_u]), "rows": _padded(table[unique], n)}
    s = _node_inputs(case, seed)
    text, off = s["text"].cpu().numpy().tobytes(), s["text_off"].tolist()
    param = struct.pack("<I", case["k"])
    head = struct.pack("<II", 2, 4) + param
    digests = []
    for a, b in zip(off, off[1:]):
        t = b" ".join(text[a:b].lower().split())
        digests.append(hashlib.sha256(head + struct.pack("<I", len(t)) + t
                                      + struct.pack("<I", 0)).digest())
    digest = np.frombuffer(b"".join(digests), np.uint8).reshape(-1, 32)
    keys = torch.from_numpy(digest[:, :8].copy().view(">i8").astype(np.int64)[:, 0]).to(DEVICE)
    n = case["requests"]
    unique, first, counts, inverse, n_u = _groups(keys, n)
    alpha, gamma, delta, eps = WEIGHTS
    units = (s["phi"].double() * 2.0 ** 24).long()     # truncated to multiples of 2^-24
    fused = torch.zeros_like(unique).scatter_add_(0, inverse, units).double() * 2.0 ** -24
    pi = (alpha / (s["s_hat"][first].double() + eps) + gamma * fused) \
        + delta * s["heavy"][first].double()
    order = torch.sort(-pi, stable=True).indices
    return {"digest": torch.from_numpy(digest.copy()), "keys": keys,
            "first": _padded(first.int(), n), "counts": _padded(counts.int(), n),
            "inverse": inverse.int(), "n_unique": torch.tensor([n_u]),
            "phi_fused": _padded(fused, n), "pi": _padded(pi, n),
            "order": _padded(order.int(), n)}
