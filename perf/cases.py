"""The calls whose speed counts: what a user of the knowledge base has it do, through the Python binding.

A case is a dict of plain values.  `kind` says which entry points a pass goes through:

  query      KnowledgeBase.query                       batched cosine scoring, optional tag filter, ordered top-k
  draw       KnowledgeBase.query_sampled               the same store, k entries drawn at random by predicted gain
  two_stage  query on the centroids, then query_probe  retrieval from the best matching groups of rows only
  grow       KnowledgeBase, append, normalize, query   a store built up block by block, asked after every block
  quantize   quantize_rows                             rows to e4m3 codes and row scales
  compact    remove, compact_into                      entries dropped, the rest moved into a new store

Sizes: N rows of d elements of type `dtype` (f32, bf16, fp8), Q queries (fp8 with q8, else f32 for f32 rows and bf16
otherwise), k results, `masked`: 64-bit tags and one mask word per query.
"""
from __future__ import annotations

import math

import torch

from paper_2602_14293_amd import kb as kbmod
from paper_2602_14293_amd import workloads as W

DTYPE = {"f32": torch.float32, "bf16": torch.bfloat16, "fp8": torch.float8_e4m3fn}
CODE = {"f32": kbmod.KB_F32, "bf16": kbmod.KB_BF16, "fp8": kbmod.KB_FP8_E4M3}
BYTES = {"f32": 4, "bf16": 2, "fp8": 1}
DEVICE = "cuda"
TEMPERATURE = 0.05
CHUNK = 1 << 17


def listed():
    return [
        # one agent's own store: some thousand float rows, a handful of states asked about; nothing but latency
        dict(name="tiny", kind="query", dtype="f32", N=4096, d=256, Q=8, k=8, masked=False, q8=False),
        # a project's store, one batch of states of a work queue: in between latency and streaming
        dict(name="clustered", kind="query", dtype="bf16", N=65536, d=768, Q=64, k=16, masked=False, q8=False),
        # rows kept in float as an embedding model gives them, a ragged number of them, few queries
        dict(name="float_rows", kind="query", dtype="f32", N=300007, d=384, Q=20, k=10, masked=False, q8=False),
        # one state against a large shared store: the keys are streamed once for a single query
        dict(name="single", kind="query", dtype="bf16", N=1000003, d=1024, Q=1, k=10, masked=True, q8=False),
        # the default workload: a large shared store, a full batch of masked queries
        dict(name="filtered", kind="query", dtype="bf16", N=1 << 20, d=1024, Q=256, k=32, masked=True, q8=False),
        # a store too large for 16 bits, the largest batches
        dict(name="compressed", kind="query", dtype="fp8", N=1 << 22, d=768, Q=1024, k=64, masked=False, q8=False),
        # ... with the queries quantised as well; odd counts
        dict(name="compressed_q8", kind="query", dtype="fp8", N=2500001, d=512, Q=500, k=20, masked=False, q8=True),
        # the weighted random choice of optimizations on the large store
        dict(name="weighted", kind="draw", dtype="bf16", N=1 << 20, d=1024, Q=256, k=32, masked=True, q8=False),
        # states matched first, then the optimizations filed below the best matching ones (N is about C * 1000)
        dict(name="two_stage", kind="two_stage", dtype="bf16", N=1 << 20, C=1024, d=1024, Q=8, k=32, nprobe=4, masked=False, q8=False),
        # the write path: blocks of new entries appended and asked about at once
        dict(name="growing", kind="grow", dtype="bf16", N=65536, blocks=4, d=1024, Q=128, k=16, masked=True, q8=False),
        # building the compressed form of a store
        dict(name="quantize", kind="quantize", dtype="bf16", N=500000, d=768),
        # clearing out a tenth of a store
        dict(name="compact", kind="compact", dtype="bf16", N=500009, d=768, masked=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["query"] * 7 + ["draw", "two_stage", "grow", "quantize", "compact"])
    dtype = rng.choice(["f32", "bf16", "bf16", "fp8"])
    if kind == "quantize":
        return dict(kind=kind, dtype=rng.choice(["f32", "bf16"]), N=_log(rng, 1000, 500000), d=16 * rng.randint(4, 64))
    if kind in ("draw", "two_stage"):
        dtype = "bf16"
    d = 64 * rng.randint(2, 16)
    if kind == "compact":
        return dict(kind=kind, dtype=dtype, N=_log(rng, 3000, 500000), d=d, masked=rng.random() < 0.5)
    k = _log(rng, 1, 128)
    if kind == "two_stage":
        C = _log(rng, 64, 1024)
        return dict(kind=kind, dtype=dtype, N=C * 1024, C=C, d=d, Q=_log(rng, 1, 32), k=k, nprobe=rng.randint(1, 16), masked=False, q8=False)
    if kind == "grow":
        blocks = rng.randint(2, 5)
        return dict(kind=kind, dtype=dtype, N=blocks * _log(rng, 500, 20000), blocks=blocks, d=d, Q=_log(rng, 1, 256), k=k, masked=rng.random() < 0.5, q8=False)
    N = _log(rng, 1000, 1 << (22 if dtype == "fp8" else 20))
    Q = _log(rng, 1, 1024 if dtype == "fp8" else 512)
    # no more work than the largest listed case: float products are an order of magnitude slower than the others
    most = {"f32": 5e10, "bf16": 8e11, "fp8": 1.6e12}[dtype]
    Q = max(1, min(Q, int(most / (N * d))))
    return dict(kind=kind, dtype=dtype, N=N, d=d, Q=Q, k=k, masked=rng.random() < 0.5, q8=dtype == "fp8" and rng.random() < 0.5)


# ---- inputs ----------------------------------------------------------------------------------------------------

def _generator(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    return g


def _rows(case, g):
    """(rows in the storage type, row scale or None): unit centres with noise around them, as the stores of the tests."""
    N, d = case["N"], case["d"]
    centers = W._unit_rows(torch.randn(min(4096, max(16, N // 1024)), d, generator=g, device=DEVICE))
    rows = torch.empty((N, d), dtype=DTYPE[case["dtype"]], device=DEVICE)
    scale = torch.empty(N, device=DEVICE) if case["dtype"] == "fp8" else None
    for s in range(0, N, CHUNK):
        e = min(N, s + CHUNK)
        x, _ = W.clustered_keys(e - s, d, centers.shape[0], 0.1, g, DEVICE, center_rows=centers)
        if scale is None:
            rows[s:e] = x.to(rows.dtype)
        else:
            rows[s:e], scale[s:e] = W.quantize_e4m3_rows(x)
    return rows, scale


def _queries(case, rows, scale, g):
    """Stored rows with noise: the states that a store is asked about resemble states it holds."""
    at = torch.randint(0, rows.shape[0], (case["Q"],), generator=g, device=DEVICE)
    x = rows[at].float()
    if scale is not None:
        x = x * scale[at][:, None]
    x = W.perturbed_queries(x, 0.05, g)
    if case["q8"]:
        return W.quantize_e4m3_rows(x)[0]
    return x.to(torch.float32 if case["dtype"] == "f32" else torch.bfloat16)


def _inputs(case, seed):
    g = _generator(seed)
    kind = case["kind"]
    if kind == "quantize":
        x = torch.randn((case["N"], case["d"]), generator=g, device=DEVICE) * torch.rand((case["N"], 1), generator=g, device=DEVICE)
        return dict(rows=x.to(DTYPE[case["dtype"]]))
    if kind == "two_stage":
        w, cent, offsets = W.grouped(seed, C=case["C"], mean_size=case["N"] // case["C"], d=case["d"], spread=0.03, Q=case["Q"], k=case["k"],
                                     dtype=DTYPE[case["dtype"]], device=DEVICE)
        return dict(rows=w.keys, scale=w.scale, tags=None, qmask=None, queries=w.queries, centroids=cent, offsets=offsets)
    rows, scale = _rows(case, g)
    t = dict(rows=rows, scale=scale, tags=W.random_bits64(case["N"], 0.3, g, DEVICE) if case["masked"] else None)
    if kind == "compact":
        t["gain"] = torch.rand(case["N"], generator=g, device=DEVICE) * 3.75 + 0.25
        t["remove"] = torch.randperm(case["N"], generator=g, device=DEVICE)[: case["N"] // 10].to(torch.int32).contiguous()
        return t
    if kind == "grow":
        per = case["N"] // case["blocks"]
        seen = [dict(rows=rows[: (b + 1) * per], scale=None if scale is None else scale[: (b + 1) * per]) for b in range(case["blocks"])]
        t["queries"] = [_queries(case, s["rows"], s["scale"], g) for s in seen]
        t["qmask"] = [W.random_bits64(case["Q"], 0.3, g, DEVICE) if case["masked"] else None for _ in seen]
        return t
    t["queries"] = _queries(case, rows, scale, g)
    t["qmask"] = W.random_bits64(case["Q"], 0.3, g, DEVICE) if case["masked"] else None
    if kind == "draw":
        t["gain"] = torch.rand(case["N"], generator=g, device=DEVICE) * 3.75 + 0.25
        t["seed"] = seed
    return t


def _store(case, rows, scale, tags):
    kb = kbmod.KnowledgeBase(case["d"], CODE[case["dtype"]], rows.shape[0], tagged=tags is not None, device=DEVICE)
    kb.append(rows, scale, tags)
    kb.normalize()
    return kb


def prepare(case, seed):
    t = _inputs(case, seed)
    t["case"] = case
    if case["kind"] in ("quantize", "grow"):
        return t
    t["kb"] = _store(case, t.pop("rows"), t.pop("scale"), t.pop("tags"))
    if case["kind"] == "two_stage":
        t["centroids"] = _store(case, t["centroids"], None, None)
    return t


# ---- one pass --------------------------------------------------------------------------------------------------

def run(t):
    case = t["case"]
    kind = case["kind"]
    if kind == "query":
        index, score = t["kb"].query(t["queries"], case["k"], t["qmask"])
        return dict(index=index, score=score)
    if kind == "draw":
        index, key = t["kb"].query_sampled(t["queries"], case["k"], t["gain"], TEMPERATURE, t["seed"], t["qmask"])
        return dict(index=index, key=key)
    if kind == "two_stage":
        probe, _ = t["centroids"].query(t["queries"], case["nprobe"])
        index, score = t["kb"].query_probe(t["queries"], case["k"], t["offsets"], probe)
        return dict(probe=probe, index=index, score=score)
    if kind == "grow":
        per = case["N"] // case["blocks"]
        kb = kbmod.KnowledgeBase(case["d"], CODE[case["dtype"]], case["N"], tagged=case["masked"], device=DEVICE)
        out = []
        for b in range(case["blocks"]):
            part = slice(b * per, (b + 1) * per)
            kb.append(t["rows"][part], None if t["scale"] is None else t["scale"][part], None if t["tags"] is None else t["tags"][part])
            kb.normalize()
            out.append(kb.query(t["queries"][b], case["k"], t["qmask"][b]))
        return dict(inv_norm=kb.inv_norm, keys=kb.keys.view(torch.uint8), index=[i for i, _ in out], score=[s for _, s in out])
    if kind == "quantize":
        codes, scale = kbmod.quantize_rows(t["rows"])
        return dict(codes=codes.view(torch.uint8), scale=scale)
    kb = t["kb"]
    kb.remove(t["remove"])
    dst = kbmod.KnowledgeBase(case["d"], CODE[case["dtype"]], case["N"], tagged=case["masked"], device=DEVICE)
    live, index_map, gain = kb.compact_into(dst, t["gain"])
    got = dict(keys=dst.keys[:live].view(torch.uint8), inv_norm=dst.inv_norm[:live], gain=gain, index_map=index_map)
    if case["masked"]:
        got["tags"] = dst.tags[:live]
    return got


# ---- what a pass cannot do without -----------------------------------------------------------------------------

def work(case):
    kind, N, d = case["kind"], case["N"], case["d"]
    row = d * BYTES[case["dtype"]]
    if kind == "quantize":
        return {"bytes": N * (row + d + 4), "flops": 0}
    side = 8 if case["masked"] else 0
    if kind == "compact":
        live = N - N // 10
        scale = 4 if case["dtype"] == "fp8" else 0
        return {"bytes": live * 2 * (row + 4 + 4 + side + scale) + N * 8, "flops": 0}
    Q, k = case["Q"], case["k"]
    batch = Q * (d * (4 if case["dtype"] == "f32" else 1 if case["q8"] else 2) + side + 8 * k)
    if kind == "two_stage":
        probed = min(N, Q * case["nprobe"] * (N // case["C"]))
        return {"bytes": (probed + case["C"]) * (row + 4) + 2 * batch, "flops": 2 * d * Q * (case["C"] + case["nprobe"] * (N // case["C"]))}
    if kind == "grow":
        per, b = N // case["blocks"], case["blocks"]
        asked = per * b * (b + 1) // 2
        return {"bytes": b * per * (2 * (row + side) + 4) + asked * (row + 4 + side) + b * batch, "flops": 2 * Q * d * asked}
    return {"bytes": N * (row + 4 + side + (4 if kind == "draw" else 0)) + batch, "flops": 2 * N * d * Q}


# ---- how far off another correct implementation may be ----------------------------------------------------------

def tolerance(case):
    """About four times what the results are off the same computed in 64 bits.  Scores are 32-bit sums of exact
    products: 1e-7 to 4e-7 off, and up to 2.4e-4 of the listed entries trade places where two scores are closer than
    that.  The fp8 matrix instruction keeps fewer bits of its 64-term sums: 2.8e-6 and 1.5e-3.  What is only moved or
    rounded once is the same in every bit."""
    if case["kind"] in ("quantize", "compact"):
        return "exact"
    if case.get("q8"):
        return {"rel": 1.2e-5, "differ": 0.006}
    return {"rel": 1.6e-6, "differ": 0.001}


# ---- the same in 64 bits ----------------------------------------------------------------------------------------

def _unit64(x):
    x = x.float().double()
    n = x.norm(dim=1, keepdim=True)
    return torch.where(n > 0, x / n, torch.zeros_like(x))


def _noise64(first, n, Q, seed):
    """Gumbel variates of rows first .. first+n (multiples of 4) and queries 0 .. Q: Philox4x32-10 on (row / 4, query, 0, 0)."""
    low = 0xFFFFFFFF
    c0 = torch.arange(first // 4, first // 4 + n // 4, device=DEVICE)[:, None].expand(-1, Q)
    c1 = torch.arange(Q, device=DEVICE)[None, :].expand(n // 4, -1)
    c2, c3 = torch.zeros_like(c0), torch.zeros_like(c0)
    k0, k1 = seed & low, (seed >> 32) & low
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57      # wrap round 2^64; the bits taken below are right all the same
        c0, c1, c2, c3 = ((p1 >> 32) & low) ^ c1 ^ k0, p1 & low, ((p0 >> 32) & low) ^ c3 ^ k1, p0 & low
        k0, k1 = (k0 + 0x9E3779B9) & low, (k1 + 0xBB67AE85) & low
    w = torch.stack([c0, c1, c2, c3], dim=1).reshape(n, Q)
    u = ((w >> 9).double() + 0.5) / 2.0**23
    return -torch.log(-torch.log(u))


def _top64(rows, queries, k, tags=None, qmask=None, value=None, allowed=None):
    """[Q, k] best values, descending, -inf where there are none."""
    q = _unit64(queries)
    best = torch.full((q.shape[0], k), -math.inf, dtype=torch.float64, device=DEVICE)
    step = max(4096, min(CHUNK, (1 << 27) // q.shape[0] // 4096 * 4096))
    for s in range(0, rows.shape[0], step):
        e = min(rows.shape[0], s + step)
        v = _unit64(rows[s:e]) @ q.T
        if value is not None:
            v = value(v, s, e)
        if qmask is not None:
            v.masked_fill_((tags[s:e, None] & qmask[None, :]) == 0, -math.inf)
        if allowed is not None:
            v.masked_fill_(~allowed[s:e], -math.inf)
        best = torch.cat([best, v.T], dim=1).topk(k, dim=1).values
    return best


def exact(case, seed):
    t = _inputs(case, seed)
    kind = case["kind"]
    if kind == "compact":
        return None
    if kind == "quantize":
        return dict(codes=None, scale=t["rows"].float().double().abs().amax(dim=1) / 448.0)
    rows, k = t["rows"], case["k"]
    if kind == "query":
        return dict(index=None, score=_top64(rows, t["queries"], k, t["tags"], t["qmask"]))
    if kind == "draw":
        log_gain = t["gain"].double().log()

        def value(v, s, e):
            n = (e - s + 3) // 4 * 4
            return v / TEMPERATURE + log_gain[s:e, None] + _noise64(s, n, case["Q"], seed)[: e - s]

        return dict(index=None, key=_top64(rows, t["queries"], k, t["tags"], t["qmask"], value=value))
    if kind == "two_stage":
        nprobe, offsets = case["nprobe"], t["offsets"]
        probe = (_unit64(t["centroids"]) @ _unit64(t["queries"]).T).topk(nprobe, dim=0).indices      # [nprobe, Q]
        owner = torch.repeat_interleave(torch.arange(case["C"], device=DEVICE), offsets[1:] - offsets[:-1])
        allowed = (owner[:, None, None] == probe[None]).any(dim=1) if nprobe * case["Q"] <= 128 else torch.stack(
            [torch.isin(owner, probe[:, r]) for r in range(case["Q"])], dim=1)
        return dict(probe=None, index=None, score=_top64(rows, t["queries"], k, allowed=allowed))
    per = case["N"] // case["blocks"]
    inv = torch.cat([1.0 / rows[s:s + CHUNK].float().double().norm(dim=1) for s in range(0, case["N"], CHUNK)])
    score = [_top64(rows[: (b + 1) * per], t["queries"][b], k, None if t["tags"] is None else t["tags"][: (b + 1) * per], t["qmask"][b])
             for b in range(case["blocks"])]
    return dict(inv_norm=inv, keys=None, index=[None] * case["blocks"], score=score)
