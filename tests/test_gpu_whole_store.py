"""The whole-store plan of kb_query (two launches, no sampling pass) at the sizes where it changes its tiles, its groups
and its selection: against the oracle and, bit for bit, against the scan pipeline (run_and_check runs both)."""
import ctypes

import pytest
import torch

from paper_2602_14293_amd import kb as kbmod
from paper_2602_14293_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    import kb_testlib

    return kb_testlib


# one wavefront per workgroup up to 16,384 rows, tiles of 64 / 128 rows; groups of a wave up to 4096 of them, of a tile
# beyond; odd and even numbers of tiles; the fewest rows; query counts at the edges of the blocks of 32, 64 and 128; the eight-wave tiles of longer rows
@pytest.mark.parametrize("kind,N,d,Q,k", [
    ("f32", 1, 32, 1, 1), ("f32", 33, 32, 3, 1), ("f32", 4096, 96, 32, 12), ("f32", 16384, 32, 7, 8), ("f32", 16385, 32, 33, 5),
    ("f32", 131072 + 129, 32, 5, 20), ("bf16", 31, 64, 2, 1), ("bf16", 5000, 128, 32, 10), ("bf16", 16385, 64, 31, 16),
    ("bf16", 65535, 64, 64, 9), ("bf16", 65537, 128, 40, 32), ("bf16", 20000, 64, 65, 16), ("bf16", 40001, 64, 128, 24),
    ("bf16", 140001, 64, 11, 64), ("bf16m", 30001, 64, 20, 12), ("bf16m", 70001, 64, 60, 20), ("bf16m", 33333, 64, 100, 16), ("bf16m", 65537, 512, 90, 20),
    ("fp8", 12000, 64, 9, 8), ("fp8", 50001, 128, 70, 16), ("q8", 9001, 64, 64, 8), ("q8", 30001, 192, 100, 16)])
def test_shapes(T, kind, N, d, Q, k):
    if kind == "f32":
        w = W.tiny(seed=N, N=N, d=d, Q=Q, k=k)
    elif kind == "bf16":
        w = W.clustered(seed=N, N=N, d=d, Q=Q, k=k, centers=max(1, min(64, N // 4)))
    elif kind == "bf16m":
        w = W.filtered(seed=N, N=N, d=d, Q=Q, k=k, centers=32, p_tag=0.02, single_bit_qmask=True)
    else:
        w = W.compressed(seed=N, N=N, d=d, Q=Q, k=k, centers=32, fp8_queries=kind == "q8")
    T.run_and_check(w, label=f"{kind} N={N} d={d} Q={Q} k={k}")


@pytest.mark.parametrize("dtype,C,mean,d,Q,k", [(torch.float32, 20, 500, 64, 8, 10), (torch.bfloat16, 100, 600, 128, 64, 32),
                                                (torch.float8_e4m3fn, 60, 500, 128, 20, 24)])
def test_rows_grouped_by_cluster(T, dtype, C, mean, d, Q, k):
    """Neighbouring rows resemble each other, some in equal copies: groups are scored again, ties go to the lower index."""
    w, _, _ = W.grouped(seed=C, C=C, mean_size=mean, d=d, spread=0.002, Q=Q, k=k, dtype=dtype, p_tag=0.4)
    w.keys[200:400:3] = w.keys[200].clone()
    w.queries[0] = (w.keys[200].float() * (1.0 if w.scale is None else w.scale[200])).to(w.queries.dtype)
    T.run_and_check(w, label=f"grouped {dtype}")


def test_all_rows_alike_and_removed(T):
    """Every group's best ties: the groups are gone through a thousand at a time and the lowest live rows win."""
    w = W.clustered(seed=3, N=90000, d=64, Q=5, k=20, centers=2)
    w.keys[:] = w.keys[0].clone()
    kb = T.build_kb(w)
    gone = torch.arange(0, 60, 2, dtype=torch.int32)
    kb.remove(gone.cuda())
    gi, gs = T.gpu_query(kb, w)
    assert gi.tolist() == [[i for i in range(100) if i >= 60 or i % 2][:20]] * 5 and len(set(gs.ravel().tolist())) == 5
    kb.close()


def _ties(kind, dtype, N, d, Q, g):
    """Stores in which many rows score alike: all equal, 3000 copies of one row among others, one of twenty rows everywhere, the
    same scaled by a factor each (equal but for the rounding), or queries of zeros."""
    def unit(n):
        return torch.nn.functional.normalize(torch.randn((n, d), generator=g, device="cuda"), dim=1)

    rows = unit(1).expand(N, d).clone() if kind == "equal" else unit(N)
    if kind in ("twenty", "scaled"):
        rows = unit(20)[torch.randint(0, 20, (N,), generator=g, device="cuda")]
    if kind == "scaled":
        rows = rows * (torch.rand((N, 1), generator=g, device="cuda") + 0.5)
    asked = torch.randint(0, N, (Q,), generator=g, device="cuda")
    if kind == "copies":
        at = torch.randperm(N, generator=g, device="cuda")[:3000]
        rows[at], asked[:] = rows[at[0]].clone(), at[0]
    queries = rows[asked] + 0.002 * torch.randn((Q, d), generator=g, device="cuda")
    if kind == "zero":
        queries.zero_()
    rows, scale = kbmod.quantize_rows(rows) if dtype == "fp8" else (rows, None)
    bf16, f32 = torch.bfloat16, torch.float32
    return rows.to({"bf16": bf16, "f32": f32}.get(dtype, torch.float8_e4m3fn)), scale, queries.to(f32 if dtype == "f32" else bf16)


@pytest.mark.parametrize("kind,dtype,N,d,Q,k", [
    ("equal", "bf16", 16384, 1024, 8, 8), ("equal", "f32", 16384, 256, 8, 8), ("equal", "bf16", 65536, 256, 40, 16), ("equal", "bf16", 140001, 128, 3, 20),
    ("copies", "bf16", 65536, 768, 64, 16), ("copies", "f32", 100000, 128, 4, 10), ("twenty", "bf16", 65536, 256, 64, 64),
    ("twenty", "bf16", 190000, 512, 100, 16), ("twenty", "fp8", 100000, 512, 16, 16), ("twenty", "f32", 4096, 256, 8, 8),
    ("scaled", "f32", 100000, 256, 20, 10), ("scaled", "f32", 300000, 128, 20, 32), ("scaled", "bf16", 40000, 128, 70, 30), ("zero", "bf16", 65536, 256, 64, 16)])
def test_rows_that_tie_cost_no_more_than_the_pipeline(T, kind, dtype, N, d, Q, k):
    """Same bits as the pipeline, and not slower: only groups with two rows better than the k-th result are scored again.  (A
    half of slack, as both are timed a few times only.)"""
    rows, scale, queries = _ties(kind, dtype, N, d, Q, torch.Generator(device="cuda").manual_seed(N + Q))
    kb = kbmod.KnowledgeBase(d, {"bf16": kbmod.KB_BF16, "f32": kbmod.KB_F32, "fp8": kbmod.KB_FP8_E4M3}[dtype], N)
    kb.append(rows, scale)
    kb.normalize()
    got, took = [], []
    for small_path in (1, 0):
        kb.set_tuning("small_path", small_path)
        got.append(kb.query(queries, k))
        times = []
        for _ in range(9):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            kb.query(queries, k)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b) * 1e3)
        took.append(sorted(times)[4])
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    assert took[0] <= 1.5 * took[1], f"{took[0]:.0f} us, the pipeline {took[1]:.0f}"
    kb.close()


@pytest.mark.parametrize("dtype,N", [(torch.float32, 90000), (torch.bfloat16, 120001)])
@pytest.mark.parametrize("spread,outliers", [(1e-2, (1.0,)), (1e-4, (-1.0,)), (1e-4, (1.0, 0.7)), (3e-6, (1.0, 0.601, -0.5)), (3e-6, (0.999,) * 9)])
def test_scores_in_a_narrow_band(T, dtype, N, spread, outliers):
    """Nearly all scores share a bin of the counting between the lowest and the highest, so the deciding bin is divided again,
    up to three times (an outlier at 1, one just above the band, the band itself).  Its negative gives the lowest of all."""
    g = torch.Generator().manual_seed(N + int(1e7 * spread) + len(outliers))
    q = torch.nn.functional.normalize(torch.randn(64, generator=g, dtype=torch.float64), dim=0)
    cosine = 0.6 + spread * torch.rand(N, generator=g, dtype=torch.float64)
    cosine[torch.randperm(N, generator=g)[: len(outliers)]] = torch.tensor(outliers, dtype=torch.float64)
    other = torch.randn((N, 64), generator=g, dtype=torch.float64)
    other = torch.nn.functional.normalize(other - (other @ q)[:, None] * q, dim=1)
    rows = (cosine[:, None] * q + (1 - cosine**2).clamp(min=0).sqrt()[:, None] * other).to(dtype)
    w = W.Workload("band", rows, torch.stack([q, -q, 3 * q]).to(dtype), 10)
    T.run_and_check(w, label=f"band {dtype} {spread} {outliers}")


def _row_at(tile, tiles, tk, place):
    """Row at a place of a tile: runs of four rows, dealt to the tiles in turn, the tile's run moving on from place to place."""
    per = tk // 4
    j = place % per
    return ((j * tiles + (tile + j * (2 if tiles % 2 else 1)) % tiles) * 4) + place // per


@pytest.mark.parametrize("kind,N,d,Q,tk", [("f32", 140000, 32, 5, 128), ("f32", 140100, 32, 5, 128), ("bf16", 140100, 64, 7, 128), ("bf16", 190001, 64, 70, 64),
                                           ("bf16", 150000, 512, 66, 128), ("fp8", 200001, 64, 9, 128), ("f32", 60000, 32, 5, 128), ("bf16", 60001, 64, 40, 64)])
@pytest.mark.parametrize("alike", ["falling", "equal", "rounding"])
@pytest.mark.parametrize("groups,k", [(1, 10), (5, 40)])
def test_best_rows_in_one_group(T, kind, N, d, Q, tk, alike, groups, k):
    """Seven of each query's best ten rows in one tile, in all four of its parts of 32 places where a group is a tile (more than 4096
    groups of a wave's rows), else in one part: what the scan cannot name is found by scoring the group again.  Their scores fall,
    are equal, or differ by the rounding of a factor only; some are removed, some do not pass the filter.  Five such groups are
    more than a step of the selecting workgroup: it first sees which of them it needs."""
    tiles = -(-N // tk)
    coarse = tiles * (tk // 32) > 4096
    g = torch.Generator().manual_seed(N + Q)
    unit = torch.nn.functional.normalize
    rows, queries = unit(torch.randn((N, d), generator=g), dim=1), unit(torch.randn((Q, d), generator=g), dim=1)
    tags = torch.ones(N, dtype=torch.int64)
    removed = torch.zeros(N, dtype=torch.bool)
    for r in range(Q):
        places = [3, tk - 1, 40, tk // 2 + 5, 31, tk - 30, 17] if coarse else [3, 31, 17, 0, 9, 22, 14]
        at = [_row_at((11 + 13 * r + 1000 * j) % tiles, tiles, tk, place) for j in range(groups) for place in places]
        at = [row for row in at if row < N]             # (a place of the last rows' runs can be past the end)
        for i, row in enumerate(at):
            if alike == "falling":
                rows[row] = queries[r] + 0.05 * (i % 7 + 1) * rows[row]
            else:
                rows[row] = queries[r] * (1.0 if alike == "equal" else 1.0 + 0.37 * i)       # (f32 and bf16 products that differ in the last places, if at all)
        if r % 2:
            removed[at[r % 7]] = True
        if r % 3 == 0:
            tags[at[(r + 2) % 7]] = 2
    rows, scale = kbmod.quantize_rows(rows.cuda()) if kind == "fp8" else (rows, None)
    w = W.Workload("one group", rows.to({"f32": torch.float32, "bf16": torch.bfloat16}.get(kind, torch.float8_e4m3fn)).cpu(),
                   queries.to(torch.float32 if kind == "f32" else torch.bfloat16), k, scale=None if scale is None else scale.cpu(), tags=tags,
                   qmask=torch.ones(Q, dtype=torch.int64))
    kb = T.build_kb(w)
    kb.remove(removed.nonzero()[:, 0].to(torch.int32).cuda())
    gi, gs = T.gpu_query(kb, w)
    assert kb.counters()["sample_keys"] == 0
    T.check_against_oracle(w, gi, gs, label=f"{kind} {alike}", removed=removed.numpy(), min_strict=0.8 if alike == "falling" else None)
    kb.set_tuning("small_path", 0)
    pi, ps = T.gpu_query(kb, w)
    assert (gi == pi).all() and (gs.view("int32") == ps.view("int32")).all()
    kb.close()


def test_replays_from_a_graph(T):
    w = W.filtered(seed=8, N=50001, d=128, Q=24, k=10, centers=32)
    kb = T.build_kb(w)
    q, qm = w.queries.cuda().contiguous(), w.qmask.cuda()
    oi, os_ = torch.empty((w.Q, w.k), dtype=torch.int32, device="cuda"), torch.empty((w.Q, w.k), device="cuda")
    want = kb.query(q, w.k, qm)
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        kb.query(q, w.k, qm, oi, os_)
    for rep in range(3):
        oi.fill_(-7)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(oi, want[0]) and torch.equal(os_, want[1]), f"replay {rep}"
    kb.close()


def test_a_workspace_that_only_the_pipeline_fits_into(T):
    w = W.clustered(seed=5, N=100000, d=128, Q=128, k=10, centers=64)
    kb = T.build_kb(w)
    L = kbmod.lib()
    q = w.queries.cuda().contiguous()
    want = kb.query(q, w.k)
    whole = L.kb_query_plan_bytes(kb._h, kb.size, w.Q, w.k, 0)
    kb.set_tuning("small_path", 0)
    pipeline = L.kb_query_plan_bytes(kb._h, kb.size, w.Q, w.k, 0)
    kb.set_tuning("small_path", 1)
    assert pipeline < whole                          # or the sizes below say nothing
    ws = torch.empty(whole, dtype=torch.uint8, device="cuda")
    oi, os_ = torch.empty((w.Q, w.k), dtype=torch.int32, device="cuda"), torch.empty((w.Q, w.k), device="cuda")
    counters = (ctypes.c_int64 * 4)()
    for have, sampled in ((whole, False), (whole - 256, True), (pipeline, True)):
        oi.fill_(-7)
        assert L.kb_query(kb._h, kbmod._ptr(q), kbmod.KB_BF16, w.Q, None, w.k, kbmod._ptr(oi), kbmod._ptr(os_), kbmod._ptr(ws), have, kbmod._stream()) == 0
        assert L.kb_query_counters(kb._h, kbmod._ptr(ws), counters, kbmod._stream()) == 0        # (synchronises)
        assert (counters[2] > 0) == sampled, have
        assert torch.equal(oi, want[0]) and torch.equal(os_, want[1])
    oi.fill_(-7)
    for have in (pipeline - 256, 256):
        assert L.kb_query(kb._h, kbmod._ptr(q), kbmod.KB_BF16, w.Q, None, w.k, kbmod._ptr(oi), kbmod._ptr(os_), kbmod._ptr(ws), have, kbmod._stream()) == 7
    torch.cuda.synchronize()
    assert (oi == -7).all()
    kb.close()


def test_a_store_scored_in_parts_takes_the_lists_it_was_told(T):
    w = W.tiny(seed=6, N=128, d=64, Q=1000, k=128)
    kb = T.build_kb(w)
    L = kbmod.lib()
    q = w.queries.cuda().contiguous()
    want = kb.query(q, w.k)
    need = L.kb_query_plan_bytes(kb._h, kb.size, w.Q, w.k, 0)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    oi, os_ = torch.empty((w.Q, w.k), dtype=torch.int32, device="cuda"), torch.empty((w.Q, w.k), device="cuda")
    for have, status in ((need - 256, 7), (need, 0)):
        assert L.kb_query(kb._h, kbmod._ptr(q), kbmod.KB_F32, w.Q, None, w.k, kbmod._ptr(oi), kbmod._ptr(os_), kbmod._ptr(ws), have, kbmod._stream()) == status
    torch.cuda.synchronize()
    assert torch.equal(oi, want[0]) and torch.equal(os_, want[1])
    T.check_against_oracle(w, oi.cpu().numpy(), os_.cpu().numpy(), label="parts")
    kb.close()


@pytest.mark.parametrize("kind,d,Q", [("bf16", 1024, 5), ("bf16", 1024, 70), ("bf16", 1024, 200), ("f32", 512, 3), ("fp8", 1024, 7),
                                      ("q8", 1024, 30), ("fp8", 1088, 2)])
def test_stores_beyond_the_infinity_cache(T, kind, d, Q):
    """Just over 320 MiB of keys: the loads' policy has changed for every batch and fp8 rows of a multiple of 128 bytes go a line at
    a time.  Checked against a plain product in double precision."""
    N = (320 << 20) // (d * {"bf16": 2, "f32": 4}.get(kind, 1)) + 77
    g = torch.Generator(device="cuda").manual_seed(d + Q)
    rows = torch.randn((N, d), generator=g, device="cuda")
    scale = None
    if kind in ("fp8", "q8"):
        rows, scale = kbmod.quantize_rows(rows)
    rows = rows.to({"bf16": torch.bfloat16, "f32": torch.float32}.get(kind, torch.float8_e4m3fn))
    queries = torch.randn((Q, d), generator=g, device="cuda")
    queries = queries if kind == "f32" else kbmod.quantize_rows(queries)[0] if kind == "q8" else queries.to(torch.bfloat16)
    kb = kbmod.KnowledgeBase(d, {"bf16": kbmod.KB_BF16, "f32": kbmod.KB_F32}.get(kind, kbmod.KB_FP8_E4M3), N)
    kb.append(rows, scale)
    kb.normalize()
    gi, gs = kb.query(queries, 6)
    kb.set_tuning("small_path", 0)
    pi, ps = kb.query(queries, 6)
    q = torch.nn.functional.normalize(queries.float().double(), dim=1)
    best = torch.cat([torch.nn.functional.normalize(rows[s:s + 65536].float().double(), dim=1) @ q.T for s in range(0, N, 65536)])
    want = best.topk(6, dim=0)
    torch.cuda.synchronize()
    assert torch.equal(gi, pi) and torch.equal(gs, ps)
    assert (gs.double() - want.values.T).abs().max() < (1e-4 if kind == "q8" else 1e-5)       # the tolerances of kb_testlib
    got = best.gather(0, gi.T.long())
    assert (got - want.values).abs().max() < (1e-4 if kind == "q8" else 1e-5)
    kb.close()
