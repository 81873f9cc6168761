"""Large batches: the main pass of the full-line kernel leaves out the rows that the sampling pass scored, and the threshold kernel
takes the results among those.  The same bits as the tiled kernel, which scores every row, and the oracle."""
import numpy as np
import pytest
import torch

from paper_2602_14293_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    import kb_testlib

    return kb_testlib


def _crowded(w, query, share, seed):
    """`share` of the rows, anywhere in the store, lie close to one query (a third of them are the very same row): several of the best rows
    fall into one group of sampled rows."""
    g = torch.Generator().manual_seed(seed)
    rows = torch.randperm(w.N, generator=g)[: int(share * w.N)]
    base = w.queries[query].float() / w.queries[query].float().norm()
    near = base + 0.02 * torch.randn(len(rows), w.d, generator=g) / w.d ** 0.5
    near[::3] = near[0]
    scale = 448.0 if w.keys.dtype == torch.float8_e4m3fn else 1.0       # (fp8 rows carry their own scale)
    if scale != 1.0:
        near = near / near.abs().amax(1, keepdim=True) * scale
    w.keys[rows] = near.to(w.keys.dtype)


# key type, config of the full-line kernel, config of the tiled kernel, rows, d, queries, k, share of rows near one query, masks
CASES = [
    ("bf16", 18, 3, 40000 + 1, 256, 300, 32, 0.0, True),
    ("bf16", 18, 3, 1 << 16, 512, 256, 128, 0.02, False),       # a power of two: the order of the runs is mixed
    ("bf16", 19, 2, (1 << 16) + 15, 256, 128, 8, 0.05, False),
    ("bf16", 18, 3, 2048, 256, 257, 1, 0.3, False),             # eight tiles, a quarter of them sampled
    ("bf16", 19, 2, 3000 + 255, 512, 100, 16, 0.1, True),
    ("fp8", 22, 3, (1 << 16) + 77, 256, 300, 64, 0.02, False),
    ("fp8", 22, 3, 2300, 384, 200, 16, 0.1, False),
]


@pytest.mark.parametrize("dtype,config,tiled,N,d,Q,k,share,masked", CASES)
def test_the_parts_add_up_to_every_row(T, dtype, config, tiled, N, d, Q, k, share, masked):
    if dtype == "fp8":
        w = W.compressed(seed=N + d, N=N, d=d, Q=Q, k=k, centers=32)
    else:
        w = (W.filtered if masked else W.clustered)(seed=N + d, N=N, d=d, Q=Q, k=k, centers=32)
    if share:
        _crowded(w, Q // 2, share, N)
    kb = T.build_kb(w)
    kb.set_tuning("scan_config", config)
    removed = np.zeros(w.N, dtype=bool)
    for rows in ([], np.arange(5, w.N, 3), np.arange(w.N - 700, w.N)):      # none, a third, the tail
        if len(rows):
            removed[rows] = True
            kb.remove(torch.from_numpy(np.asarray(rows, dtype=np.int32)).cuda())
        got = T.gpu_query(kb, w)
        assert kb.counters()["sample_keys"] > 0
        kb.set_tuning("scan_config", tiled)
        ref = T.gpu_query(kb, w)
        kb.set_tuning("scan_config", config)
        assert np.array_equal(got[0], ref[0]) and np.array_equal(got[1].view(np.uint32), ref[1].view(np.uint32))
        if not share:
            T.check_against_oracle(w, *got, label=f"{dtype} N={N} d={d} Q={Q}", removed=removed)
    kb.close()


@pytest.mark.parametrize("N,Q,k,temperature", [((1 << 16) + 3, 256, 32, 0.02), (1 << 16, 129, 8, 1.0), (2050, 300, 4, 0.1)])
def test_draws_add_up_too(T, N, Q, k, temperature):
    """(The weighted selection scores every row in its main pass: the full-line kernel behind the tiled kernel's sample.)"""
    w = W.clustered(seed=N, N=N, d=256, Q=Q, k=k, centers=32)
    _crowded(w, 3, 0.05, N)
    gain = torch.from_numpy(np.random.default_rng(N).uniform(0.25, 4.0, size=N).astype(np.float32)).cuda()
    gain[::11] = 0
    kb = T.build_kb(w)
    kb.remove(torch.arange(1, N, 5, dtype=torch.int32).cuda())
    got = {}
    for config in (18, 3):
        kb.set_tuning("scan_config", config)
        i, s = kb.query_sampled(w.queries.cuda().contiguous(), k, gain, temperature, 77)
        torch.cuda.synchronize()
        got[config] = i.cpu().numpy(), s.cpu().numpy()
    kb.close()
    assert np.array_equal(got[18][0], got[3][0]) and np.array_equal(got[18][1].view(np.uint32), got[3][1].view(np.uint32))


def test_replays_of_a_graph(T):
    w = W.clustered(seed=9, N=30000 + 9, d=256, Q=300, k=16, centers=32)
    kb = T.build_kb(w)
    kb.set_tuning("scan_config", 18)
    q = w.queries.cuda().contiguous()
    oi, os_ = torch.empty((300, 16), dtype=torch.int32, device="cuda"), torch.empty((300, 16), dtype=torch.float32, device="cuda")
    for _ in range(2):
        kb.query(q, 16, None, oi, os_)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        kb.query(q, 16, None, oi, os_)
    for r in range(4):
        q.copy_(w.queries.roll(r, 0).cuda())
        oi.zero_()
        g.replay()
        torch.cuda.synchronize()
        ri, rs = oi.clone(), os_.clone()
        ei, es = kb.query(q, 16)
        torch.cuda.synchronize()
        assert torch.equal(ri, ei) and torch.equal(rs.view(torch.int32), es.view(torch.int32))
    kb.close()


@pytest.mark.parametrize("config,N", [(18, 20000 + 9), (0, 20000 + 9), (0, 5000)])
@pytest.mark.parametrize("bits", [1, 60])
def test_numbers_that_are_none(T, config, N, bits):
    """Queries and rows with infinities, NaN or lengths past the largest float, masks that let one row in `bits` through: an entry whose score
    is not a number is not listed, whatever stands for its group, and the rest is found."""
    w = W.clustered(seed=N, N=N, d=256, Q=200, k=16, centers=32)
    g = torch.Generator().manual_seed(1)
    rows = torch.randperm(N, generator=g)[: N // 10]
    w.keys[rows[0::3], 3] = float("inf")
    w.keys[rows[1::3], 3] = float("nan")
    w.keys[rows[2::3]] = 0
    w.tags = torch.ones(N, dtype=torch.int64) << torch.randint(0, bits, (N,), generator=g)
    w.qmask = torch.ones(200, dtype=torch.int64) << torch.randint(0, bits, (200,), generator=g)
    w.queries[0] = 0
    w.queries[1, 3] = float("inf")
    w.queries[2, 5] = float("nan")
    w.queries[3] = 3e38
    w.queries[4, 7] = -float("inf")
    kb = T.build_kb(w)
    kb.set_tuning("scan_config", config)
    a = T.gpu_query(kb, w)
    kb.remove(torch.cat((rows[0::3], rows[1::3])).to(torch.int32).cuda())        # what remains has a score for every query but the first five
    kb.set_tuning("scan_config", 3)
    kb.set_tuning("small_path", 0)
    b = T.gpu_query(kb, w)
    kb.close()
    assert not np.isnan(a[1]).any() and not np.isnan(b[1][5:]).any()
    assert np.array_equal(a[0][5:], b[0][5:]) and np.array_equal(a[1][5:].view(np.uint32), b[1][5:].view(np.uint32))


@pytest.mark.parametrize("dtype,config,N,d", [("bf16", 18, 40000 + 1, 256), ("bf16", 19, (1 << 16) + 5, 256), ("fp8", 22, 50000 + 3, 256)])
def test_queries_without_a_length_stay_on_their_lists(T, dtype, config, N, d):
    """A batch filled up with zero rows, whose masks let nothing or little through: no such query scores the whole store.  One past the
    largest length has to, if its mask lets anything through."""
    Q, k = (100 if config == 19 else 200), 16
    w = W.clustered(seed=N, N=N, d=d, Q=Q, k=k, centers=32) if dtype == "bf16" else W.compressed(seed=N, N=N, d=d, Q=Q, k=k, centers=32)
    g = torch.Generator().manual_seed(2)
    w.tags = torch.ones(N, dtype=torch.int64) << torch.randint(0, 8, (N,), generator=g)
    few = torch.randperm(N, generator=g)[:20]
    w.tags[few] = 1 << 62
    w.qmask = torch.full((Q,), 0x3f, dtype=torch.int64)
    w.queries[:40] = 0
    w.qmask[:20] = 0
    w.qmask[20:40] = 1 << 62
    w.queries[40:42, 3] = float("nan")
    w.queries[42, 3] = float("inf")
    w.queries[43] = 3e38
    w.qmask[40], w.qmask[41], w.qmask[42:44] = 0, 1 << 62, 0
    kb = T.build_kb(w)
    kb.set_tuning("scan_config", config)
    got = T.gpu_query(kb, w)
    counters = kb.counters()
    assert counters["sample_keys"] > 0 and counters["exhaustive_queries"] == 0
    assert (got[0][:20] == -1).all() and (got[0][40:44] == -1).all()
    assert np.array_equal(got[0][20:40], np.tile(np.sort(few.numpy())[:k], (20, 1))) and (got[1][20:40] == 0).all()
    kb.set_tuning("scan_config", 3)
    ref = T.gpu_query(kb, w)
    assert np.array_equal(got[0], ref[0]) and np.array_equal(got[1].view(np.uint32), ref[1].view(np.uint32))
    kb.set_tuning("scan_config", config)
    w.qmask[42:44] = 1 << 62
    got = T.gpu_query(kb, w)
    assert kb.counters()["exhaustive_queries"] == 2 and not np.isnan(got[1]).any()
    kb.close()


def test_lists_hold_what_a_sample_in_whole_rounds_lets_through(T):
    """k = 2, a sample rounded down by a fifth: the second best of it scatters by a factor of ten from query to query, and no list runs over."""
    w = W.clustered(seed=7, N=1284972, d=256, Q=850 * 9, k=2, centers=1254, device="cuda")
    kb = T.build_kb(w)
    kb.set_tuning("scan_config", 18)
    for batch in w.queries.split(850):
        kb.query(batch.contiguous(), 2)
        counters = kb.counters()
        assert counters["sample_keys"] > 0 and counters["exhaustive_queries"] == 0
    kb.close()
