"""The dense plan (every product written, one workgroup per query selects) and the whole-store plan for more than 128 queries:
against the oracle and, bit for bit, against the scan pipeline (run_and_check runs both)."""
import numpy as np
import pytest
import torch

from oracle import compare, kb_oracle
from paper_2602_14293_amd import kb as kbmod
from paper_2602_14293_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    import kb_testlib

    return kb_testlib


def _work(kind, N, d, Q, k):
    if kind == "f32":
        return W.tiny(seed=N + Q, N=N, d=d, Q=Q, k=k)
    if kind == "bf16":
        return W.clustered(seed=N + Q, N=N, d=d, Q=Q, k=k, centers=max(1, min(64, N // 4)))
    if kind == "bf16m":
        return W.filtered(seed=N + Q, N=N, d=d, Q=Q, k=k, centers=max(1, min(32, N)), p_tag=0.02, single_bit_qmask=True)
    return W.compressed(seed=N + Q, N=N, d=d, Q=Q, k=k, centers=max(1, min(32, N)), fp8_queries=kind == "q8")


# tiles of 16, 32, 64 and 128 rows and their edges, blocks of 16 to 128 queries, 4, 8 and 16 pieces a thread of the selection, the
# first and last row counts of the plan, k beyond the rows, more queries than one block
@pytest.mark.parametrize("kind,N,d,Q,k", [
    ("f32", 1, 32, 1, 1), ("f32", 17, 32, 17, 128), ("f32", 1000, 96, 16, 20), ("f32", 4095, 64, 33, 128), ("f32", 4097, 32, 300, 128), ("f32", 16384, 32, 40, 128),
    ("bf16", 3, 64, 200, 5), ("bf16", 33, 64, 31, 33), ("bf16", 4096, 128, 65, 16), ("bf16", 8193, 64, 300, 128), ("bf16", 16383, 64, 129, 128),
    ("bf16", 16384, 64, 512, 100), ("bf16m", 1023, 64, 130, 12), ("bf16m", 5001, 64, 70, 100), ("fp8", 100, 64, 9, 8), ("fp8", 3001, 192, 20, 64),
    ("fp8", 8192, 64, 200, 128), ("q8", 61, 64, 64, 8), ("q8", 4001, 128, 500, 40), ("q8", 12001, 64, 100, 128)])
def test_dense_shapes(T, kind, N, d, Q, k):
    T.run_and_check(_work(kind, N, d, Q, k), label=f"dense {kind} N={N} d={d} Q={Q} k={k}")


# the whole-store plan: several query blocks, its largest products of rows and queries, k at its limit
@pytest.mark.parametrize("kind,N,d,Q,k", [("bf16", 20001, 64, 129, 16), ("bf16", 65536, 64, 256, 20), ("bf16m", 33001, 64, 300, 24), ("bf16", 16385, 128, 1000, 60),
                                          ("f32", 16385, 32, 64, 60), ("f32", 50001, 32, 200, 16), ("f32", 200001, 32, 50, 10), ("f32", 196608, 64, 64, 33), ("fp8", 30001, 64, 520, 64),
                                          ("q8", 65536, 128, 300, 16)])
def test_whole_store_with_many_queries(T, kind, N, d, Q, k):
    T.run_and_check(_work(kind, N, d, Q, k), label=f"whole {kind} N={N} d={d} Q={Q} k={k}")


@pytest.mark.parametrize("kind", ["bf16", "f32", "fp8", "q8"])
@pytest.mark.parametrize("N,Q,k", [(1, 1, 1), (130, 3, 128), (4096, 33, 16), (9001, 130, 100)])
def test_weighted_selection(T, kind, N, Q, k):
    """The keys of the pipeline, and the oracle's draw; removed rows and rows without gain are never drawn."""
    w = _work(kind, N, 64, Q, k)
    gain = np.random.default_rng(N).uniform(0.25, 4.0, size=N).astype(np.float32)
    gain[3::7] = 0.0
    removed = np.zeros(N, dtype=bool)
    removed[5::11] = True
    kb = T.build_kb(w)
    if removed.any():
        kb.remove(torch.from_numpy(np.flatnonzero(removed).astype(np.int32)).cuda())
    g, q = torch.from_numpy(gain).cuda(), w.queries.cuda().contiguous()
    gi, gk = kb.query_sampled(q, k, g, 0.1, 99, None, 5)
    assert kb.counters()["sample_keys"] == 0
    kb.set_tuning("small_path", 0)
    pi, pk = kb.query_sampled(q, k, g, 0.1, 99, None, 5)
    torch.cuda.synchronize()
    assert torch.equal(gi, pi) and torch.equal(gk, pk)
    keys = kb_oracle.without_removed(kb_oracle.selection_keys(T.oracle_scores(w), gain, 0.1, 99, 5), removed)
    rep, _ = compare.check(gi.cpu().numpy(), gk.cpu().numpy(), keys, k, 2e-4, label=f"draw {kind}", tight_tau=2e-4)
    assert rep.queries == Q
    kb.close()


@pytest.mark.parametrize("N,k", [(16384, 100), (5000, 128), (4096, 8)])
def test_equal_rows_and_removed_rows(T, N, k):
    """Every score ties: the buffer of the selection is cut down again and again, and the lowest live rows win."""
    w = W.clustered(seed=3, N=N, d=64, Q=5, k=k, centers=2)
    w.keys[:] = w.keys[0].clone()
    w.queries[4] = 0
    kb = T.build_kb(w)
    kb.remove(torch.arange(0, 60, 2, dtype=torch.int32).cuda())
    gi, gs = T.gpu_query(kb, w)
    assert gi.tolist() == [[i for i in range(k + 60) if i >= 60 or i % 2][:k]] * 5 and not gs[4].any()
    kb.close()


def test_replays_from_a_graph(T):
    w = W.filtered(seed=8, N=3001, d=128, Q=200, k=40, centers=32)
    kb = T.build_kb(w)
    q, qm = w.queries.cuda().contiguous(), w.qmask.cuda()
    gain = torch.rand(w.N, device="cuda") + 0.25
    for call in (lambda *out: kb.query(q, w.k, qm, *out), lambda *out: kb.query_sampled(q, w.k, gain, 0.1, 3, qm, 0, *out)):
        oi, os_ = torch.empty((w.Q, w.k), dtype=torch.int32, device="cuda"), torch.empty((w.Q, w.k), device="cuda")
        want = call()
        graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=side):
            call(oi, os_)
        for rep in range(3):
            oi.fill_(-7)
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(oi, want[0]) and torch.equal(os_, want[1]), f"replay {rep}"
    kb.close()


@pytest.mark.parametrize("N,Q,k,draw", [(2000, 160, 16, False), (2000, 160, 128, False), (500, 200, 16, False), (3000, 20, 10, True), (16000, 300, 128, False)])
def test_less_memory_than_the_plan_wants(T, N, Q, k, draw):
    """The same bits from whichever plan the memory is enough for; one step below the least, the call is refused."""
    w = W.clustered(seed=N, N=N, d=64, Q=Q, k=k, centers=16)
    kb = T.build_kb(w)
    L = kbmod.lib()
    q, gain = w.queries.cuda().contiguous(), torch.rand(N, device="cuda") + 0.25
    oi, os_ = torch.empty((Q, k), dtype=torch.int32, device="cuda"), torch.empty((Q, k), device="cuda")

    def call(ws, have):
        oi.fill_(-7)
        p = kbmod._ptr
        if draw:
            import ctypes

            return L.kb_query_sampled(kb._h, p(q), kbmod.KB_BF16, Q, None, k, p(gain), ctypes.c_float(0.1), ctypes.c_uint64(5), 0, p(oi), p(os_), p(ws), have, kbmod._stream())
        return L.kb_query(kb._h, p(q), kbmod.KB_BF16, Q, None, k, p(oi), p(os_), p(ws), have, kbmod._stream())

    want = kb.query_sampled(q, k, gain, 0.1, 5) if draw else kb.query(q, k)
    kind = 1 if draw else 0
    told = L.kb_query_plan_bytes(kb._h, N, Q, k, kind)
    kb.set_tuning("small_path", 0)
    pipeline = L.kb_query_plan_bytes(kb._h, N, Q, k, kind)
    kb.set_tuning("small_path", 1)
    most = max(told, pipeline, kb.workspace_bytes(Q, k))
    ws = torch.empty(most, dtype=torch.uint8, device="cuda")
    for have in sorted({told, pipeline, most, max(told, pipeline) - 256}):
        st = call(ws, have)
        torch.cuda.synchronize()
        assert st == (0 if have >= min(told, pipeline) else 7), have
        if st == 0:
            assert torch.equal(oi, want[0]) and torch.equal(os_, want[1]), have
    assert call(ws, 256) == 7
    torch.cuda.synchronize()
    assert (oi == -7).all()
    kb.close()
