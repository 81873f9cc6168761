"""Calls that bring less memory than the fastest plan wants: every plan that fits gives the same bits, down to the least, below which
the call is refused."""
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


def _store(T, dtype, N, d, Q, k):
    if dtype == "f32":
        w = W.clustered(seed=N + d, N=N, d=d, Q=Q, k=k, centers=32)
        w.keys, w.queries = w.keys.float(), w.queries.float()
    elif dtype == "bf16":
        w = W.clustered(seed=N + d, N=N, d=d, Q=Q, k=k, centers=32)
    else:
        w = W.compressed(seed=N + d, N=N, d=d, Q=Q, k=k, centers=32)
        if dtype == "q8":
            w.queries = W.quantize_e4m3_rows(w.queries.float())[0]
    return w, T.build_kb(w)


# (the full-line kernels; the weighted selection, which has one plan; rows too short for their rings; f32 rows scored whole and by the pipeline)
@pytest.mark.parametrize("dtype,N,d,Q,k,draw,steps", [
    ("bf16", 140003, 384, 200, 64, False, 2), ("bf16", 70003, 256, 400, 20, True, 1), ("fp8", 100007, 384, 400, 40, False, 2),
    ("bf16", 300003, 768, 100, 40, False, 2),
    ("bf16", 124776, 128, 271, 71, False, 1), ("fp8", 250000 + 5, 192, 300, 37, False, 2), ("q8", 250000, 128, 370, 72, False, 2),
    ("f32", 116098, 64, 34, 1, False, 2), ("f32", 1929, 64, 116, 3, False, 3), ("f32", 22637, 128, 43, 9, True, 2)])
def test_the_same_bits_from_every_plan_that_fits(T, dtype, N, d, Q, k, draw, steps):
    w, kb = _store(T, dtype, N, d, Q, k)
    L, p = kbmod.lib(), kbmod._ptr
    q, gain = w.queries.cuda().contiguous(), torch.rand(N, device="cuda") + 0.25
    oi, os_ = torch.empty((Q, k), dtype=torch.int32, device="cuda"), torch.empty((Q, k), device="cuda")
    kind = (1 if draw else 0) + (2 if dtype == "q8" else 0)
    told = L.kb_query_plan_bytes(kb._h, N, Q, k, kind)
    ws = torch.empty(told, dtype=torch.uint8, device="cuda")

    def call(have):
        oi.fill_(-7)
        if draw:
            return L.kb_query_sampled(kb._h, p(q), kbmod._CODE_OF[q.dtype], Q, None, k, p(gain), ctypes.c_float(0.1), ctypes.c_uint64(5), 0, p(oi), p(os_), p(ws), have,
                                      kbmod._stream())
        return L.kb_query(kb._h, p(q), kbmod._CODE_OF[q.dtype], Q, None, k, p(oi), p(os_), p(ws), have, kbmod._stream())

    want, have, seen = None, told, 0
    out = (ctypes.c_int64 * 4)()
    while L.kb_query_plan(kb._h, N, Q, k, kind, have, out) == 0:
        need = out[1]
        ws.fill_(0xA5)
        assert call(need) == 0
        torch.cuda.synchronize()
        if want is None:
            want = oi.clone(), os_.clone()
            assert (oi >= 0).all()
        assert torch.equal(oi, want[0]) and torch.equal(os_.view(torch.int32), want[1].view(torch.int32)), (need, out[0])
        seen, have = seen + 1, need - 1
    assert seen >= steps
    assert call(have) == 7                                                          # KB_ERR_WORKSPACE
    torch.cuda.synchronize()
    assert (oi == -7).all()
    kb.close()


def test_static_scratch_takes_large_batches_on_large_stores(T):
    """2^20 x 1024 bf16 rows, 256 queries, k = 64: the plan that scores the sampled rows once wants 32.02 MiB, the array is 32."""
    w = W.filtered(seed=17, N=1 << 20, d=1024, Q=256, k=64, device="cuda")
    kb = T.build_kb(w)
    q, qm = w.queries.cuda().contiguous(), w.qmask.cuda()
    want_i, want_s = kb.query(q, 64, qm)
    oi, os_ = torch.full_like(want_i, -7), torch.full_like(want_s, float("nan"))
    kb.query_static(q, 64, qm, oi, os_)
    torch.cuda.synchronize()
    assert torch.equal(oi, want_i) and torch.equal(os_.view(torch.int32), want_s.view(torch.int32))
    kb.close()
