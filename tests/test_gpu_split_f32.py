"""Long calls on f32 rows, whose scan takes two f16 values an element: the results of the f32 instruction, bit for bit, where the two kinds of
scores could tell rows apart differently.  (A configuration asked for by name keeps to the f32 instruction.)"""
import pytest
import torch

from paper_2602_14293_amd import kb as kbmod
from paper_2602_14293_amd import workloads as W

pytestmark = pytest.mark.gpu

# the scan with the queries in LDS on both sides of the rows that the tiled kernel's whole-store plan takes (the second: several tiles a group), the tiled kernel's
# tiles of 64 x 64 and 128 x 128 in the whole-store plan, of 128 x 128 and 128 x 256 in the pipeline
SHAPES = [(150001, 704, 20, 1), (330001, 160, 20, 1), (190000, 768, 60, 2), (60001, 640, 120, 2), (400001, 128, 90, 2), (150001, 128, 450, 3)]
PLANS = ["whole", "whole", "whole", "whole", "pipeline", "pipeline"]


def _store(rows, tags=None):
    kb = kbmod.KnowledgeBase(rows.shape[1], kbmod.KB_F32, rows.shape[0], tagged=tags is not None)
    kb.append(rows, None, tags)
    kb.normalize()
    return kb


def _check(kb, q, k, config, qmask=None):
    got = kb.query(q, k, qmask)
    kb.set_tuning("scan_config", config)
    want = kb.query(q, k, qmask)
    kb.set_tuning("scan_config", 0)
    assert torch.equal(got[0], want[0]), f"{int((got[0] != want[0]).sum())} entries of {got[0].numel()} differ"
    assert torch.equal(got[1].view(torch.int32), want[1].view(torch.int32))
    return got


def _rows(N, d, Q, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn((N, d), generator=g, device="cuda"), torch.randn((Q, d), generator=g, device="cuda"), g


@pytest.mark.parametrize("shape,plan", zip(SHAPES, PLANS))
def test_the_plans_that_are_meant(shape, plan):
    N, d, Q, config = shape
    kb = _store(torch.ones((N, d), device="cuda"))
    assert kb.plan(Q, 10)["plan"] == plan
    kb.close()


# `copies` rows that are one vector but for noise, for half of the queries: a handful that straddle the k-th place, more than the first selection has (all
# rows as close are scored again), more than that takes (the f32 instruction decides), copies with no noise at all; noise from where f32 sums tell them apart to where they don't
@pytest.mark.parametrize("copies,noise", [(8, 1e-6), (24, 1e-5), (60, 1e-7), (60, 1e-6), (60, 1e-4), (60, 1e-3), (150, 0.0), (165, 1e-6), (255, 0.0), (258, 0.0), (280, 1e-6), (3000, 1e-6), (3000, 0.0)])
@pytest.mark.parametrize("shape", SHAPES)
def test_rows_that_lie_close(shape, copies, noise):
    N, d, Q, config = shape
    rows, q, g = _rows(N, d, Q, N + copies)
    at = torch.randperm(N, generator=g, device="cuda")[:copies]
    rows[at] = rows[at[0]].clone() * (1.0 + noise * torch.randn((copies, d), generator=g, device="cuda"))
    q[: (Q + 1) // 2] = rows[at[0]] + 0.3 * q[: (Q + 1) // 2]
    tags, qmask = W.random_bits64(N, 0.3, g, "cuda"), W.random_bits64(Q, 0.3, g, "cuda")
    kb = _store(rows, tags)
    for k in (5, 10, 32):
        _check(kb, q, k, config)
    _check(kb, q, 10, config, qmask)
    kb.close()


# the largest k: a pair of rows that f32 sums hardly tell apart at the k-th place of every query
@pytest.mark.parametrize("k", [123, 124, 125, 126, 127, 128])
@pytest.mark.parametrize("N,d,Q,config", [(16400, 1024, 256, 3), (150001, 128, 450, 3), (60001, 640, 120, 2)])
def test_close_rows_at_the_last_place_of_a_large_k(N, d, Q, config, k):
    rows, q, g = _rows(N, d, Q, 11)
    kb = _store(rows)
    kb.set_tuning("scan_config", config)
    index, _ = kb.query(q, k)
    kb.close()
    taken = torch.unique(index)
    free = torch.ones(N, dtype=torch.bool, device="cuda")
    free[taken.long()] = False
    free = free.nonzero()[:, 0]
    last = index[:, k - 1].long()
    rows[free[:Q]] = rows[last] * (1.0 + 1e-6 * torch.randn((Q, d), generator=g, device="cuda"))
    kb = _store(rows)
    _check(kb, q, k, config)
    kb.close()


# Rows whose squared length is past the largest float: their products are finite or overflow, which leaves no number; queries of that kind, and
# zero queries and rows.  Few entries qualify, so these are among the ones selected.
@pytest.mark.parametrize("shape", SHAPES)
def test_lengths_that_are_no_number(shape):
    N, d, Q, config = shape
    rows, q, g = _rows(N, d, Q, 5)
    rows[::2] *= 1e30
    rows[1::4] *= -1.0
    rows[7::500] = 0
    q[1::4] *= 1e30
    q[2::8] = 0
    tags = torch.ones(N, dtype=torch.int64, device="cuda")
    tags[torch.randperm(N, generator=g, device="cuda")[:30]] = 2
    qmask = torch.full((Q,), 2, dtype=torch.int64, device="cuda")
    qmask[::3] = 1
    kb = _store(rows, tags)
    for k in (1, 10, 32):
        got = _check(kb, q, k, config, qmask)
        assert int((got[0][:3] >= 0).sum()) > 0
        _check(kb, q, k, config)
    kb.close()


# Lengths at both ends of what counts as ordinary and beyond: rows alone, queries alone, both
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("row_exp,query_exp", [((-74, -40), (0, 0)), ((55, 63), (0, 0)), ((0, 0), (-74, -40)), ((0, 0), (55, 63)), ((-74, 63), (-74, 63))])
def test_lengths_out_of_the_ordinary(shape, row_exp, query_exp):
    N, d, Q, config = shape
    rows, q, g = _rows(N, d, Q, 6)

    def scaled(x, lo, hi, part):
        x /= x.norm(dim=1, keepdim=True)
        e = torch.randint(lo, hi + 1, (x.shape[0], 1), generator=g, device="cuda").double()
        e[torch.rand(e.shape, generator=g, device="cuda") > part] = 0
        return (x.double() * torch.exp2(e)).float()

    rows, q = scaled(rows, *row_exp, 0.01), scaled(q, *query_exp, 0.5)
    q[0] = rows[17] / rows[17].norm().clamp_min(1e-38)
    kb = _store(rows)
    for k in (1, 10, 32):
        _check(kb, q, k, config)
    kb.close()


# A call that the f32 instruction has to do again, in a graph: replayed on other queries, some of which need it
@pytest.mark.parametrize("shape", SHAPES)
def test_in_a_graph(shape):
    N, d, Q, config = shape
    rows, q, g = _rows(N, d, Q, 9)
    at = torch.randperm(N, generator=g, device="cuda")[:200]
    rows[at] = rows[at[0]].clone()
    close = q.clone()
    close[Q // 2] = rows[at[0]]
    kb = _store(rows)
    now = q.clone()
    index, score = kb.query(now, 10)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        kb.query(now, 10, None, index, score)
    for what in (q, close, q, close):
        now.copy_(what)
        index.fill_(-7)
        score.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        got = (index.clone(), score.clone())
        want = _check(kb, what, 10, config)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    kb.close()


# Less memory than the plan asks for, down to where the call is refused, and the library's own scratch array: the same results
@pytest.mark.parametrize("shape", SHAPES)
def test_with_less_memory(shape):
    N, d, Q, config = shape
    rows, q, g = _rows(N, d, Q, 10)
    at = torch.randperm(N, generator=g, device="cuda")[:60]
    rows[at] = rows[at[0]].clone() * (1.0 + 1e-6 * torch.randn((60, d), generator=g, device="cuda"))
    q[: Q // 2] = rows[at[0]] + 0.3 * q[: Q // 2]
    kb = _store(rows)
    want = _check(kb, q, 10, config)
    served = 0
    have = kb.plan(Q, 10)["bytes"]
    while have > 0:
        ws = torch.full((have,), 0xA5, dtype=torch.uint8, device="cuda")
        index, score = torch.full_like(want[0], -7), torch.full_like(want[1], float("nan"))
        st = kbmod.lib().kb_query(kb._h, kbmod._ptr(q), kbmod.KB_F32, Q, None, 10, kbmod._ptr(index), kbmod._ptr(score), kbmod._ptr(ws), have, kbmod._stream())
        if st == 7:                     # KB_ERR_WORKSPACE
            break
        torch.cuda.synchronize()
        assert st == 0 and torch.equal(index, want[0]) and torch.equal(score, want[1]), have
        served += 1
        have = min(kb.plan(Q, 10, workspace_bytes=have)["bytes"], have) - 1
    assert served >= 1
    index, score = torch.empty_like(want[0]), torch.empty_like(want[1])
    try:
        kb.query_static(q, 10, None, index, score)
    except kbmod.KBError as e:
        assert e.status == 7
    else:
        assert torch.equal(index, want[0]) and torch.equal(score, want[1])
    kb.close()
