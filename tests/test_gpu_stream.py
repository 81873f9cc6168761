"""The scan that keeps up to 64 queries in LDS (whole-store and dense plan): the same bits as the scan pipeline at the sizes where its
tiles, layers and groups change, for every type of keys and queries; the plan with few groups that a call with little memory gets."""
import ctypes

import pytest
import torch

from paper_2602_14293_amd import kb as kbmod
from paper_2602_14293_amd import workloads as W

pytestmark = pytest.mark.gpu


def _store(kind, N, d, Q, k, seed, powers=False):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    rows = torch.randn((N, d), generator=g, device="cuda")
    rows[N // 3: N // 3 + min(40, N - N // 3)] = rows[N // 3].clone()                    # neighbours that tie
    rows[torch.randint(0, N, (min(N, 60),), generator=g, device="cuda")] = rows[N // 2].clone()   # rows far apart that tie
    if N > 4:
        rows[N - 2] = 0
    if powers:
        rows *= torch.exp2(torch.randint(-30, 31, (N, 1), generator=g, device="cuda").float())
    q = rows[torch.randint(0, N, (Q,), generator=g, device="cuda")] + 0.3 * torch.randn((Q, d), generator=g, device="cuda")
    if Q > 2:
        q[1] = rows[N // 3]
        q[2] = 0
    if powers:
        q *= torch.exp2(torch.randint(-30, 31, (Q, 1), generator=g, device="cuda").float())
    q = q.to(torch.float32 if kind == "f32" else torch.bfloat16)
    scale = None
    if kind in ("fp8", "q8"):
        rows, scale = kbmod.quantize_rows(rows)
        if kind == "q8":
            q, _ = kbmod.quantize_rows(q)
    elif kind == "bf16":
        rows = rows.to(torch.bfloat16)
    tags, qmask = W.random_bits64(N, 0.3, g, "cuda"), W.random_bits64(Q, 0.3, g, "cuda")
    code = {"f32": kbmod.KB_F32, "bf16": kbmod.KB_BF16}.get(kind, kbmod.KB_FP8_E4M3)
    kb = kbmod.KnowledgeBase(d, code, N, tagged=True)
    kb.append(rows, scale, tags)
    kb.normalize()
    if N > 10:
        kb.remove(torch.randperm(N, generator=g, device="cuda")[: N // 10].to(torch.int32).contiguous())
    return kb, q.contiguous(), qmask


def _same(a, b, what):
    assert torch.equal(a[0], b[0]) and torch.equal(a[1].view(torch.int32), b[1].view(torch.int32)), what


# rows around tiles of 16 and 32, one and two layers of 2048 tiles, one tile of a third layer, groups of two tiles, the last size that is
# scored whole and the first that is not; one query, a block that is one short, a full one; pieces that end in half a line (fp8)
@pytest.mark.parametrize("kind,N,d,Q,k", [
    ("bf16", 1, 64, 1, 1), ("bf16", 15, 64, 3, 8), ("bf16", 17, 128, 32, 20), ("bf16", 4096, 192, 31, 16), ("bf16", 4097, 64, 32, 5),
    ("bf16", 5000, 1024, 32, 10), ("bf16", 16385, 256, 7, 9), ("bf16", 65535, 64, 32, 12), ("bf16", 65569, 128, 5, 33), ("bf16", 131073, 64, 32, 4),
    ("bf16", 196700, 64, 9, 10), ("bf16", 327681, 64, 32, 16), ("bf16", (1 << 20) - 1, 64, 3, 90), ("bf16", 1 << 20, 64, 3, 90),
    ("bf16", 3000, 2048, 30, 7), ("bf16", 40000, 1536, 32, 7), ("bf16", 9000, 4096, 12, 3), ("bf16", 700, 64, 200, 9),
    ("fp8", 33, 64, 2, 8), ("fp8", 4096, 320, 32, 16), ("fp8", 20000, 64, 32, 8), ("fp8", 70001, 192, 17, 20), ("fp8", 400001, 64, 32, 24), ("fp8", 1000, 960, 100, 3),
    ("q8", 33, 64, 2, 8), ("q8", 4096, 320, 32, 16), ("q8", 20000, 64, 32, 8), ("q8", 70001, 192, 17, 20), ("q8", 400001, 64, 32, 24), ("q8", 1000, 960, 100, 3),
    # two blocks of queries: one of a single query, one that is short, a full one; both ends of the sizes that take them
    ("bf16", 65535, 64, 64, 5), ("bf16", 65536, 512, 33, 5), ("bf16", 131073, 64, 47, 9), ("bf16", 196608, 192, 50, 4), ("bf16", 196609, 704, 64, 3), ("bf16", (1 << 20) - 1, 64, 40, 24),
    ("fp8", 100, 64, 64, 3), ("fp8", 5000, 320, 33, 5), ("fp8", 131073, 64, 63, 9), ("fp8", 30001, 768, 64, 3), ("fp8", 327681, 128, 34, 12), ("fp8", 400001, 704, 64, 30),
    ("q8", 131072, 64, 63, 9), ("q8", 131073, 64, 63, 9), ("q8", 150001, 1344, 64, 3), ("q8", 400001, 256, 41, 30)])
def test_the_bits_of_the_pipeline(kind, N, d, Q, k):
    kb, q, qmask = _store(kind, N, d, Q, k, seed=N + d)
    for mask in (None, qmask):
        kb.set_tuning("small_path", 1)
        got = kb.query(q, k, mask)
        kb.set_tuning("small_path", 0)
        _same(got, kb.query(q, k, mask), f"{kind} N={N} d={d} Q={Q} k={k} masked={mask is not None}")
    kb.close()


# Calls whose scan takes f32 rows as two f16 values an element: the bits of the f32 instruction (a configuration asked for by name keeps to it),
# from the whole-store plan and from the pipeline.  Just as many rows as few queries take, and the most, the longest rows and the largest k, the largest k and
# two query blocks of many, lists of the pipeline; rows whose lengths are powers of two apart.  (The second half: calls under the limits, which keep to the f32 instruction.)
@pytest.mark.parametrize("N,d,Q,k,config", [
    ((1 << 20) - 1, 64, 7, 32, 1), (524300, 96, 32, 20, 1), (164000, 640, 22, 4, 1), (327681, 160, 31, 32, 1), (218500, 480, 9, 32, 1), (105800, 992, 14, 14, 1),
    (70001, 512, 120, 12, 2), (49152, 1024, 128, 124, 2), (49152, 1024, 128, 128, 2), (33000, 512, 256, 128, 3), (40000, 160, 700, 40, 3), (8200, 2048, 257, 9, 3), (400001, 704, 33, 16, 26),
    (78700, 640, 22, 4, 1), (224800, 224, 31, 32, 1), (105000, 480, 9, 32, 1), (51000, 992, 14, 19, 1), (16400, 1024, 256, 124, 3), (16400, 1024, 256, 128, 3), (400001, 352, 33, 16, 26)])
def test_split_f32_rows_have_the_bits_of_the_f32_instruction(N, d, Q, k, config):
    kb, q, qmask = _store("f32", N, d, Q, k, seed=N + d, powers=True)
    for mask in (None, qmask):
        kb.set_tuning("small_path", 1)
        got = kb.query(q, k, mask)
        kb.set_tuning("small_path", 0)
        _same(got, kb.query(q, k, mask), f"pipeline N={N} d={d} Q={Q} k={k} masked={mask is not None}")
        kb.set_tuning("scan_config", config)
        _same(got, kb.query(q, k, mask), f"f32 instruction N={N} d={d} Q={Q} k={k} masked={mask is not None}")
        kb.set_tuning("scan_config", 0)
    kb.close()


# the memory that the plan in groups of 128 rows took is enough for a plan without a sampling pass
@pytest.mark.parametrize("kind,N,d,Q,k", [("bf16", 200001, 64, 20, 10), ("q8", 9000, 64, 8, 4), ("fp8", 327680, 128, 32, 16), ("bf16", 131073, 1024, 32, 8)])
def test_few_groups_where_there_is_little_memory(kind, N, d, Q, k):
    kb, q, qmask = _store(kind, N, d, Q, k, seed=7)
    want = kb.query(q, k, qmask)
    have = 768 + sum((Q * -(-N // 128) * b + 255) // 256 * 256 for b in (4, 16))
    if N <= 16384:
        have = max(have, 768 + Q * 64 * k * 8 + 256)
    L, out = kbmod.lib(), (ctypes.c_int64 * 4)()
    assert L.kb_query_plan(kb._h, N, Q, k, 2 if kind == "q8" else 0, have, out) == 0 and out[0] in (1, 2) and out[1] <= have
    ws = torch.full((have,), 0xA5, dtype=torch.uint8, device="cuda")
    oi, os_ = torch.full_like(want[0], -7), torch.full_like(want[1], float("nan"))
    assert L.kb_query(kb._h, kbmod._ptr(q), kbmod._CODE_OF[q.dtype], Q, kbmod._ptr(qmask), k, kbmod._ptr(oi), kbmod._ptr(os_), kbmod._ptr(ws), have, kbmod._stream()) == 0
    torch.cuda.synchronize()
    _same((oi, os_), want, f"{kind} N={N}")
    kb.close()


# Where the plan without this scan is the faster one (its workgroups are as many as its tiles up to 512, or there is a sampling pass; this scan has
# 256), and the sizes beside: rows of a multiple of 4 KB, of 64 bytes in large stores, few tiles a compute unit
@pytest.mark.parametrize("kind,N,d,Q,workgroups", [
    ("bf16", 48 << 10, 2048, 8, 256), ("bf16", (48 << 10) + 1, 2048, 8, 385), ("fp8", 60000, 4096, 2, 469), ("q8", 60000, 4096, 2, 469), ("bf16", 60000, 3072, 8, 256),
    ("fp8", 1 << 17, 64, 8, 256), ("fp8", (1 << 17) + 1, 64, 8, 512), ("fp8", 327681, 64, 8, 256), ("fp8", 700000, 64, 8, None), ("q8", 150000, 64, 8, 256), ("q8", 700000, 64, 8, None),
    ("bf16", 20000, 1024, 8, 157), ("bf16", 17000, 1024, 8, 256), ("bf16", 17000, 1024, 32, 133), ("bf16", 20000, 768, 8, 256), ("bf16", 33000, 1024, 32, 256),
    ("bf16", 45000, 1536, 32, 352), ("bf16", 38000, 1536, 32, 256), ("bf16", 92000, 1536, 32, 512), ("bf16", 70000, 1536, 32, 256),
    ("fp8", 45000, 1280, 8, 352), ("fp8", 40000, 1280, 8, 256), ("q8", 45000, 1280, 8, 256), ("fp8", 917504, 1024, 32, 256), ("fp8", 917505, 1024, 32, None),
    # two blocks of queries
    ("bf16", 65536, 768, 40, 512), ("bf16", 65537, 768, 40, 256), ("bf16", 65536, 512, 40, 256), ("bf16", 786432, 64, 40, 256), ("bf16", 786433, 64, 40, None),
    ("bf16", 917504, 768, 40, 256), ("bf16", 917505, 768, 40, None), ("fp8", 917505, 128, 40, None), ("q8", 917505, 256, 40, 256), ("bf16", (1 << 20) - 1, 128, 64, 256),
    ("bf16", 1 << 20, 128, 64, None)])
def test_where_the_queries_in_lds_lose(kind, N, d, Q, workgroups):
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    rows, q = torch.randn((N, d), generator=g, device="cuda", dtype=torch.bfloat16), torch.randn((Q, d), generator=g, device="cuda", dtype=torch.bfloat16)
    scale = None
    if kind != "bf16":
        rows, scale = kbmod.quantize_rows(rows)
        q = kbmod.quantize_rows(q)[0] if kind == "q8" else q
    kb = kbmod.KnowledgeBase(d, kbmod.KB_BF16 if kind == "bf16" else kbmod.KB_FP8_E4M3, N)
    kb.append(rows, scale)
    kb.normalize()
    got = kb.query(q, 10)
    said = kb.counters()
    if workgroups is None:
        assert said["sample_keys"] > 0
    else:
        assert said["sample_keys"] == 0 and said["scan_workgroups"] == workgroups
    kb.set_tuning("small_path", 0)
    _same(got, kb.query(q, 10), f"{kind} N={N} d={d} Q={Q}")
    kb.close()
