"""kb_append moves rows, scales and tags in one launch where it can read them, and by copies of the runtime where it cannot."""
import ctypes

import pytest
import torch

from paper_2602_14293_amd import kb as kbmod

pytestmark = pytest.mark.gpu


def _at(t, shift):
    """The same values `shift` elements behind an aligned place."""
    flat = torch.empty(t.numel() + shift, dtype=t.dtype, device="cuda")
    flat[shift:].copy_(t.reshape(-1))
    return flat[shift:].view(t.shape)


# one piece of 16 bytes more and less than the workgroups move, words of scale and tag in the last workgroup; sources that are not aligned for the kernel
@pytest.mark.parametrize("dtype,d", [("f32", 32), ("bf16", 64), ("fp8", 64), ("fp8", 192)])
@pytest.mark.parametrize("n", [1, 3, 127, 128, 255, 257, 4099])
@pytest.mark.parametrize("shift", [0, 1])
def test_what_is_appended_is_there(dtype, d, n, shift):
    g = torch.Generator(device="cuda")
    g.manual_seed(n + d)
    code = {"f32": kbmod.KB_F32, "bf16": kbmod.KB_BF16, "fp8": kbmod.KB_FP8_E4M3}[dtype]
    kb = kbmod.KnowledgeBase(d, code, 3 * n + 5, tagged=True)
    kb.keys.view(torch.uint8).fill_(7)
    rows, scales, tags = [], [], []
    for part in range(3):
        x = torch.randn((n, d), generator=g, device="cuda")
        x = x.to(torch.bfloat16) if dtype == "bf16" else x
        s = None
        if dtype == "fp8":
            x, s = kbmod.quantize_rows(x)
        t = torch.randint(0, 1 << 62, (n,), generator=g, device="cuda")
        assert kb.append(_at(x.view(torch.uint8), shift * 8).view(x.dtype) if shift else x, s if s is None or not shift else _at(s, 1), _at(t, shift)) == part * n
        rows.append(x.view(torch.uint8)), tags.append(t)
        if s is not None:
            scales.append(s)
    kb.normalize()
    torch.cuda.synchronize()
    assert torch.equal(kb.keys.view(torch.uint8)[: 3 * n], torch.cat(rows)) and bool((kb.keys.view(torch.uint8)[3 * n:] == 7).all())
    assert torch.equal(kb.tags[: 3 * n], torch.cat(tags)) and bool((kb.tags[3 * n:] == 0).all())
    if scales:
        assert torch.equal(kb.scale[: 3 * n], torch.cat(scales))
    kb.close()


@pytest.mark.parametrize("d", [64, 384])
def test_append_in_a_graph(d):
    n = 300
    kb = kbmod.KnowledgeBase(d, kbmod.KB_BF16, 2 * n, tagged=True)
    x, t = torch.zeros((n, d), dtype=torch.bfloat16, device="cuda"), torch.zeros(n, dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        kb.append(x, tags=t)
    for again in range(3):
        x.fill_(again + 1)
        t.fill_(again + 11)
        kb.keys.zero_()
        kb.tags.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert bool((kb.keys[:n] == again + 1).all()) and bool((kb.keys[n:] == 0).all())
        assert bool((kb.tags[:n] == again + 11).all()) and bool((kb.tags[n:] == 0).all())
    kb.close()


# the launch takes rows at 16 bytes, scales and tags at their own alignment; rows that lie where they belong already, scales and tags that do not
@pytest.mark.parametrize("n", [1, 255, 257, 4099])
@pytest.mark.parametrize("rows_shift,scale_shift,tag_shift,in_place", [(0, 1, 0, False), (0, 3, 1, False), (0, 0, 1, False), (1, 0, 0, False), (0, 0, 0, True), (0, 1, 1, True)])
def test_each_source_at_its_own_alignment(n, rows_shift, scale_shift, tag_shift, in_place):
    d = 192
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    kb = kbmod.KnowledgeBase(d, kbmod.KB_FP8_E4M3, 2 * n + 3, tagged=True)
    for part in range(2):
        x, s = kbmod.quantize_rows(torch.randn((n, d), generator=g, device="cuda"))
        t = torch.randint(0, 1 << 62, (n,), generator=g, device="cuda")
        at = slice(part * n, (part + 1) * n)
        if in_place:
            kb.keys[at].view(torch.uint8).copy_(x.view(torch.uint8))
        rows = kb.keys[at] if in_place else _at(x.view(torch.uint8), rows_shift * 8).view(x.dtype)
        assert kb.append(rows, _at(s, scale_shift), _at(t, tag_shift)) == part * n
        torch.cuda.synchronize()
        assert torch.equal(kb.keys[at].view(torch.uint8), x.view(torch.uint8)) and torch.equal(kb.scale[at], s) and torch.equal(kb.tags[at], t)
    assert kb.size == 2 * n and bool((kb.tags[2 * n:] == 0).all())
    kb.close()


# an error of the caller's that nobody has asked for yet is not taken for one of the append's, and is still there afterwards
def test_a_pending_error_of_the_caller():
    hip = ctypes.CDLL("libamdhip64.so")
    kb = kbmod.KnowledgeBase(64, kbmod.KB_BF16, 300, tagged=True)
    x, t = torch.ones((300, 64), dtype=torch.bfloat16, device="cuda"), torch.arange(300, device="cuda")
    torch.cuda.synchronize()
    hip.hipGetLastError()
    pending = hip.hipSetDevice(4096)         # no such device
    try:
        assert pending != 0 and hip.hipPeekAtLastError() == pending
        assert kb.append(x, tags=t) == 0 and kb.size == 300
        assert hip.hipPeekAtLastError() == pending
    finally:
        hip.hipGetLastError()
    torch.cuda.synchronize()
    assert torch.equal(kb.keys, x) and torch.equal(kb.tags, t)
    kb.close()
