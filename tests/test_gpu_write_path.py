"""The write path on both sides of the sizes where its kernels change: rows beyond the caches, rows that share a wavefront,
row scales at the limits of the short division."""
import numpy as np
import pytest
import torch

from oracle import kb_oracle
from paper_2602_14293_amd import kb as kbmod
from paper_2602_14293_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,n,d", [(torch.bfloat16, 45000, 768), (torch.float32, 33000, 528), (torch.bfloat16, 66000, 1040)])
def test_quantize_beyond_the_caches_equals_its_parts(dtype, n, d):
    g = torch.Generator(device="cuda").manual_seed(d)
    x = (torch.randn((n, d), generator=g, device="cuda") * torch.rand((n, 1), generator=g, device="cuda")).to(dtype)
    assert x.numel() * x.element_size() > 64 << 20
    codes, scale = kbmod.quantize_rows(x)
    for s in range(0, n, 10000):
        c, sc = kbmod.quantize_rows(x[s:s + 10000])
        assert torch.equal(c.view(torch.uint8), codes[s:s + 10000].view(torch.uint8)) and torch.equal(sc, scale[s:s + 10000])


@pytest.mark.parametrize("dtype,d", [(torch.float32, 512), (torch.float32, 528), (torch.bfloat16, 1024), (torch.bfloat16, 1040)])
def test_quantize_scales_at_the_limits_of_the_short_division(dtype, d):
    """Rows whose scale runs through 2^-64 .. 2^-56 and 2^56 .. 2^64, with elements down to the smallest codes, zeros of
    either sign among them: bit for bit the oracle's, whichever division a row takes."""
    g = torch.Generator().manual_seed(d)
    exps = list(range(-64, -55)) + [-9, 0, 7] + list(range(56, 65))
    x = torch.randn((len(exps), d), generator=g) * torch.exp2(torch.randint(-18, 1, (len(exps), d), generator=g).float())
    x[:, 0] = 448.0
    x[:, 1], x[:, 2] = 0.0, -0.0
    x = (x * torch.exp2(torch.tensor(exps, dtype=torch.float32))[:, None]).to(dtype)
    codes, scale = kbmod.quantize_rows(x.cuda().contiguous())
    torch.cuda.synchronize()
    o_codes, o_scale = kb_oracle.quantize_rows(W.key_bits(x), kb_oracle.F32 if dtype == torch.float32 else kb_oracle.BF16)
    assert np.array_equal(scale.cpu().numpy(), o_scale) and np.array_equal(codes.view(torch.uint8).cpu().numpy(), o_codes)


@pytest.mark.parametrize("n,d", [(60001, 768), (20001, 768)])
def test_compact_on_both_sides_of_the_cache_size(n, d):
    g = torch.Generator(device="cuda").manual_seed(n)
    rows = torch.randn((n, d), generator=g, device="cuda").to(torch.bfloat16)
    kb = kbmod.KnowledgeBase(d, kbmod.KB_BF16, n)
    kb.append(rows)
    kb.normalize()
    gone = torch.randperm(n, generator=g, device="cuda")[: n // 7].to(torch.int32)
    kb.remove(gone)
    dst = kbmod.KnowledgeBase(d, kbmod.KB_BF16, n)
    live, index_map, _ = kb.compact_into(dst)
    keep = torch.ones(n, dtype=torch.bool, device="cuda")
    keep[gone.long()] = False
    assert live == int(keep.sum()) and torch.equal(dst.keys[:live].view(torch.int16), rows[keep].view(torch.int16))
    assert torch.equal(dst.inv_norm[:live], kb.inv_norm[:n][keep]) and int((index_map >= 0).sum()) == live
    kb.close()
    dst.close()
