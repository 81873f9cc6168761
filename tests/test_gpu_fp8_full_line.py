"""The full-line kernel for fp8 keys with bf16 queries against the kernel with 64-byte row pieces: the same bits, and the oracle."""
import numpy as np
import pytest
import torch

from paper_2602_14293_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    import kb_testlib

    return kb_testlib


# (rows of 256: the shortest the kernel takes; 384: an odd number of key pieces; several tiles and query blocks per workgroup, ragged last ones)
@pytest.mark.parametrize("N,d,Q,k", [(17000 + 77, 256, 300, 64), (300, 384, 129, 5), (70000 + 3, 256, 520, 16), (20000 + 255, 640, 256, 128), (9000 + 1, 1024, 700, 1)])
def test_full_line_kernel_gives_the_bits_of_the_pipelined_one(T, N, d, Q, k):
    w = W.compressed(seed=N + d, N=N, d=d, Q=Q, k=k, centers=32)
    kb = T.build_kb(w)
    removed = np.zeros(w.N, dtype=bool)
    removed[7::53] = True
    kb.remove(torch.from_numpy(np.flatnonzero(removed).astype(np.int32)).cuda())
    got = {}
    for config in (22, 4):
        kb.set_tuning("scan_config", config)
        got[config] = T.gpu_query(kb, w)
        assert kb.counters()["exhaustive_queries"] == 0
    assert np.array_equal(got[22][0], got[4][0]) and np.array_equal(got[22][1].view(np.uint32), got[4][1].view(np.uint32))
    T.check_against_oracle(w, *got[22], label=f"fp8 full line N={N} d={d} Q={Q}", removed=removed)
    kb.close()
