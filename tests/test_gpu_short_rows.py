"""Large batches against short rows: the pipelined kernel with rings of three and four chunks, on rows of as few chunks as its rings allow.
The same bits as the tiled kernel, and the oracle."""
import numpy as np
import pytest
import torch

from paper_2602_14293_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    import kb_testlib

    return kb_testlib


# (several items and query blocks a workgroup, a ragged last tile and block; a single item; a row count below one tile)
SHAPES = [(70000 + 3, 700, 16), (40000 + 255, 200, 128), (257, 129, 5), (90, 300, 8)]


@pytest.mark.parametrize("N,Q,k", SHAPES)
@pytest.mark.parametrize("kind,d,config,tiled", [("q8", 128, 27, 8), ("q8", 192, 27, 8), ("q8", 256, 5, 8), ("q8", 320, 5, 8), ("q8", 256, 27, 8),
                                                 ("fp8", 192, 4, 3), ("fp8", 320, 4, 3), ("bf16", 128, 17, 3), ("bf16", 192, 17, 3)])
def test_short_rows_give_the_bits_of_the_tiled_kernel(T, kind, d, config, tiled, N, Q, k):
    if kind == "bf16":
        w = W.filtered(seed=N + d, N=N, d=d, Q=Q, k=k, centers=32)
    else:
        w = W.compressed(seed=N + d, N=N, d=d, Q=Q, k=k, centers=32, fp8_queries=kind == "q8")
        g = torch.Generator().manual_seed(d)
        w.tags = W.random_bits64(N, 0.3, g, "cpu")
        w.qmask = W.random_bits64(Q, 0.3, g, "cpu")
    kb = T.build_kb(w)
    kb.set_tuning("small_path", 0)
    got = {}
    for c in (config, tiled):
        kb.set_tuning("scan_config", c)
        got[c] = T.gpu_query(kb, w)
    assert np.array_equal(got[config][0], got[tiled][0]) and np.array_equal(got[config][1].view(np.uint32), got[tiled][1].view(np.uint32))
    T.check_against_oracle(w, *got[config], label=f"{kind} N={N} d={d} Q={Q}")
    kb.set_tuning("sample_keys", 256)           # another sample
    kb.set_tuning("scan_config", config)
    again = T.gpu_query(kb, w)
    kb.close()
    assert np.array_equal(again[0], got[config][0]) and np.array_equal(again[1].view(np.uint32), got[config][1].view(np.uint32))
