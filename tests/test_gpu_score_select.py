"""Rows whose scores and selection are one launch (stored logits, a capacity of
at most 16384 tokens), at the edges of that launch: the words each wave scores
(4, 8, 16 of 64 tokens), the last capacity it serves and the first it does
not, several queries per group, a budget above the candidates, candidates past
the LDS list, and the token count from which the full-attention splits are no
longer the short ones (256 tokens for each of 256 items)."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2609_26368_amd import workloads as W
from tests.test_gpu_parity import note, parity_case

pytestmark = pytest.mark.gpu

EDGES = [  # B, ctx, ctx_min, C, Hq, Hkv, D, k, window
    (1, 4096 + 63, 0, 1, 16, 2, 128, 256, 64), (2, 8192 + 65, 8192 - 3, 2, 8, 1, 128, 300, 1),
    (1, 16384, 0, 1, 32, 4, 128, 2048, 128), (1, 16385, 0, 1, 32, 4, 128, 2048, 128), (3, 777, 1, 1, 3, 1, 256, 900, 0),
    (1, 16384, 0, 16, 1, 1, 128, 64, 0),
]


@pytest.mark.parametrize("case", EDGES, ids=["L%d_c%d_g%d" % (e[1], e[3], e[4] // e[5]) for e in EDGES])
def test_score_select_edges(case):
    B, ctx, ctx_min, C, Hq, Hkv, D, k, win = case
    parity_case(W.Workload(f"score_select_{ctx}", B, ctx, C, Hq, Hkv, D, k, win, 1, ctx_min=max(ctx_min, C) if ctx_min else 0),
                seed=41)


@pytest.mark.parametrize("L", [70, 4096, 9000, 16384])
def test_equal_scores_take_the_lowest_tokens(L):
    """Keys of zero give every candidate the same score: all of them tie at the threshold (more than the LDS list
    holds from 4096 on), and the lowest token indices win."""
    from paper_2609_26368_amd import hs2
    note(f"[equal scores] L {L}")
    k, win = 50, 10
    blk = hs2.HybridBlock(1, 1, 8, 2, 128, L, k, win)
    K = torch.zeros(1, 2, L, 128, dtype=torch.bfloat16, device="cuda")
    V = torch.randn(1, 2, L, 128, device="cuda").to(torch.bfloat16)
    q = torch.randn(1, 1, 8, 128, device="cuda").to(torch.bfloat16)
    _, idx = blk.full(q, K, V, torch.tensor([L], dtype=torch.int32, device="cuda"))
    torch.cuda.synchronize()
    want = np.concatenate([np.arange(k), np.arange(L - win, L)])
    assert (idx.cpu().numpy()[0, :, 0] == want).all()
