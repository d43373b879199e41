"""Many KV heads at once: the merge with a row per slot group (at least 2048
rows of about 8 partials on average, their capacity at most a split per 40
rows), and the full-attention splits sized for several rounds of workgroups
(more than a quarter, or 0.6, of a round's slots in KV heads), ragged down to
the chunk itself, in both cache formats; one long sequence among short ones,
whose rows have about 50 and over a hundred partials, on both sides of that
capacity."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2609_26368_amd import workloads as W
from tests.test_gpu_parity import parity_case

pytestmark = pytest.mark.gpu

SHAPES = [  # B, Hkv, G, C, D, ctx, kv
    (48, 4, 16, 1, 128, 400, "bf16"), (64, 8, 4, 1, 128, 700, "bf16"), (64, 8, 5, 1, 128, 700, "fp8"),
    (64, 8, 16, 2, 128, 300, "bf16"), (40, 4, 3, 6, 256, 300, "bf16"), (65, 3, 8, 8, 128, 200, "fp8"),
    (100, 8, 4, 1, 256, 600, "bf16"),
]


@pytest.mark.parametrize("B,Hkv,G,C,D,ctx,kv", SHAPES, ids=["b%d_kv%d_g%d_c%d_d%d_%s" % (s[:5] + s[6:]) for s in SHAPES])
def test_many_kv_heads(B, Hkv, G, C, D, ctx, kv):
    parity_case(W.Workload("many_heads", B, ctx, C, G * Hkv, Hkv, D, 40, 20, 1, ctx_min=C), seed=51, kv=kv)


@pytest.mark.parametrize("cap", [6500, 8192, 8193, 16384])  # 2048 rows: 8192 tokens are 64 shortest splits
def test_one_long_sequence(cap, monkeypatch):
    lens = np.full(64, 40, dtype=np.int32)
    lens[37] = cap
    monkeypatch.setattr(W, "draw_lengths", lambda w, seed: lens.copy())
    parity_case(W.Workload("one_long", 64, cap, 2, 16, 1, 128, 40, 20, 1), seed=52)


def _fa_us(hs2, blk, q, K, V, lens):
    """Shortest full-attention pass of five calls."""
    lens = torch.tensor(lens, dtype=torch.int32, device="cuda")
    best = float("inf")
    for _ in range(5):
        hs2.hs2_timing_enable(True)
        hs2.hs2_timing_reset()
        blk.full(q, K, V, lens)
        torch.cuda.synchronize()
        best = min(best, 1e3 * hs2.hs2_timing_read()["fa_split"][1])
        hs2.hs2_timing_enable(False)
    hs2.hs2_timing_reset()
    return best


@pytest.mark.parametrize("G,C,D", [(16, 2, 128), (64, 1, 128), (64, 1, 256)])
def test_one_long_sequence_among_as_many_heads_as_slots_is_cut(G, C, D):
    """512 KV heads fill the grid with an item each; one of 8000 tokens among 300 then has to get more than one. Uncut
    it takes 4 to 6.5 times the pass of equal lengths of the same sum (120-265 us), cut 1.7 times."""
    from paper_2609_26368_amd import hs2
    cap, n = 8000, 512
    K = torch.randn(n, 1, cap, D, device="cuda", dtype=torch.bfloat16)
    q = torch.randn(n, C, G, D, device="cuda").to(torch.bfloat16)
    blk = hs2.HybridBlock(n, C, G, 1, D, cap, 40, 20)
    long_one = [300] * n
    long_one[77] = cap
    even = [sum(long_one) // n] * n
    t_even, t_long = _fa_us(hs2, blk, q, K, K, even), _fa_us(hs2, blk, q, K, K, long_one)
    print(f"[one long] G {G} C {C} D {D}: even {t_even:.1f} us, one long {t_long:.1f} us", flush=True)
    assert t_long < 2.5 * t_even


def test_equal_splits_of_a_mebibyte_are_made_longer(monkeypatch):
    """32 KV heads of 32000 tokens, 32 query rows: the balanced split is 2048 tokens, 1 MiB of K and V, and the heads
    lie 15.625 MiB apart; the pass takes splits of 2304 then, so its results are those of that fixed length."""
    from paper_2609_26368_amd import hs2
    B, Hkv, L = 8, 4, 32000
    KV = torch.randn(B, Hkv, L, 256, device="cuda", dtype=torch.bfloat16)
    q = torch.randn(B, 2, 16 * Hkv, 128, device="cuda").to(torch.bfloat16)
    blk = hs2.HybridBlock(B, 2, 16 * Hkv, Hkv, 128, L, 40, 20, kv_strides=(Hkv * L * 256, L * 256, 256))
    lens = torch.full((B,), L, dtype=torch.int32, device="cuda")
    got = []
    for split in ("0", "2304"):
        monkeypatch.setenv("HS2_FA_SPLIT", split)
        stats = torch.empty(B, 2, 16 * Hkv, 2, device="cuda")
        out, idx = blk.full(q, KV[..., :128], KV[..., 128:], lens, stats=stats)
        torch.cuda.synchronize()
        got.append((out.view(torch.int16), idx, stats))
    assert all(torch.equal(a, b) for a, b in zip(*got))
