"""The sparse kernels against the oracle, each forced: the one-workgroup-per-row
kernel with either wave count, and the split kernel with its merge ("0") in
every shape it is built in (head groups of 1, 2 and 4 tiles, head dim 128 and
256).  At the edges of their tiles, waves and splits: one slot, a tile less
and more one, a wave's last tile, the largest split and one slot more; head
groups below, at and above one 16-head tile; unused and out-of-range slots, an
empty row, sinks and gates.  The bar is the one of every other sparse layer
(checker.check_out); in the one-workgroup kernel a cache in either format that
holds the same values has to give the same bits, since both take the same
tiles in the same order."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from oracle import hs2_oracle as O
from paper_2609_26368_amd import workloads as W
from tests import checker as CK
from tests.test_gpu_parity import dev_bf16, host_bits, note

pytestmark = pytest.mark.gpu

CASES = [  # slots, G, Hkv, D, C, sink and gate
    (1, 8, 2, 128, 1, False), (15, 1, 2, 128, 3, True), (17, 16, 1, 128, 1, False), (65, 17, 1, 128, 2, True),
    (129, 64, 1, 128, 1, False), (640, 5, 4, 128, 1, True), (2304, 8, 1, 128, 1, True), (2305, 8, 1, 128, 1, True),
    (16, 64, 1, 256, 2, True), (129, 3, 2, 256, 1, False), (2304, 8, 1, 256, 1, True), (2400, 16, 1, 256, 1, False),
    (4096, 1, 8, 128, 16, True), (4097, 1, 8, 128, 16, False),  # 256 rows: the largest split, and one slot more
    (300, 32, 1, 128, 1, False), (97, 33, 1, 128, 2, True), (300, 32, 1, 256, 1, True), (97, 33, 1, 256, 1, False),
]


@pytest.mark.parametrize("waves", ["0", "4", "8"])
@pytest.mark.parametrize("slots,G,Hkv,D,C,extras", CASES, ids=["s%d_g%d_d%d" % (c[0], c[1], c[3]) for c in CASES])
def test_sparse_unit(slots, G, Hkv, D, C, extras, waves, monkeypatch):
    from paper_2609_26368_amd import hs2
    B, L = 2, max(2500, slots + 100)
    w = W.Workload("unit", B, L, C, G * Hkv, Hkv, D, slots, 0, 1, ctx_min=min(L // 2, 2048))
    inp = W.make_inputs(w, seed=7, kv="fp8")
    note(f"[sparse unit] waves {waves} slots {slots} G {G} Hkv {Hkv} D {D} C {C}")
    rng = np.random.default_rng(slots * 131 + G)
    idx = np.full((B, Hkv, C, slots), -1, dtype=np.int32)
    for b in range(B):
        for g in range(Hkv):
            for c in range(C):
                n = min(slots, int(inp.lens[b]))
                idx[b, g, c, :n] = np.sort(rng.choice(int(inp.lens[b]), size=n, replace=False))
                if slots > 16:  # unused slots in the middle, and tokens past the length
                    idx[b, g, c, rng.integers(0, slots, 5)] = -1
                    idx[b, g, c, rng.integers(0, slots, 3)] = int(inp.lens[b]) + 3
    if slots == 640:
        idx[1, 0, 0] = -1  # a row with nothing selected
    sink = rng.standard_normal(G * Hkv).astype(np.float32) if extras else None
    gate = W.normal_bf16((B, C, G * Hkv, D), 7, 99) if extras else None
    # power-of-two scales (exact in bf16) that give the cache about unit variance again: the bar's absolute part
    # is for such values.  Probabilities rounded to bf16 move an output by at most 2^-8 sum p |v| <= 2^-8 max |v|,
    # and max |v| = 448 * 2^-7 = 3.5 makes that 0.014, inside its 2e-2 (at 448 * 2^-2 it would be 0.44)
    ks = np.array([2.0 ** -(6 + g % 2) for g in range(Hkv)], dtype=np.float32)
    vs = np.array([2.0 ** -(7 + g % 2) for g in range(Hkv)], dtype=np.float32)
    ref_idx = np.where(idx >= inp.lens[:, None, None, None], -1, idx)
    ref = O.sparse_attention(inp.q_sa[0], inp.K, inp.V, ref_idx, sink=sink, gate=gate, k_scale=ks, v_scale=vs)

    blk = hs2.HybridBlock(B, C, G * Hkv, Hkv, D, inp.K.shape[2], slots, 0)
    lens, q, didx = torch.from_numpy(inp.lens).cuda(), dev_bf16(inp.q_sa[0]), torch.from_numpy(idx).cuda()
    extra = {"sink": torch.from_numpy(sink).cuda() if extras else None, "gate": dev_bf16(gate) if extras else None}
    K8, V8 = torch.from_numpy(inp.K).cuda(), torch.from_numpy(inp.V).cuda()
    sc = (torch.from_numpy(ks).cuda(), torch.from_numpy(vs).cuda())
    wide = lambda X, s: dev_bf16(W.f32_to_bf16_bits((O.e4m3_to_f64(X) * s[None, :, None, None]).astype(np.float32)))  # noqa: E731
    Kd, Vd = wide(inp.K, ks), wide(inp.V, vs)
    monkeypatch.setenv("HS2_SA_UNIT", waves)
    out8 = blk.sparse(q, K8, V8, lens, didx, kv_scales=sc, **extra)
    out = blk.sparse(q, Kd, Vd, lens, didx, **extra)
    torch.cuda.synchronize()
    CK.check_out(CK.bf16_bits_to_f64(host_bits(out8)), ref, "sparse layer, E4M3 cache")
    CK.check_out(CK.bf16_bits_to_f64(host_bits(out)), ref, "sparse layer, bf16 cache")
    if waves != "0":
        assert torch.equal(out8.view(torch.int16), out.view(torch.int16)), "the same values in a bf16 cache"
    for stream in ("0", "1"):  # the gathers' cache policy changes no result
        monkeypatch.setenv("HS2_SA_STREAM", stream)
        for o, k, v, s in ((out8, K8, V8, sc), (out, Kd, Vd, None)):
            got = blk.sparse(q, k, v, lens, didx, kv_scales=s, **extra)
            torch.cuda.synchronize()
            assert torch.equal(got.view(torch.int16), o.view(torch.int16)), f"gather policy {stream}"


ROUTES = [  # B, Hkv, G, D, kv, slots, whether the split kernel and its merge run
    (32, 8, 64, 128, "bf16", 2176, True), (32, 8, 64, 128, "bf16", 320, False), (16, 8, 64, 128, "bf16", 1152, False),
    (16, 8, 33, 256, "bf16", 2176, True), (16, 8, 64, 128, "fp8", 2176, False), (32, 8, 64, 128, "fp8", 2176, True),
    (32, 8, 17, 256, "bf16", 1152, True), (32, 8, 16, 256, "bf16", 1152, False), (8, 8, 64, 128, "bf16", 2176, False),
]


@pytest.mark.parametrize("B,Hkv,G,D,kv,slots,merged", ROUTES, ids=["b%d_g%d_d%d_%s_s%d" % (r[0], *r[2:6]) for r in ROUTES])
def test_rows_of_many_head_tiles_are_gathered_once(B, Hkv, G, D, kv, slots, merged):
    """More than 16 heads per KV head over many long rows stay with the kernel that gathers a row once for all
    heads: head dim 128, 64 heads, 256 rows of 2176 slots take 175 us with a gather per head tile, 82 without."""
    from paper_2609_26368_amd import hs2
    note(f"[sparse route] B {B} Hkv {Hkv} G {G} D {D} {kv} slots {slots}")
    blk = hs2.HybridBlock(B, 1, G * Hkv, Hkv, D, slots, slots, 0)
    K = torch.randint(0, 64, (B, Hkv, slots, D), device="cuda", dtype=torch.uint8)
    K = K if kv == "fp8" else K.to(torch.bfloat16)
    sc = (torch.ones(Hkv, device="cuda"),) * 2 if kv == "fp8" else None
    q = torch.randn(B, 1, G * Hkv, D, device="cuda").to(torch.bfloat16)
    idx = torch.arange(slots, dtype=torch.int32, device="cuda").expand(B, Hkv, 1, slots).contiguous()
    lens = torch.full((B,), slots, dtype=torch.int32, device="cuda")
    hs2.hs2_timing_enable(True)
    hs2.hs2_timing_reset()
    blk.sparse(q, K, K, lens, idx, kv_scales=sc)
    torch.cuda.synchronize()
    ran = hs2.hs2_timing_read()
    hs2.hs2_timing_enable(False)
    hs2.hs2_timing_reset()
    assert ("sa_combine" in ran) == merged, ran
