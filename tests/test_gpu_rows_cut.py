"""The one-stream GEMM where the row count decides how many feature blocks a workgroup takes: two and
three row blocks with counts that the host knows and counts that it does not, K in two parts and whole, and
two streams whose row count lies on either side of the limit between it and the many-rows GEMM, with lists so
short that only the latter is launched and with lists so long that both are.  Against the oracle; the tolerance is that of the operand roundings."""
import numpy as np
import pytest

import synth
from oracle import vlac_oracle as O
from helpers import GpuModel, oracle_model

pytestmark = pytest.mark.gpu
TOL = {"f16": 2e-2, "f16w8": 2e-2, "bf16": 8e-2}


@pytest.mark.parametrize("d,F,hq,operand", [
    (320, 8240, 4, "f16"),     # gate/up: 515 blocks, 3 per workgroup, 5 with two row blocks
    (320, 8240, 4, "bf16"),
    (320, 4400, 4, "f16"),     # gate/up: 275 blocks, pairs with K in two parts or more blocks with K whole
    (320, 272, 128, "f16"),    # QKV: 264 blocks, K in two parts, 2 per workgroup up to 6 row tiles, 3 with two row blocks
    (320, 272, 128, "f16w8"),
])
def test_feature_blocks_by_row_count(d, F, hq, operand):
    cfg = synth.ModelCfg(2, d, hq, 2, 64, F, 96)
    std = 1.0 / np.sqrt(d)
    om = oracle_model(cfg, seed=5, std=std, w8=operand == "f16w8")
    gm = GpuModel(cfg, seed=5, max_batch=2, max_seq=512, std=std, operand=operand)
    rng = np.random.default_rng(d + F + hq)
    try:
        n_vis = 496
        emb = synth.round_bf16(rng.standard_normal((n_vis + 8, d)))
        for L in (192, 257, 289, 384, 385, 449, 504):  # known to the host
            want = O.dense_forward(om, emb[-L:], L - 8, O.new_cache(cfg, 512))
            got = gm.prefill(emb[None, -L:], L - 8)
            assert np.abs(got["hidden"][0] - want["hidden"]).max() <= TOL[operand], L
        # two streams of 288 tokens: 160 to 512 rows in all, counted on the device
        n_vis, two = 280, np.stack([emb[:288], emb[200:488]])
        caches = [O.new_cache(cfg, 512) for _ in range(2)]
        for b in range(2):
            O.dense_forward(om, two[b], n_vis, caches[b])
        gm.prefill(two, n_vis)

        def check(lists, counts):
            nonlocal two
            two = synth.round_bf16(two + 0.1 * rng.standard_normal(two.shape))
            got = gm.prefill(two, n_vis, lists, counts)
            for b in range(2):
                want = O.sparse_forward(om, two[b], n_vis, caches[b], [lists[b][:m] for m in counts[b]])
                alive = ~np.isnan(want["hidden"][:, 0])
                assert np.abs(got["hidden"][b][alive] - want["hidden"][alive]).max() <= TOL[operand], (counts, b)
                assert np.abs(got["attn_mean"][:, b] - want["attn_mean"]).max() <= TOL[operand], (counts, b)

        # lists as long as they are used: 257 rows and more are certain, and only the many-rows GEMM is launched
        for reused in ((150, 150), (128, 0), (64, 63), (60, 5)):  # 276, 448, 449, 511 rows
            assert 2 * (288 - max(reused)) >= 257
            check([rng.permutation(n_vis)[:max(k, 1)].tolist() for k in reused], [[k, k] for k in reused])
        # long lists, used in part: both are launched, and the count says which works (up to 448 rows the one-stream
        # GEMM); its partial rows are added up in its own format, also where the next layer's count is the other's
        assert 2 * (288 - 208) < 257
        lists = [rng.permutation(n_vis)[:208].tolist() for _ in range(2)]
        for first, last in ((160, 160), (256, 256), (257, 257), (288, 288), (384, 384), (385, 385), (447, 447), (448, 448),
                            (449, 449), (450, 450), (512, 512), (449, 448), (450, 257), (512, 160)):
            check(lists, [[(576 - n + b) // 2 for n in (first, last)] for b in range(2)])
    finally:
        gm.close()


@pytest.mark.parametrize("operand", ["f16", "bf16", "f16w8"])
def test_rows_do_not_depend_on_who_counts_them(operand):
    """K and V of the first layer come from the embeddings through QKV alone (264 feature blocks, K in two
    parts), so a full recompute (rows counted by the host) and a pass with reuse lists of which no
    entry is used (the same rows, counted on the device) must leave the same cache bit for bit."""
    import torch
    d, F, hq, n_txt = 320, 272, 128, 8
    cfg = synth.ModelCfg(1, d, hq, 2, 64, F, 96)
    gm = GpuModel(cfg, seed=6, max_batch=1, max_seq=512, std=1.0 / np.sqrt(d), operand=operand)
    rng = np.random.default_rng(7)
    try:
        emb = synth.round_bf16(rng.standard_normal((504, d)))
        # (from 449 rows on a known count of this shape takes K whole, which is the cheaper cut there)
        for L in (64, 192, 193, 224, 257, 288, 289, 352, 384, 385, 448):
            one = emb[None, -L:]
            gm.prefill(one, L - n_txt)
            known = gm.kv.clone()
            gm.prefill(one + np.float32(0.25), L - n_txt)
            assert not torch.equal(gm.kv, known), L
            gm.prefill(one, L - n_txt, [list(range(L // 2))], [[0]])
            assert torch.equal(gm.kv, known), L
    finally:
        gm.close()


def test_rows_do_not_depend_on_how_many_streams_share_a_call():
    """A stream of 256 tokens alone (a capacity of 256 rows: the one-stream GEMM) and beside another one (512
    rows: both GEMMs are launched, the one-stream one works): K of the projections with a residual is split as
    for few rows in either case, so every row must come out the same, bit for bit."""
    d, n_vis, n_txt = 1536, 240, 16
    cfg = synth.ModelCfg(2, d, 12, 2, 128, 8960, 96)
    gm = GpuModel(cfg, seed=6, max_batch=2, max_seq=256, std=1.28 / np.sqrt(d), gen_device="cuda:0")
    rng = np.random.default_rng(9)
    try:
        first = synth.round_bf16(rng.standard_normal((2, n_vis + n_txt, d)))
        then = synth.round_bf16(first + 0.2 * rng.standard_normal(first.shape))
        lists = [rng.permutation(n_vis)[:200].tolist() for _ in range(2)]
        for n in (200, 198, 130):  # 56 to 126 rows a stream (the list's whole length in none but the first)
            out = []
            for B in (1, 2):
                gm.prefill(first, n_vis)
                out.append(gm.prefill(then[:B], n_vis, lists[:B], [[n, n]] * B))
            for k in ("hidden", "logits", "attn_mean"):
                a, b = (o[k][:, :1] if k == "attn_mean" else o[k][:1] for o in out)
                assert np.array_equal(a, b, equal_nan=True), (n, k)
    finally:
        gm.close()
