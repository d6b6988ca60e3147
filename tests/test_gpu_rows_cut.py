"""The one-stream GEMM where the row count decides how many feature blocks a workgroup takes: two and
three row blocks with counts that the host knows and counts that it does not, launches that hold both
forms (K in two parts or not), and two streams whose row count lies on either side of the limit
between it and the many-rows GEMM.  Against the oracle; the tolerance is that of the operand roundings."""
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
    (320, 272, 128, "f16"),    # QKV: 264 blocks, 2 per workgroup up to 6 row tiles, 3 with two row blocks
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
        for reused in ((208, 208), (150, 169), (128, 0), (64, 63), (60, 5)):  # 160, 257, 448, 449, 511 rows
            keep = [rng.permutation(n_vis)[:k].tolist() for k in reused]
            two = synth.round_bf16(two + 0.1 * rng.standard_normal(two.shape))
            got = gm.prefill(two, n_vis, [k + [] for k in keep])
            for b in range(2):
                want = O.sparse_forward(om, two[b], n_vis, caches[b], [keep[b]] * 2)
                alive = ~np.isnan(want["hidden"][:, 0])
                assert np.abs(got["hidden"][b][alive] - want["hidden"][alive]).max() <= TOL[operand], (reused, b)
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
